// relres_md.hip -- gfx950 kernels of the molecular model around the RelRes
// pair potential (Sec. 3.2 of the paper): bonded terms, scaled 1-4 pairs and
// a Nose-Hoover velocity-Verlet integrator.
//
// Bonded terms: a block owns a range of consecutive atoms and evaluates every
// term that touches them once in FP64, waves of one term kind; each atom then
// adds its terms' forces from LDS in a fixed order.  In a dynamics step the
// drift is part of the same kernel, and the force launch that follows gives the
// half kick.  A term's energy and virial are counted by
// the block that owns its first atom (a 1-4 pair's by halves).  No atomics, so
// results are deterministic.  Formulas
// (forces are -dE/dx):
//   bond      E = K (r - r0)^2, d = x_i - x_j: F_i = -2K (r - r0) d / r
//   angle     E = K (theta - theta0)^2, a = x_i - x_j, b = x_k - x_j:
//             F_i = (dE/dtheta / sin theta)(b/|b| - cos(theta) a/|a|)/|a|,
//             F_k likewise with a and b exchanged, F_j = -F_i - F_k
//   dihedral  E = K (1 + cos(n phi - d)), b1 = x_j - x_i, b2 = x_k - x_j,
//             b3 = x_l - x_k, m = b1 x b2, n = b2 x b3,
//             phi = atan2(|b2| b1.n, m.n); p = b1.b2/|b2|^2, q = b3.b2/|b2|^2;
//             dphi/dx_i = -|b2| m/|m|^2, dphi/dx_l = |b2| n/|n|^2,
//             dphi/dx_j = -(1 + p) dphi/dx_i + q dphi/dx_l,
//             dphi/dx_k = p dphi/dx_i - (1 + q) dphi/dx_l
// (the gradient of phi as in Blondel and Karplus, J. Comput. Chem. 17, 1132
// (1996)).  1-4 pairs: the pair potential of Eq. 20 of the pair (FG and CG
// parts, the pair's own distances) times the 1-4 factor.
#include "relres_internal.h"
#include "relres_pair.h"
#include "relres_lanes.h"

namespace relres {
namespace {

constexpr int kMdBlock = 256;

// d = x_a - x_b with the single-shift minimum image, from positions already
// read.  The shift is taken by selects (both shifted values computed), so the
// same roundings as subtracting or adding the box under a branch.
__device__ __forceinline__ void mi_diff(const double xa[3], const double xb[3],
                                        const double box[3], double d[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double v = xa[k] - xb[k];
        const double h = 0.5 * box[k];
        const double lo = v - box[k], hi = v + box[k];
        d[k] = v > h ? lo : (v < -h ? hi : v);
    }
}

__device__ __forceinline__ double dot3(const double* a, const double* b)
{
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

__device__ __forceinline__ void cross3(const double* a, const double* b, double* c)
{
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ void add_virial(double* w, const double* lever, const double* f)
{
    w[0] += lever[0] * f[0];
    w[1] += lever[1] * f[1];
    w[2] += lever[2] * f[2];
    w[3] += lever[0] * f[1];
    w[4] += lever[0] * f[2];
    w[5] += lever[1] * f[2];
}

// Fixed-order sum over the block (kMdBlock threads) of v[0..K): the result
// lands in threads 0..K-1 (component threadIdx.x).  Lane moves within each
// wave (the K chains interleaved), then the waves' sums through LDS: two
// block barriers, where a tree through LDS takes one per halving.
template <int K>
__device__ __forceinline__ double block_sum(const double* v, double (*red)[kMdBlock / 64])
{
    double s[K];
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = v[k];
    wave_sums(s);                      // complete in lane 63
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    if (lane == 63) {
#pragma unroll
        for (int k = 0; k < K; ++k) red[k][w] = s[k];
    }
    __syncthreads();
    double r = 0.0;
    if ((int)threadIdx.x < K)
        for (int q = 0; q < kMdBlock / 64; ++q) r += red[threadIdx.x][q];
    __syncthreads();
    return r;
}

// The forces of one term on its atoms at x, f[slot]; with `own` the term's
// energy and virial are added to acc (energies 0..3, virial 4..9).
__device__ __forceinline__ void bond_force(const BondedArgs& b, const double par[4],
                                           const double x[4][3], bool own, double f[4][3],
                                           double acc[10])
{
    double d[3];
    mi_diff(x[0], x[1], b.box, d);
    const double r = sqrt(dot3(d, d));
    const double dr = r - par[1];
    const double sc = -2.0 * par[0] * dr / r;
    for (int c = 0; c < 3; ++c) {
        f[0][c] = sc * d[c];
        f[1][c] = -f[0][c];
    }
    if (own) {
        acc[0] += par[0] * dr * dr;
        add_virial(acc + 4, d, f[0]);
    }
}

__device__ __forceinline__ void angle_force(const BondedArgs& b, const double par[4],
                                            const double x[4][3], bool own, double f[4][3],
                                            double acc[10])
{
    double u[3], v[3];
    mi_diff(x[0], x[1], b.box, u);
    mi_diff(x[2], x[1], b.box, v);
    // reciprocals once: a divide is a long instruction sequence in FP64
    const double ilu = 1.0 / sqrt(dot3(u, u)), ilv = 1.0 / sqrt(dot3(v, v));
    double c = dot3(u, v) * ilu * ilv;
    c = c > 1.0 ? 1.0 : (c < -1.0 ? -1.0 : c);
    const double th = acos(c);
    const double dth = th - par[1];
    const double g = 2.0 * par[0] * dth / sqrt((1.0 - c) * (1.0 + c));   // sin theta
    for (int q = 0; q < 3; ++q) {
        f[0][q] = g * (v[q] * ilv - c * u[q] * ilu) * ilu;
        f[2][q] = g * (u[q] * ilu - c * v[q] * ilv) * ilv;
        f[1][q] = -f[0][q] - f[2][q];
    }
    if (own) {
        acc[1] += par[0] * dth * dth;
        add_virial(acc + 4, u, f[0]);
        add_virial(acc + 4, v, f[2]);
    }
}

// par: K, n, cos d, sin d
__device__ __forceinline__ void dihedral_force(const BondedArgs& b, const double par[4],
                                               const double x[4][3], bool own, double f[4][3],
                                               double acc[10])
{
    double b1[3], b2[3], b3[3], m[3], nn[3];
    mi_diff(x[1], x[0], b.box, b1);
    mi_diff(x[2], x[1], b.box, b2);
    mi_diff(x[3], x[2], b.box, b3);
    cross3(b1, b2, m);
    cross3(b2, b3, nn);
    const double lb2 = sqrt(dot3(b2, b2));
    // phi = atan2(y, x) without the library calls: cos phi = x / r,
    // sin phi = y / r (r = |m||n|), cos and sin of n phi by repeated
    // angle addition, then of n phi - d with cos d, sin d from the host
    const double cx = dot3(m, nn), y = lb2 * dot3(b1, nn);
    const double ir = 1.0 / sqrt(cx * cx + y * y);
    const double cp = cx * ir, sp = y * ir;
    double cn = 1.0, sn = 0.0;
    for (int k = 0; k < (int)par[1]; ++k) {
        const double c2 = cn * cp - sn * sp;
        sn = sn * cp + cn * sp;
        cn = c2;
    }
    const double cos_arg = cn * par[2] + sn * par[3];
    const double sin_arg = sn * par[2] - cn * par[3];
    const double dE = -par[0] * par[1] * sin_arg;
    const double imm = lb2 / dot3(m, m), in2 = lb2 / dot3(nn, nn);
    const double ib2 = 1.0 / (lb2 * lb2);
    const double p = dot3(b1, b2) * ib2, q = dot3(b3, b2) * ib2;
    for (int c = 0; c < 3; ++c) {
        const double gi = -m[c] * imm, gl = nn[c] * in2;
        f[0][c] = -dE * gi;
        f[3][c] = -dE * gl;
        f[1][c] = -dE * (-(1.0 + p) * gi + q * gl);
        f[2][c] = -dE * (p * gi - (1.0 + q) * gl);
    }
    if (own) {
        acc[2] += par[0] * (1.0 + cos_arg);
        const double li[3] = {-b1[0], -b1[1], -b1[2]};
        const double ll[3] = {b2[0] + b3[0], b2[1] + b3[1], b2[2] + b3[2]};
        add_virial(acc + 4, li, f[0]);
        add_virial(acc + 4, b2, f[2]);
        add_virial(acc + 4, ll, f[3]);
    }
}

// The scaled 1-4 pair through Eq. 20 (FG and CG parts, the pair's own
// distances), type-pair index pi; half of its energy and virial for each of
// its atoms that the block owns (share = 0.5 or 1).
__device__ __forceinline__ void pair14_force(const BondedArgs& b, int pi, const double x[4][3],
                                             double share, double f[4][3], double acc[10])
{
    double d[3];
    mi_diff(x[0], x[1], b.box, d);
    const double r2 = dot3(d, d);
    const Cutoffs<double>& cut = b.pcut64[pi];
    double fp = 0.0, en = 0.0;
    if (r2 < cut.rso2) {
        double f1, e1;
        fg_term<MathF64<2>>(b.coef64[pi], cut, r2, f1, e1);
        fp += f1;
        en += e1;
    }
    if (r2 < cut.rco2) {
        double f2, e2;
        cg_term<MathF64<2>>(b.coef64[pi], cut, r2, f2, e2);
        fp += f2;
        en += e2;
    }
    const double s = b.scale14 * fp;           // F_0 = s (x_0 - x_1)
    for (int c = 0; c < 3; ++c) {
        f[0][c] = s * d[c];
        f[1][c] = -f[0][c];
    }
    acc[3] += share * b.scale14 * en;
    const double hd[3] = {share * d[0], share * d[1], share * d[2]};
    add_virial(acc + 4, hd, f[0]);
}

// What thread tid of a bonded block reads first: its first term.
__device__ __forceinline__ void first_term(const BondedArgs& b, const BondPass& ps, BondTerm& it,
                                           double4& par)
{
    const int tid = (int)threadIdx.x;
    it.kind = -1;
    par = make_double4(0.0, 0.0, 0.0, 0.0);
    if (tid < ps.nterms) {
        it = b.terms[ps.term0 + tid];
        par = b.term_par[ps.term0 + tid];
    }
}

// Force slots of an atom that one thread adds up; more are left to its wave (an
// atom of 128 bonds: the launch 9.6 us by one thread, 4.0 by its wave; of 512
// 29.2 and 5.0, of 4000 211 and 19).
constexpr int kHubSlots = 32;

// The bonded forces on the block's atoms at the positions in lpos (thread tid:
// atom bb.atom0 + tid, its force in fa), it and par being the thread's first
// term.  Thread t evaluates the block's terms t, t + 256, ..., which the host
// has grouped so that a wave holds terms of one kind, and leaves each owned
// atom's force in that atom's slots in LDS; then one thread per atom adds its
// slots in order.  Without Cross every atom of every term is the block's own.
template <bool Sums, bool Cross>
__device__ __forceinline__ void bonded_forces(const BondedArgs& b, const BondBlock& bb, double* lpos,
                                              double* lf, BondTerm it, double4 par, double fa[3],
                                              double acc[10])
{
    const int tid = (int)threadIdx.x;
    BondPass ps = bb.pass;
    __syncthreads();
    for (int p = 0; ps.nterms > 0; ++p) {
        for (int t = tid; t < ps.nterms; t += kMdBlock) {
            if (p > 0 || t > tid) {
                it = b.terms[ps.term0 + t];
                par = b.term_par[ps.term0 + t];
            }
            if (it.kind < 0) continue;
            // positions: an owned atom's from LDS, another block's from memory
            double x[4][3];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int c = 0; c < 3; ++c) x[q][c] = lpos[c * b.max_atoms + max(it.atom[q], 0)];
            if (Cross && (it.atom[0] | it.atom[1] | it.atom[2] | it.atom[3]) < 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (it.atom[q] < 0)
                        for (int c = 0; c < 3; ++c) x[q][c] = b.pos[3 * (size_t)~it.atom[q] + c];
            }
            const double pr[4] = {par.x, par.y, par.z, par.w};
            const bool own = Sums && it.atom[0] >= 0;
            double f[4][3] = {};
            if (it.kind == 0) bond_force(b, pr, x, own, f, acc);
            else if (it.kind == 1) angle_force(b, pr, x, own, f, acc);
            else if (it.kind == 2) dihedral_force(b, pr, x, own, f, acc);
            else pair14_force(b, it.pair, x, Sums ? (it.atom[0] >= 0 ? 0.5 : 0.0) +
                                                   (it.atom[1] >= 0 ? 0.5 : 0.0) : 0.0, f, acc);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (it.slot[q] == kNoSlot) continue;
#pragma unroll
                for (int c = 0; c < 3; ++c) lf[c * b.max_slots + it.slot[q]] = f[q][c];
            }
        }
        __syncthreads();
        int s0 = 0, s1 = 0;
        if (tid < bb.natoms) {
            s0 = b.atom_slot[ps.slot0 + tid];
            s1 = b.atom_slot[ps.slot0 + tid + 1];
        }
        // an atom of many terms is summed by its wave, afterwards
        const bool hub = s1 - s0 > kHubSlots;
        const int end = hub ? s0 : s1;
        for (int k = s0; k < end; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) fa[c] += lf[c * b.max_slots + k];
        for (uint64_t hubs = __ballot(hub); hubs != 0ull; hubs &= hubs - 1) {
            const int l = __ffsll((long long)hubs) - 1, lane = tid & 63;
            const int k1 = __shfl(s1, l);
            double v[3] = {0.0, 0.0, 0.0};
            for (int k = __shfl(s0, l) + lane; k < k1; k += 64)
#pragma unroll
                for (int c = 0; c < 3; ++c) v[c] += lf[c * b.max_slots + k];
            wave_sums(v);                  // complete in lane 63
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double t = __shfl(v[c], 63);
                if (lane == l) fa[c] += t;
            }
        }
        if (p >= bb.nmore) break;
        ps = b.passes[bb.more0 + p];
        __syncthreads();               // the slots are used again
    }
}

// Bonded and 1-4 forces, one block per range of consecutive atoms
// (BondBlock), whose positions are staged in LDS.  Every term
// is evaluated once per block that owns an atom of it, so once for molecules
// that do not straddle blocks, by waves that take one branch: bound by the
// dependent reads (term, then position) and the arithmetic of one term.
// (One lane per atom and term, the version
// before, evaluated each term two to four times in waves of all four kinds:
// 48000-atom hexane 29.8 us in the kernel trace, so 7.4; 6000 atoms 8.0 and
// 4.7, the launch and three dependent memory round trips.)
// With Sums every block writes its 10 sums to b.partial (energies: bonds,
// angles, dihedrals, 1-4; virial).  No atomics, so results are deterministic.
template <typename TF, bool Sums>
__global__ __launch_bounds__(kMdBlock) void k_bonded(BondedArgs b)
{
    extern __shared__ double lds[];
    __shared__ double red[Sums ? 10 : 1][kMdBlock / 64];
    double* lpos = lds;                                  // [3][max_atoms]
    double* lf = lds + 3 * b.max_atoms;                  // [3][max_slots]
    const BondBlock bb = b.blocks[blockIdx.x];
    const int tid = (int)threadIdx.x;
    const int a = bb.atom0 + tid;
    const bool live = tid < bb.natoms;                   // this thread's atom
    double acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    double fa[3] = {0.0, 0.0, 0.0};
    // the first term and the atom's own data: none of these reads waits on another
    BondTerm it;
    double4 par;
    first_term(b, bb.pass, it, par);
    TF* F = (TF*)b.forces;
    TF f0[3] = {TF(0), TF(0), TF(0)};
    if (live)
        for (int c = 0; c < 3; ++c) {
            lpos[c * b.max_atoms + tid] = b.pos[3 * (size_t)a + c];
            if (b.add) f0[c] = F[3 * (size_t)a + c];
        }
    bonded_forces<Sums, true>(b, bb, lpos, lf, it, par, fa, acc);
    if (live)
        for (int c = 0; c < 3; ++c) F[3 * (size_t)a + c] = f0[c] + (TF)fa[c];
    if constexpr (Sums) {
        const double r = block_sum<10>(acc, red);
        if (tid < 10) b.partial[(size_t)blockIdx.x * 10 + tid] = r;
    }
}

// Sum over the blocks' partials in a fixed order: lane l of a wave adds
// blocks l, l + 64, ... of p1 and then of p2, and the wave adds its lanes.
// A lane's loads are issued kSumLoads at a time before any is added, so a
// few hundred partials cost one or two memory round trips, not one per
// block of the lane.
constexpr int kSumLoads = 8;

__device__ __forceinline__ void add_blocks(const double* __restrict__ p, int n, int K, int k,
                                           int lane, double& s)
{
    auto round = [&](int base) {
        double x[kSumLoads];
#pragma unroll
        for (int u = 0; u < kSumLoads; ++u) {
            const int blk = base + 64 * u;
            x[u] = blk < n ? p[(size_t)blk * K + k] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kSumLoads; ++u)
            if (base + 64 * u < n) s += x[u];
    };
    // the first round outside the loop: its reads are not held back until
    // the caller's earlier reads are in
    if (lane < n) round(lane);
    for (int base = lane + 64 * kSumLoads; base < n; base += 64 * kSumLoads) round(base);
}

__device__ __forceinline__ double sum_blocks(const double* __restrict__ p1, int n1,
                                             const double* __restrict__ p2, int n2, int K, int k)
{
    const int lane = (int)threadIdx.x & 63;
    double s = 0.0;
    add_blocks(p1, n1, K, k, lane, s);
    add_blocks(p2, n2, K, k, lane, s);
    return wave_sum(s);                // complete in lane 63
}

// Sum of the kinetic partials over a block of kMdBlock threads in a fixed
// order (thread t adds t, t + kMdBlock, ..., the block its threads): the force
// launch of 48000 atoms leaves about 2000 partials, one round of 8 reads in
// flight per thread.  Thread 0 gets the sum.
__device__ __forceinline__ double sum_kinetic(const double* __restrict__ p, int n,
                                              double (*red)[kMdBlock / 64])
{
    double s = 0.0;
    for (int base = (int)threadIdx.x; base < n; base += kMdBlock * kSumLoads) {
        double x[kSumLoads];
#pragma unroll
        for (int u = 0; u < kSumLoads; ++u) {
            const double v = p[min(base + kMdBlock * u, n - 1)];
            x[u] = base + kMdBlock * u < n ? v : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kSumLoads; ++u) s += x[u];
    }
    return block_sum<1>(&s, red);
}

// Sums of groups of kMdGroup kinetic partials, one block each, in the order of
// sum_kinetic.  Drift blocks read them from L2, a few partials faster than
// the launch costs: a step of 48000 atoms (2100 partials) takes 37.2 us without
// and 39.4 with it, of 120000 69.3 both, of 360000 169.8 and 154.6, of 1.02
// million 573 and 428, of 3 million 2565 and 1254.
constexpr int kMdGroup = kMdBlock * kSumLoads;
constexpr int kMdParts = 4096;

__global__ __launch_bounds__(kMdBlock) void k_md_gather(const double* __restrict__ partial, int n,
                                                        double* __restrict__ sums)
{
    __shared__ double red[1][kMdBlock / 64];
    const int first = (int)blockIdx.x * kMdGroup;
    const double s = sum_kinetic(partial + first, min(kMdGroup, n - first), red);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// out[k] = the sums over blocks of p1[blk * K + k] and of p2 (one wave per
// component k).
__global__ void k_sum_partials(const double* __restrict__ p1, int n1,
                               const double* __restrict__ p2, int n2, int K,
                               double* __restrict__ out)
{
    const int k = (int)threadIdx.x >> 6;
    const double s = sum_blocks(p1, n1, p2, n2, K, k);
    if (((int)threadIdx.x & 63) == 63) out[k] = s;
}

// ---------------------------------------------------------------------------
// Nose-Hoover velocity Verlet.  Stored velocities v_s; the true velocities
// are v_s * st.s2 (the scale of the last thermostat half step, applied
// together with the next one).  Thermostat half step over dt/2:
//   xi += dt/4 G(K);  v *= exp(-xi dt/2) (K *= its square);  eta += dt/2 xi;
//   xi += dt/4 G(K),   G(K) = (2K - g kT)/Q.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void thermostat_half(MdState* st)
{
    const double dt = st->dt;
    st->xi += 0.25 * dt * (2.0 * st->K - st->g * st->kT) / st->Q;
    const double s = exp(-st->xi * 0.5 * dt);
    st->K *= s * s;
    st->eta += 0.5 * dt * st->xi;
    st->xi += 0.25 * dt * (2.0 * st->K - st->g * st->kT) / st->Q;
    st->s_last = s;
}

// The scalar work between two steps on a copy of the state: the kinetic
// energy from the partial sum; with `second` the second thermostat half
// step of the step just done (and, with `row`, its thermodynamic output: the
// non-bonded energy of Eq. 3, the 1-4, bond, angle and dihedral energies,
// the kinetic energy, the extended energy K + U + Q xi^2/2 + g kT eta and
// the trace of the virial); with `first` the first half step of the next
// step, whose drift applies s2 s1 to the stored velocities.
__device__ void scalar_step(MdState& st, double ksum, double ftm2v, int second, int first,
                            const double* __restrict__ e_nb, const double* __restrict__ w_nb,
                            const double* __restrict__ eb, double* __restrict__ row)
{
    st.K = 0.5 * ksum / ftm2v;
    if (second) {
        thermostat_half(&st);
        st.s2 = st.s_last;
        if (row) {
            const double u = e_nb[0] + eb[3] + eb[0] + eb[1] + eb[2];
            row[0] = e_nb[0];
            row[1] = eb[3];
            row[2] = eb[0];
            row[3] = eb[1];
            row[4] = eb[2];
            row[5] = st.K;
            row[6] = st.K + u + 0.5 * st.Q * st.xi * st.xi + st.g * st.kT * st.eta;
            row[7] = w_nb[0] + w_nb[1] + w_nb[2] + eb[4] + eb[5] + eb[6];
        }
    }
    if (first) {
        thermostat_half(&st);
        st.s_apply = st.s2 * st.s_last;
        st.s2 = 1.0;
    }
}

// The atom's data of a drift: none of it depends on the scalar work, so its
// reads overlap the sum of the partials.
template <typename TF>
struct DriftAtom {
    double v[3], x[3], xref[3], mass;
    TF f[3];
};

template <typename TF>
__device__ __forceinline__ DriftAtom<TF> drift_read(const MdArgs& m, int i, bool in)
{
    DriftAtom<TF> d;
    const TF* F = (const TF*)m.forces;
    d.mass = 1.0;
    for (int c = 0; c < 3; ++c) {
        d.v[c] = d.x[c] = d.xref[c] = 0.0;
        d.f[c] = TF(0);
    }
    if (in) {
        for (int c = 0; c < 3; ++c) {
            d.v[c] = m.vel[3 * i + c];
            d.x[c] = m.pos[3 * i + c];
            d.xref[c] = m.xref[3 * i + c];
            d.f[c] = F[3 * i + c];
        }
        d.mass = m.mass[i];
    }
    return d;
}

// Scale of the stored velocities in a drift.  With d.scalar every block first
// does the scalar work between the previous step and this one (the same sums
// in the same order, so every block gets the same state; block 0 stores it in
// st_out and writes the row), which saves a launch per step; st_in is not
// written, so no block can see a half-updated state.  Without it the state in
// st_in is current.  All threads of the block.
__device__ __forceinline__ double drift_scale(const MdArgs& m, const DriftArgs& d, double* s_sh,
                                              double (*red)[kMdBlock / 64])
{
    if (!d.scalar) return d.st_in->s_apply;
    MdState st;
    if (threadIdx.x == 0) st = *d.st_in;
    const double ks = sum_kinetic(m.partial, d.nparts, red);
    if (threadIdx.x == 0) {
        scalar_step(st, ks, m.ftm2v, 1, 1, d.e_nb, d.w_nb, d.eb, blockIdx.x == 0 ? d.row : nullptr);
        if (blockIdx.x == 0) *d.st_out = st;
        *s_sh = st.s_apply;
    }
    __syncthreads();
    return *s_sh;
}

// The drift of atom i; its new position goes to a.x.
template <typename TF>
__device__ __forceinline__ void drift_atom(const MdArgs& m, int i, bool in, double dt, double s,
                                           DriftAtom<TF>& a)
{
    const double am = m.ftm2v / a.mass;
    double dmax2 = 0.0;
    if (in)
        for (int c = 0; c < 3; ++c) {
            const double v = a.v[c] * s + 0.5 * dt * am * (double)a.f[c];
            m.vel[3 * i + c] = v;
            a.x[c] += dt * v;
            m.pos[3 * i + c] = a.x[c];
            const double dx = a.x[c] - a.xref[c];
            dmax2 += dx * dx;
        }
    // an atom that moved more than half the skin since the last build (or whose
    // position is no number: the comparison is false) invalidates the lists; the
    // host checks the count with the next build's status
    const uint64_t far = __ballot(!(dmax2 <= m.half_skin2));
    if (far != 0ull && ((int)threadIdx.x & 63) == __ffsll((long long)far) - 1) atomicAdd(m.stale, 1u);
}

// Drift of one step, one thread per atom.
template <typename TF>
__global__ __launch_bounds__(kMdBlock) void k_md_drift(MdArgs m, DriftArgs d)
{
    __shared__ double s_sh;
    __shared__ double red[1][kMdBlock / 64];
    const int i = blockIdx.x * kMdBlock + threadIdx.x;
    const bool in = i < m.n;
    DriftAtom<TF> a = drift_read<TF>(m, i, in);
    const double dt = d.st_in->dt;
    const double s = drift_scale(m, d, &s_sh, red);
    drift_atom(m, i, in, dt, s, a);
}

// Drift of one step and the bonded forces at the new positions (written to
// b.forces), one block per bonded block, for blocks whose terms hold only atoms
// of the block.  The force launch that follows adds them and gives the half
// kick, so a step is two launches: each launch of a 6000-atom step is bound by
// its dependent reads (about 3 us with the gap), not by its work.  Kernel trace
// of a step, drift + forces + bonded before, this kernel + forces now: 6000
// atoms 3.6 + 6.7 + 5.0 to 5.9 + 7.2 us (a run 20.5 to 18.6 us a step), 48000
// atoms 4.5 + 15.9 + 7.6 to 9.3 + 17.2 us (40.4 to 39.2).
template <typename TF, bool Sums>
__global__ __launch_bounds__(kMdBlock) void k_md_drift_bonded(MdArgs m, DriftArgs d, BondedArgs b)
{
    extern __shared__ double lds[];
    __shared__ double s_sh;
    __shared__ double red[Sums ? 10 : 1][kMdBlock / 64];
    double* lpos = lds;                                  // [3][max_atoms]
    double* lf = lds + 3 * b.max_atoms;                  // [3][max_slots]
    const BondBlock bb = b.blocks[blockIdx.x];
    const int tid = (int)threadIdx.x;
    const int i = bb.atom0 + tid;
    const bool in = tid < bb.natoms;
    DriftAtom<TF> a = drift_read<TF>(m, i, in);
    BondTerm it;
    double4 par;
    first_term(b, bb.pass, it, par);
    const double dt = d.st_in->dt;
    const double s = drift_scale(m, d, &s_sh, red);
    drift_atom(m, i, in, dt, s, a);
    if (in)
        for (int c = 0; c < 3; ++c) lpos[c * b.max_atoms + tid] = a.x[c];
    double acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    double fa[3] = {0.0, 0.0, 0.0};
    bonded_forces<Sums, false>(b, bb, lpos, lf, it, par, fa, acc);
    if (in)
        for (int c = 0; c < 3; ++c) ((TF*)b.forces)[3 * (size_t)i + c] = (TF)fa[c];
    if constexpr (Sums) {
        const double r = block_sum<10>(acc, red);
        if (tid < 10) b.partial[(size_t)blockIdx.x * 10 + tid] = r;
    }
}

// Everything a run needs to go on from a list build: the reference positions
// of the displacement check, the velocities and the thermostat state.
__global__ __launch_bounds__(kMdBlock) void k_md_mark(MdArgs m, double* __restrict__ vsave,
                                                      MdState* __restrict__ ssave)
{
    const int i = blockIdx.x * kMdBlock + threadIdx.x;      // one component each
    if (i < 3 * m.n) {
        m.xref[i] = m.pos[i];
        vsave[i] = m.vel[i];
    }
    if (i == 0) *ssave = *m.st;
}

// Kinetic partials of the stored velocities (no kick), at the start of a run.
__global__ __launch_bounds__(kMdBlock) void k_md_kinetic(MdArgs m)
{
    __shared__ double red[1][kMdBlock / 64];
    const int i = blockIdx.x * kMdBlock + threadIdx.x;
    double ke = 0.0;
    if (i < m.n)
        for (int c = 0; c < 3; ++c) ke += m.mass[i] * m.vel[3 * i + c] * m.vel[3 * i + c];
    const double r = block_sum<1>(&ke, red);
    if (threadIdx.x == 0) m.partial[blockIdx.x] = r;
}

// The scalar work between two steps as a kernel of its own (one block; at
// the start and the end of a run, where no drift follows): scalar_step on
// the state in place.
__global__ __launch_bounds__(kMdBlock) void k_md_scalar(MdState* st, const double* __restrict__ partial,
                                                        int nblocks, double ftm2v, int second, int first,
                                                        const double* __restrict__ e_nb,
                                                        const double* __restrict__ w_nb,
                                                        const double* __restrict__ eb,
                                                        double* __restrict__ row)
{
    __shared__ double red[1][kMdBlock / 64];
    const double s = sum_kinetic(partial, nblocks, red);
    if (threadIdx.x != 0) return;
    MdState cur = *st;
    scalar_step(cur, s, ftm2v, second, first, e_nb, w_nb, eb, row);
    *st = cur;
}

// Make the stored velocities the true ones (v_s *= s2), at the end of a run.
__global__ __launch_bounds__(kMdBlock) void k_md_finish(MdArgs m)
{
    const int i = blockIdx.x * kMdBlock + threadIdx.x;
    if (i >= m.n) return;
    const double s = m.st->s2;
    for (int c = 0; c < 3; ++c) m.vel[3 * i + c] *= s;
}

__global__ void k_md_unit_scale(MdState* st) { st->s2 = 1.0; }

}  // namespace

namespace {
size_t bonded_lds(const BondedArgs& b)
{
    return sizeof(double) * 3 * (size_t)(b.max_atoms + b.max_slots);
}
}  // namespace

hipError_t launch_bonded(const BondedArgs& b, int force_prec, hipStream_t s)
{
    if (b.n == 0) return hipSuccess;
    const dim3 grid(b.nblocks);
    const size_t lds = bonded_lds(b);
#define RELRES_BONDED(TF, SUMS)                                                                  \
    hipLaunchKernelGGL((k_bonded<TF, SUMS>), grid, dim3(kMdBlock), lds, s, b)
    if (force_prec == 64) {
        if (b.partial) RELRES_BONDED(double, true); else RELRES_BONDED(double, false);
    } else {
        if (b.partial) RELRES_BONDED(float, true); else RELRES_BONDED(float, false);
    }
#undef RELRES_BONDED
    return hipGetLastError();
}

int md_blocks(int n) { return (n + kMdBlock - 1) / kMdBlock; }

hipError_t launch_sum_partials(const double* p1, int n1, const double* p2, int n2, int K,
                               double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(64 * K), 0, s, p1, n1, p2, n2, K, out);
    return hipGetLastError();
}

hipError_t launch_md_drift(const MdArgs& m, const DriftArgs& d, int force_prec, hipStream_t s)
{
    const int blocks = (m.n + kMdBlock - 1) / kMdBlock;
    if (force_prec == 64)
        hipLaunchKernelGGL(k_md_drift<double>, dim3(blocks), dim3(kMdBlock), 0, s, m, d);
    else
        hipLaunchKernelGGL(k_md_drift<float>, dim3(blocks), dim3(kMdBlock), 0, s, m, d);
    return hipGetLastError();
}

hipError_t launch_md_drift_bonded(const MdArgs& m, const DriftArgs& d, const BondedArgs& b,
                                  int force_prec, hipStream_t s)
{
    const dim3 grid(b.nblocks);
    const size_t lds = bonded_lds(b);
#define RELRES_STEP(TF, SUMS)                                                                    \
    hipLaunchKernelGGL((k_md_drift_bonded<TF, SUMS>), grid, dim3(kMdBlock), lds, s, m, d, b)
    if (force_prec == 64) {
        if (b.partial) RELRES_STEP(double, true); else RELRES_STEP(double, false);
    } else {
        if (b.partial) RELRES_STEP(float, true); else RELRES_STEP(float, false);
    }
#undef RELRES_STEP
    return hipGetLastError();
}

hipError_t launch_md_mark(const MdArgs& m, double* vsave, MdState* ssave, hipStream_t s)
{
    hipLaunchKernelGGL(k_md_mark, dim3((unsigned)((3LL * m.n + kMdBlock - 1) / kMdBlock)),
                       dim3(kMdBlock), 0, s, m, vsave, ssave);
    return hipGetLastError();
}

int md_groups(int nparts)
{
    return nparts > kMdParts ? (nparts + kMdGroup - 1) / kMdGroup : nparts;
}

hipError_t launch_md_gather(const double* partial, int nparts, double* sums, hipStream_t s)
{
    hipLaunchKernelGGL(k_md_gather, dim3((nparts + kMdGroup - 1) / kMdGroup), dim3(kMdBlock), 0, s,
                       partial, nparts, sums);
    return hipGetLastError();
}

hipError_t launch_md_kinetic(const MdArgs& m, hipStream_t s)
{
    hipLaunchKernelGGL(k_md_kinetic, dim3((m.n + kMdBlock - 1) / kMdBlock), dim3(kMdBlock), 0, s, m);
    return hipGetLastError();
}

hipError_t launch_md_scalar(MdState* st, const double* partial, int nblocks, double ftm2v,
                            int second, int first, const double* e_nb, const double* w_nb,
                            const double* eb, double* row, hipStream_t s)
{
    hipLaunchKernelGGL(k_md_scalar, dim3(1), dim3(kMdBlock), 0, s, st, partial, nblocks, ftm2v, second,
                       first, e_nb, w_nb, eb, row);
    return hipGetLastError();
}

hipError_t launch_md_finish(const MdArgs& m, hipStream_t s)
{
    const int blocks = (m.n + kMdBlock - 1) / kMdBlock;
    hipLaunchKernelGGL(k_md_finish, dim3(blocks), dim3(kMdBlock), 0, s, m);
    hipLaunchKernelGGL(k_md_unit_scale, dim3(1), dim3(1), 0, s, m.st);
    return hipGetLastError();
}

}  // namespace relres
