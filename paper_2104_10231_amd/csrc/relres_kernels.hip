// relres_kernels.hip -- gfx950 kernels of the RelRes Lennard-Jones hot path.
//
// Build (every rebuild):  k_bin -> k_place -> k_lists_wave
//   Two cell grids are built side by side: the atom grid (cells >= r_s+ + skin,
//   all atoms) and the site grid (cells >= r_c+ + skin, hybrid atoms only).
//   Cells are numbered in Morton order so that neighbouring cells, and the
//   atoms they hold, sit close together in memory.  Within a cell, members are
//   ordered by caller index, which makes every list row deterministic.  k_bin
//   files the members into buckets of their cells and k_place puts them into
//   cell order (more than 8192 cells: k_place_totals first); crowded or sparse
//   grids take k_scan -> k_scatter -> k_cellsort instead.
//   A wave of k_lists_wave takes a few home rows, tests 64 candidates of their
//   cells' stencils at a time and appends the survivors to each row with a
//   ballot + mbcnt prefix.
// Forces (every call): k_forces
//   One launch covers both lists.  Rows of ordinary atoms take the FG part over
//   their atom-list row; rows of hybrid atoms take the FG part over their
//   atom-list row plus the CG part over their site-list row.  Each row is owned
//   by a group of lanes that accumulate its force in registers and reduce it
//   with cross-lane shuffles, so no force atomics are needed.  Energy and
//   virial are accumulated in FP64 and reduced in a fixed order by the blocks
//   of highest number.
#include "relres_internal.h"
#include "relres_pair.h"
#include "relres_lanes.h"

#include <cstdlib>

namespace relres {
namespace {

constexpr int kWave = 64;
constexpr int kChunk = 256;    // candidates staged in LDS per pass

// Pointers read from the grid descriptors live in device memory, so the
// compiler cannot tell they are global and would use flat instructions, which
// may alias LDS and make every LDS access wait for outstanding global stores.
// Casting them to the global address space gives plain global loads/stores.
#define RELRES_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ RELRES_GLOBAL T* gbl(T* p) { return (RELRES_GLOBAL T*)p; }
// HIP vector types cannot be copied through such pointers; read them as scalars.
// A cell-sorted member carries its list entry and molecule in the fourth
// component of its position: the low 32 bits are the entry (caller index |
// type << kIdxBits), the high 32 bits the molecule.  One 32-byte read gives
// everything the list kernel needs of a member.
__device__ __forceinline__ double member_tag(int u, int type, int mol)
{
    const uint32_t entry = (uint32_t)u | ((uint32_t)type << kIdxBits);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)mol << 32) | entry));
}
__device__ __forceinline__ void load_member(const double4* base, int i, double& x, double& y,
                                            double& z, uint32_t& entry, int& mol)
{
    RELRES_GLOBAL const double* p = (RELRES_GLOBAL const double*)base + 4 * (size_t)i;
    x = p[0];
    y = p[1];
    z = p[2];
    const uint64_t w = (uint64_t)__double_as_longlong(p[3]);
    entry = (uint32_t)w;
    mol = (int)(uint32_t)(w >> 32);
}
constexpr int kHomeMax = 256;  // home atoms whose counters live in LDS at once

// Wrap one coordinate into [0, L):  w = x - L floor(x / L), fixed into range.
// Separately rounded operations; the oracle performs the same sequence.
__device__ __forceinline__ double wrap_coord(double x, double L)
{
#pragma clang fp contract(off)
    double w = x - L * floor(x / L);
    if (w < 0.0) w += L;
    if (w >= L) w -= L;
    if (w < 0.0 || w >= L) w = 0.0;
    return w;
}

__device__ __forceinline__ int cell_coord(double w, double inv, int n)
{
    int c = (int)(w * inv);
    return c < n ? c : n - 1;
}

// List membership in FP64 on wrapped positions (a = home atom, b = candidate):
// single-shift minimum image, r2 = (dx dx + dy dy) + dz dz, strict r2 < rl2.
// The shift is chosen by selects, not branches: d + (-L) rounds exactly as
// d - L, and adding 0 leaves d (a -0 becomes +0, which squares the same).
__device__ __forceinline__ double min_image(double d, double L, double h)
{
#pragma clang fp contract(off)
    const double s = d > h ? -L : (d < -h ? L : 0.0);
    return d + s;
}

__device__ __forceinline__ bool member(const double4 a, const double4 b, double Lx, double Ly,
                                       double Lz, double hx, double hy, double hz, double rl2)
{
#pragma clang fp contract(off)
    const double dx = min_image(b.x - a.x, Lx, hx);
    const double dy = min_image(b.y - a.y, Ly, hy);
    const double dz = min_image(b.z - a.z, Lz, hz);
    const double r2 = (dx * dx + dy * dy) + dz * dz;
    return r2 < rl2;
}

__device__ __forceinline__ int lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// ---------------------------------------------------------------------------
// build kernels
// ---------------------------------------------------------------------------

// A grid's geometry in the binning kernel: one system's is read through the
// scalar cache, several systems' per lane.
template <bool Multi>
struct BinGeomOf {
    using type = const GeomDev RELRES_GLOBAL*;
};
template <>
struct BinGeomOf<false> {
    using type = const GeomDev __attribute__((address_space(4)))*;
};
template <bool Multi>
using BinGeom = typename BinGeomOf<Multi>::type;

// Minimum-image squared distance of (x, y, z) from a wrapped position.
__device__ __forceinline__ double image_dist2(double x, double y, double z, double4 w,
                                              const double* L)
{
    double dx = x - w.x, dy = y - w.y, dz = z - w.z;
    dx -= L[0] * rint(dx / L[0]);
    dy -= L[1] * rint(dy / L[1]);
    dz -= L[2] * rint(dz / L[2]);
    return dx * dx + dy * dy + dz * dz;
}

// Add the lanes of the wave with `flag` set to *count (one atomic per wave).
__device__ __forceinline__ void count_wave(bool flag, unsigned* count)
{
    const unsigned long long m = __ballot(flag);
    if (m != 0ull && (int)(threadIdx.x & (kWave - 1)) == __ffsll((long long)m) - 1)
        atomicAdd(count, (unsigned)__popcll(m));
}

// The slots of a wave's members in their cells: lanes of the wave that share a
// cell take consecutive slots after one atomic add by the first of them, so a
// cell sees one atomic per wave rather than one per atom (same-address atomics
// serialise).  Slot order within a cell is arbitrary; the cell sort orders
// members by caller index afterwards.
struct SlotGroup {
    int lead, rank;          // first lane of the lane's group, place in it
    int n_lead;              // lead lane: members of its group, others 0
};

__device__ __forceinline__ SlotGroup slot_group(int r, bool want)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t todo = __ballot(want);
    SlotGroup g{0, 0, 0};
    while (todo != 0ull) {
        const int l = __ffsll((long long)todo) - 1;
        const int rl = __builtin_amdgcn_readlane(r, l);
        const uint64_t grp = todo & __ballot(r == rl);
        if ((grp >> lane) & 1ull) {
            g.lead = l;
            g.rank = lanes_below(grp);
        }
        if (lane == l) g.n_lead = __popcll(grp);
        todo &= ~grp;
    }
    return g;
}

// One atomic instruction for all the groups (their cells are distinct).
__device__ __forceinline__ int claim_slots(RELRES_GLOBAL int* count, int r, const SlotGroup& g)
{
    int got = 0;
    if (g.n_lead > 0)
        got = __hip_atomic_fetch_add(count + r, g.n_lead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return got;
}

// One-launch placement: member i goes straight into its cell's bucket; one that
// finds it full goes to the head of one of the cell's chains, in turn by its
// slot, and the member before it is returned as its key's second word (the first
// of a chain gets the head of an earlier build: a chain is followed for as many
// members as the cell's count says).  Otherwise that word is the slot.
__device__ __forceinline__ int file_member(const GridDev& g, int cell, int slot, int i)
{
    if (g.bucket_cap <= 0) return slot;
    if (slot < g.bucket_cap) {
        gbl(g.user_unsorted)[(size_t)cell * g.bucket_cap + slot] = i;
        return slot;
    }
    const size_t chain = (size_t)cell * kPlaceChains + (slot - g.bucket_cap) % kPlaceChains;
    return __hip_atomic_exchange(gbl(g.chain_head) + chain, i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int lin_cell(const double w[3], const double inv[3], const int n[3])
{
    return (cell_coord(w[0], inv[0], n[0]) * n[1] + cell_coord(w[1], inv[1], n[1])) * n[2] +
           cell_coord(w[2], inv[2], n[2]);
}

// Wrapped positions, cells and slots of all atoms.  Bound by its chain of
// dependent memory round trips, so every read that waits on no other goes out
// first and both grids' slot claims (round trips past the XCD's L2) are in
// flight together, with the displacement check under them: position, type and
// system -> geometry (in scalar registers with one system) -> cell ranks ->
// claims -> stores.  (Builds of 1500 propane atoms 16.2 to 15.4 us, 20480
// neopentane atoms 22.3 to 21.5, 256 replicas of 1.2 million atoms 439.9 to 432.7.)
template <bool Multi>
__global__ __launch_bounds__(256) void k_bin(int n, const double* __restrict__ pos, TopoDev topo,
                                             const GridDev* __restrict__ grids,
                                             double4* __restrict__ wpos, int2* __restrict__ key_a,
                                             int2* __restrict__ key_s, Status* __restrict__ st,
                                             int check_moved)
{
    // every lane takes part in the wave's slot claims; lanes past n only vote
    const int i0 = blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = i0 < n;
    const int i = in ? i0 : n - 1;
    // grids[1] is grids[0] again when there are no sites (no hybrid lanes then)
    const GridDev &ga = grids[0], &gs = grids[1];
    RELRES_GLOBAL int *const count_a = gbl(ga.count), *const count_s = gbl(gs.count);
    RELRES_GLOBAL const int *const rank_a = gbl(ga.rank_of_lin), *const rank_s = gbl(gs.rank_of_lin);
    const int ty = topo.types[i];
    const int sy = Multi ? topo.sys[i] : 0;
    double x[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) x[k] = pos[3 * i + k];
    const double4 ref = wpos[i];       // of the previous build (unused before the first)
    const BinGeom<Multi> G = (BinGeom<Multi>)(ga.geom + sy), H = (BinGeom<Multi>)(gs.geom + sy);
    double L[3], inv[3], inv_s[3];
    int nc[3], nc_s[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        L[k] = G->box[k];
        inv[k] = G->inv_cell[k];
        nc[k] = G->n[k];
        inv_s[k] = H->inv_cell[k];
        nc_s[k] = H->n[k];
    }
    const int base = G->cell_base, base_s = H->cell_base;
    const double half_skin2 = G->half_skin2;
    if (!(isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]))) {
        count_wave(in, &st->nonfinite);
        x[0] = x[1] = x[2] = 0.0;
    }
    const bool hyb = topo.hybrid[ty] != 0 && in;
    double w[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = wrap_coord(x[k], L[k]);
    const int r = rank_a[base + lin_cell(w, inv, nc)];
    const int ls = base_s + lin_cell(w, inv_s, nc_s);
    const int rs = rank_s[hyb ? ls : 0];   // a system may have no sites and no cell of its own
    const SlotGroup qa = slot_group(r, in), qs = slot_group(rs, hyb);
    const int got_a = claim_slots(count_a, r, qa);
    const int got_s = claim_slots(count_s, rs, qs);
    if (check_moved)   // displacement since the previous build (same boxes and skins)
        count_wave(in && image_dist2(x[0], x[1], x[2], ref, L) > half_skin2, &st->moved);
    if (in) wpos[i] = make_double4(w[0], w[1], w[2], 0.0);
    const int slot = __shfl(got_a, qa.lead) + qa.rank, slot_s = __shfl(got_s, qs.lead) + qs.rank;
    if (in) {
        key_a[i] = make_int2(r, file_member(ga, r, slot, i));
        key_s[i] = hyb ? make_int2(rs, file_member(gs, rs, slot_s, i)) : make_int2(-1, -1);
    }
}

// Atoms now more than half the skin from their position at the last build.
__global__ void k_moved(int n, const double* __restrict__ pos, TopoDev topo,
                        const GridDev* __restrict__ grids, const double4* __restrict__ wpos,
                        Status* __restrict__ st)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int sy = topo.sys ? topo.sys[i] : 0;
    const double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
    const GeomDev& G = grids[0].geom[sy];
    // a non-finite position counts as moved (the comparison is false for NaN)
    count_wave(!(image_dist2(x, y, z, wpos[i], G.box) <= G.half_skin2), &st->moved_query);
}

// One block per grid: exclusive scan of the per-cell counts into `start`,
// then the counts are cleared for the next build.  Counts are staged through
// LDS in segments of kScanSeg cells with coalesced loads; each thread scans a
// contiguous run of its segment.  Block 0 also clears the list statistics.
constexpr int kScanThreads = 1024;
constexpr int kScanSeg = 8192;

// Exclusive prefix sum over the block of one int per thread (in thread
// order); every thread also gets the block's total.  Each wave scans its
// lanes with cross-lane shuffles, then adds the totals of the waves before
// it: two block barriers in all.
__device__ __forceinline__ int block_exclusive_scan(int v, int* wtot, int& total)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) wtot[w] = x;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / kWave; ++k) {
        const int t = wtot[k];
        before += k < w ? t : 0;
        all += t;
    }
    __syncthreads();            // wtot is reused by the next call
    total = all;
    return before + x - v;
}

// One segment of the scan (all threads of the block): start[seg + k] =
// carry + the exclusive prefix of the segment's counts, the counts cleared.
// Returns the segment's total in every thread.
__device__ __forceinline__ int scan_segment(int* vals, int* sums, RELRES_GLOBAL int* gcount,
                                            RELRES_GLOBAL int* gstart, int seg, int len, int carry)
{
    const int t = threadIdx.x;
    constexpr int per = kScanSeg / kScanThreads;
    for (int k = t; k < kScanSeg; k += kScanThreads) vals[k] = k < len ? gcount[seg + k] : 0;
    __syncthreads();
    int s = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) s += vals[t * per + k];
    int total;
    int run = carry + block_exclusive_scan(s, sums, total);
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const int v = vals[t * per + k];
        vals[t * per + k] = run;
        run += v;
    }
    __syncthreads();
    for (int k = t; k < len; k += kScanThreads) {
        gstart[seg + k] = vals[k];
        gcount[seg + k] = 0;
    }
    __syncthreads();            // vals is reused by the next segment
    return total;
}

// Sum of one int per thread over the block (every thread gets it).
__device__ __forceinline__ int block_sum_int(int v, int* sums)
{
    int total;
    block_exclusive_scan(v, sums, total);
    return total;
}

// One block per grid: exclusive scan of the per-cell counts into `start`,
// then the counts are cleared for the next build.  Counts are staged through
// LDS in segments of kScanSeg cells with coalesced loads; each thread scans a
// contiguous run of its segment.
__global__ __launch_bounds__(kScanThreads) void k_scan(GridDev* __restrict__ grids)
{
    __shared__ int vals[kScanSeg];
    __shared__ int sums[kScanThreads];
    const GridDev& g = grids[blockIdx.x];
    const int nc = g.ncell;
    int carry = 0;
    for (int seg = 0; seg < nc; seg += kScanSeg)
        carry += scan_segment(vals, sums, gbl(g.count), gbl(g.start), seg, min(kScanSeg, nc - seg),
                              carry);
    if (threadIdx.x == 0) gbl(g.start)[nc] = carry;
}

// Grids of more than one segment: the same scan with every segment in a
// block of its own.  Blocks 0 .. nseg0-1 are the segments of grid 0, the
// rest those of grid 1.  First each block sums its segment's counts ...
__global__ __launch_bounds__(kScanThreads) void k_scan_totals(const GridDev* __restrict__ grids,
                                                              int nseg0, int* __restrict__ seg_tot)
{
    __shared__ int sums[kScanThreads];
    const int b = blockIdx.x;
    const int gi = b >= nseg0 ? 1 : 0;
    const int seg = (gi ? b - nseg0 : b) * kScanSeg;
    const GridDev& g = grids[gi];
    const int len = min(kScanSeg, g.ncell - seg);
    RELRES_GLOBAL const int* gcount = gbl(g.count);
    int s = 0;
    for (int k = threadIdx.x; k < len; k += kScanThreads) s += gcount[seg + k];
    s = block_sum_int(s, sums);
    if (threadIdx.x == 0) seg_tot[b] = s;
}

// ... then each block adds the totals of its grid's earlier segments and
// scans its own segment (the grid's last segment also writes start[ncell]).
__global__ __launch_bounds__(kScanThreads) void k_scan_segments(GridDev* __restrict__ grids,
                                                                int nseg0,
                                                                const int* __restrict__ seg_tot)
{
    __shared__ int vals[kScanSeg];
    __shared__ int sums[kScanThreads];
    const int b = blockIdx.x;
    const int gi = b >= nseg0 ? 1 : 0;
    const int q = gi ? b - nseg0 : b;
    const int first = gi ? nseg0 : 0;
    const GridDev& g = grids[gi];
    const int nc = g.ncell;
    const int seg = q * kScanSeg;
    int carry = 0;
    for (int j = threadIdx.x; j < q; j += kScanThreads) carry += seg_tot[first + j];
    carry = block_sum_int(carry, sums);
    const int len = min(kScanSeg, nc - seg);
    const int total = scan_segment(vals, sums, gbl(g.count), gbl(g.start), seg, len, carry);
    if (threadIdx.x == 0 && seg + len == nc) gbl(g.start)[nc] = carry + total;
}

__global__ void k_scatter(int n, const GridDev* __restrict__ grids, const int2* __restrict__ key_a,
                          const int2* __restrict__ key_s)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int2 ka = key_a[i];
    gbl(grids[0].user_unsorted)[gbl(grids[0].start)[ka.x] + ka.y] = i;
    const int2 ks = key_s[i];
    if (ks.x >= 0) gbl(grids[1].user_unsorted)[gbl(grids[1].start)[ks.x] + ks.y] = i;
}

__device__ __forceinline__ int readlane_i(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
// A wave-uniform double moved to scalar registers.
__device__ __forceinline__ double readfirst_d(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffff));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ float readfirst_f(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ float readlane_f(float v, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

__device__ __forceinline__ double readlane_d(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Cell sort: order the members of every cell by caller index (rank by
// counting) and write the sorted position / (type, molecule) / index / cell
// arrays.  A wave takes kWave / G consecutive cells, one group of G lanes
// each; a cell of at most G members is ranked within its group by cross-lane
// reads, a larger one by the whole wave after the small ones.  G = 16 suits
// grids of a few members per cell, G = 64 (one cell per wave) crowded ones.

__device__ __forceinline__ void place_read(const GridDev& g, bool site, int c, int dst, int u,
                                           double4 p, int ty, int mol,
                                           int* __restrict__ user2arow)
{
    gbl(g.user)[dst] = u;
    g.pos[dst] = make_double4(p.x, p.y, p.z, member_tag(u, ty, mol));   // generic store (no LDS use here)
    g.meta[dst] = make_int2(ty, mol);
    gbl(g.row_cell)[dst] = c;
    if (!site) user2arow[u] = dst;
}

__device__ __forceinline__ void place_member(const GridDev& g, bool site, int c, int dst, int u,
                                             const double4* __restrict__ wpos, const TopoDev& topo,
                                             int* __restrict__ user2arow)
{
    place_read(g, site, c, dst, u, wpos[u], topo.types[u], topo.mol[u], user2arow);
}

template <int kSortGroup>
__global__ void k_cellsort(const GridDev* __restrict__ grids, int ncell_a, int ncell_total,
                           const double4* __restrict__ wpos, TopoDev topo,
                           int* __restrict__ user2arow)
{
    constexpr int kSortCells = kWave / kSortGroup;
    const int lane = threadIdx.x & (kWave - 1);
    const int q = lane / kSortGroup, gl = lane & (kSortGroup - 1);
    const int wave = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) / kWave);
    const int nwaves = (gridDim.x * blockDim.x) / kWave;
    for (int c0 = wave * kSortCells; c0 < ncell_total; c0 += nwaves * kSortCells) {
        // group q: cell c0 + q (cells past the end are empty)
        const int cell = c0 + q;
        const bool site = cell >= ncell_a;
        const GridDev& g = grids[site ? 1 : 0];
        const int c = site ? cell - ncell_a : cell;
        int b = 0, len = 0;
        if (cell < ncell_total) {
            RELRES_GLOBAL const int* gstart = gbl(g.start);
            b = gstart[c];
            len = gstart[c + 1] - b;
        }
        const bool small = len <= kSortGroup;
        const int u = (small && gl < len) ? gbl(g.user_unsorted)[b + gl] : 0x7fffffff;
        int r = 0;
        if constexpr (kSortGroup < kWave) {
#pragma unroll
            for (int k = 0; k < kSortGroup; ++k)
                r += __shfl(u, (lane & ~(kSortGroup - 1)) + k) < u;
        } else {
            const int m = small ? len : 0;      // one cell per wave: len is uniform
            for (int k = 0; k < m; ++k) r += __shfl(u, k) < u;
        }
        if (small && gl < len) place_member(g, site, c, b + r, u, wpos, topo, user2arow);
        // the larger cells of this wave, one at a time with the whole wave
        for (int k = 0; k < kSortCells; ++k) {
            const int lenk = readlane_i(len, k * kSortGroup);
            if (lenk <= kSortGroup) continue;
            const int cellk = c0 + k;
            const bool sitek = cellk >= ncell_a;
            const GridDev& gk = grids[sitek ? 1 : 0];
            const int ck = sitek ? cellk - ncell_a : cellk;
            const int bk = readlane_i(b, k * kSortGroup);
            RELRES_GLOBAL const int* guu = gbl(gk.user_unsorted);
            if (lenk <= kWave) {
                const int v = lane < lenk ? guu[bk + lane] : 0x7fffffff;
                int rk = 0;
                for (int j = 0; j < lenk; ++j) rk += __shfl(v, j) < v;
                if (lane < lenk) place_member(gk, sitek, ck, bk + rk, v, wpos, topo, user2arow);
                continue;
            }
            for (int base = 0; base < lenk; base += kWave) {
                const int t = base + lane;
                if (t < lenk) {
                    const int v = guu[bk + t];
                    int rk = 0;
                    for (int j = 0; j < lenk; ++j) rk += guu[bk + j] < v;
                    place_member(gk, sitek, ck, bk + rk, v, wpos, topo, user2arow);
                }
            }
        }
    }
}


// Scan, scatter and cell sort in one launch, for grids whose members k_bin has filed into per-cell buckets of bucket_cap slots.  A block
// takes kCells consecutive cells of one grid (the atom grid's blocks first):
// it adds up the counts of every cell before its own (each block repeats
// this, so it suits a few thousand cells; larger grids have k_place_totals
// run first), writes its cells' starts, then
// ranks each cell's members by caller index as k_cellsort does and writes
// the sorted arrays.  A cell with more members than its bucket holds finds the
// others in its chains, or, above kPlaceWide members, all of them, already in
// caller order, by a wave-wide pass over the key array.
// The counts stay as they are: the list kernel clears them.
constexpr int kPlaceThreads = 256;
constexpr int kPlaceWide = 1024;      // most members of a cell that a wave ranks in LDS

// Orders a wave's LDS writes before its lanes' later reads of each other's.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Grids of many cells: the members of every kPlaceSeg consecutive cells, one
// block each (blocks 0 .. nseg_a - 1 the atom grid's, the rest the site
// grid's), so that a block of k_place adds up segments and the counts of part
// of its own segment instead of every count before its cells.
__global__ __launch_bounds__(kPlaceThreads) void k_place_totals(const GridDev* __restrict__ grids,
                                                                int nseg_a, int* __restrict__ seg_tot)
{
    __shared__ int wtot[kPlaceThreads / kWave];
    const int b = (int)blockIdx.x;
    const GridDev& g = grids[b >= nseg_a ? 1 : 0];
    const int seg = (b >= nseg_a ? b - nseg_a : b) * kPlaceSeg, nc = g.ncell;
    RELRES_GLOBAL const int* gcount = gbl(g.count);
    int s = 0;
#pragma unroll
    for (int u = 0; u < kPlaceSeg / kPlaceThreads; ++u) {
        const int c = seg + u * kPlaceThreads + (int)threadIdx.x;
        const int v = gcount[min(c, nc - 1)];
        s += c < nc ? v : 0;
    }
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & (kWave - 1)) == 0) wtot[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < kPlaceThreads / kWave; ++k) t += wtot[k];
        seg_tot[b] = t;
    }
}

template <int kSortGroup>
__global__ __launch_bounds__(kPlaceThreads) void k_place(const GridDev* __restrict__ grids,
                                                         int blocks_a,
                                                         const int* __restrict__ seg_tot,
                                                         int nseg_a, int n,
                                                         const int2* __restrict__ key_a,
                                                         const int2* __restrict__ key_s,
                                                         const double4* __restrict__ wpos,
                                                         TopoDev topo, int* __restrict__ user2arow)
{
    constexpr int kWaves = kPlaceThreads / kWave;
    constexpr int kCellsPerWave = kWave / kSortGroup;
    constexpr int kCells = kWaves * kCellsPerWave;     // at most 64: one wave scans them
    __shared__ int wtot[kWaves];
    __shared__ int cnt_sh[kCells], first_sh[kCells];
    __shared__ int wide[kWaves][kPlaceWide];
    const bool site = (int)blockIdx.x >= blocks_a;
    const GridDev& g = grids[site ? 1 : 0];
    const int c0 = ((int)blockIdx.x - (site ? blocks_a : 0)) * kCells;
    const int nc = g.ncell;
    const int cap = g.bucket_cap;
    RELRES_GLOBAL const int* gcount = gbl(g.count);
    RELRES_GLOBAL int* gstart = gbl(g.start);
    RELRES_GLOBAL const int* bucket = gbl(g.user_unsorted);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    // group q of G lanes: cell c0 + wave * kCellsPerWave + q
    const int q = lane / kSortGroup, gl = lane & (kSortGroup - 1);
    const int ci = wave * kCellsPerWave + q;
    const int c = c0 + ci;
    const int in_group = kSortGroup < cap ? kSortGroup : cap;

    // Every read that does not depend on another is issued first: the
    // block's own counts (wave 0), the first in_group bucket slots of each
    // group's cell (whatever the cell's count; slots past it are dropped
    // below) and the counts of the cells before this block's.
    const int own_cnt = (wave == 0 && lane < kCells && c0 + lane < nc) ? gcount[c0 + lane] : 0;
    const int u_slot = (c < nc && gl < in_group) ? bucket[(size_t)c * cap + gl] : 0x7fffffff;
    // members of the grid's cells before this block's: c0 is a multiple of 4,
    // so the counts are read as int4, four loads per thread in flight at once
    // (the first round outside the loop, so its reads go out with the ones
    // above; grids of more than 4096 cells before the block loop further)
    // (global 16-byte reads of clamped index, the ones past the end dropped,
    // so no branch splits them)
    // (with segment totals the counts start at the block's own segment, and
    // the earlier segments' totals are added)
    int s = 0;
    const int seg = seg_tot ? c0 / kPlaceSeg : 0;
    if (seg > 0) {
        const int* __restrict__ tot = seg_tot + (site ? nseg_a : 0);
        for (int k = (int)threadIdx.x; k < seg; k += kPlaceThreads) s += tot[k];
    }
    const int n4 = (c0 - seg * kPlaceSeg) >> 2;
    if (n4 > 0) {
        typedef int int4v __attribute__((ext_vector_type(4)));
        RELRES_GLOBAL const int4v* c4 = (RELRES_GLOBAL const int4v*)(gcount + seg * kPlaceSeg);
        auto round = [&](int base) {
            int4v q4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = base + u * kPlaceThreads + (int)threadIdx.x;
                const int4v v = c4[min(k, n4 - 1)];
                q4[u] = k < n4 ? v : (int4v)(0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) s += (q4[u].x + q4[u].y) + (q4[u].z + q4[u].w);
        };
        round(0);
        for (int base = 4 * kPlaceThreads; base < n4; base += 4 * kPlaceThreads) round(base);
    }
    // the slot's member (position, type, molecule) is read once its index
    // and the counts are in, while the counts are summed and scanned: a slot past its cell's count
    // holds an index of an earlier build (garbage before the first), so only
    // indices below n are read, and such a read is dropped
    const int u_pre = (unsigned)u_slot < (unsigned)n ? u_slot : 0;
    const double4 p_pre = wpos[u_pre];
    const int ty_pre = topo.types[u_pre], mol_pre = topo.mol[u_pre];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) s += __shfl_xor(s, o);
    if (lane == 0) wtot[wave] = s;
    __syncthreads();
    if (wave == 0) {
        int carry = 0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) carry += wtot[k];
        const int v = own_cnt;
        int x = v;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane < kCells) {
            cnt_sh[lane] = v;
            first_sh[lane] = carry + x - v;
            if (c0 + lane < nc) gstart[c0 + lane] = carry + x - v;
            if (c0 + lane == nc - 1) gstart[nc] = carry + x;
        }
    }
    __syncthreads();

    const int len = c < nc ? cnt_sh[ci] : 0;
    const int b = first_sh[ci];
    const bool small = len <= in_group;
    const int u = (small && gl < len) ? u_slot : 0x7fffffff;
    int r = 0;
    if constexpr (kSortGroup < kWave) {
#pragma unroll
        for (int k = 0; k < kSortGroup; ++k) r += __shfl(u, (lane & ~(kSortGroup - 1)) + k) < u;
    } else {
        const int m = small ? len : 0;      // one cell per wave: len is uniform
        for (int k = 0; k < m; ++k) r += __shfl(u, k) < u;
    }
    if (small && gl < len) place_read(g, site, c, b + r, u, p_pre, ty_pre, mol_pre, user2arow);
    // the larger cells of this wave, one at a time with the whole wave
    for (int k = 0; k < kCellsPerWave; ++k) {
        const int lenk = readlane_i(len, k * kSortGroup);
        if (lenk <= in_group) continue;
        const int ck = c0 + wave * kCellsPerWave + k;
        const int bk = readlane_i(b, k * kSortGroup);
        if (lenk <= cap) {                  // cap <= 64: one member per lane
            const int v = lane < lenk ? bucket[(size_t)ck * cap + lane] : 0x7fffffff;
            int rk = 0;
            for (int j = 0; j < lenk; ++j) rk += __shfl(v, j) < v;
            if (lane < lenk) place_member(g, site, ck, bk + rk, v, wpos, topo, user2arow);
            continue;
        }
        const int2* __restrict__ key = site ? key_s : key_a;
        if (lenk <= kPlaceWide) {
            // the cell outgrew its bucket: the members beyond it from its chains,
            // one lane each (dependent reads, 1 / kPlaceChains of them), then all
            // ranked from LDS.  A slab of 405000 atoms in a box ten times as long,
            // every site cell beyond its bucket: build 889 us; 6600 with a pass over
            // the keys for each cell of more than 64 members beyond, and 1172 with
            // the scan, scatter and sort launches
            int* all = wide[wave];
            const int over = lenk - cap;
            if (lane < cap) all[lane] = bucket[(size_t)ck * cap + lane];
            if (lane < kPlaceChains) {
                int j = gbl(g.chain_head)[(size_t)ck * kPlaceChains + lane];
                for (int t = lane; t < over; t += kPlaceChains) {
                    const bool in = (unsigned)j < (unsigned)n;
                    all[cap + t] = in ? j : 0x7fffffff;
                    j = in ? key[j].y : -1;
                }
            }
            wave_lds_fence();
            for (int t = lane; t < lenk; t += kWave) {
                const int v = all[t];
                int rk = 0;
#pragma unroll 8
                for (int u = 0; u < lenk; ++u) rk += all[u] < v;
                if (v != 0x7fffffff) place_member(g, site, ck, bk + rk, v, wpos, topo, user2arow);
            }
            wave_lds_fence();                   // used again for the wave's next cell
            continue;
        }
        // far more members than the bucket holds: in caller order from the keys
        int run = 0;
        for (int i0 = 0; i0 < n; i0 += kWave) {
            const int i = i0 + lane;
            const bool mine = i < n && key[i].x == ck;
            const uint64_t m = __ballot(mine);
            if (mine) place_member(g, site, ck, bk + run + lanes_below(m), i, wpos, topo, user2arow);
            run += __popcll(m);
        }
    }
}

// After a one-launch placement the cell counts are still set: the list
// kernel, the next launch of the build, clears them for the next build (the
// grid array always has two entries; the second repeats the first when there
// are no sites).
__device__ __forceinline__ void clear_bucket_counts(const GridDev* __restrict__ grids)
{
    const int stride = (int)(gridDim.x * blockDim.x);
    for (int gi = 0; gi < 2; ++gi) {
        const GridDev& g = grids[gi];
        if (g.bucket_cap <= 0) continue;
        RELRES_GLOBAL int* cnt = gbl(g.count);
        for (int c = (int)(blockIdx.x * blockDim.x + threadIdx.x); c < g.ncell; c += stride)
            cnt[c] = 0;
    }
}

// A compile-time bool as a value (selects one of two instantiations of a
// generic lambda).
template <bool B>
struct BoolC {
    static constexpr bool value = B;
};

// Stencil geometry: S cells per axis around the home cell (3 for cells of at
// least the list radius, 5 for cells of at least half of it), S^3 slots in
// x-major order, slot tables of kSlotTab entries per wave.
template <int S>
struct Stencil {
    static constexpr int kHalf = S / 2;
    static constexpr int kSlots = S * S * S;
    static constexpr int kTab = S == 3 ? 32 : 128;
    static constexpr int kPerLane = S == 3 ? 1 : 2;   // slots a lane holds: lane, lane + 64
    // the offset of slot s along axis a (0 = x) in cells
    static __device__ __forceinline__ int off(int s, int a)
    {
        const int d = a == 0 ? s / (S * S) : (a == 1 ? (s / S) % S : s % S);
        return d - kHalf;
    }
};

// Global rank of the cell at offset (ox, oy, oz) from the cell (hx, hy, hz)
// of a grid of n cells per axis, or -1 when the offset repeats a cell that a
// smaller offset already reaches (an axis of fewer than S cells keeps its
// first n offsets, which reach every cell once).
template <int S>
__device__ __forceinline__ int stencil_rank(const GeomDev& G, RELRES_GLOBAL const int* grank,
                                            int hx, int hy, int hz, int s)
{
    using St = Stencil<S>;
    if (s >= St::kSlots) return -1;
    const int ox = St::off(s, 0), oy = St::off(s, 1), oz = St::off(s, 2);
    const int n0 = G.n[0], n1 = G.n[1], n2 = G.n[2];
    if ((n0 < S && ox + St::kHalf >= n0) || (n1 < S && oy + St::kHalf >= n1) ||
        (n2 < S && oz + St::kHalf >= n2))
        return -1;
    const int x = (hx + ox + 2 * n0) % n0, y = (hy + oy + 2 * n1) % n1, z = (hz + oz + 2 * n2) % n2;
    return grank[G.cell_base + (x * n1 + y) * n2 + z];
}

// Neighbour lists, one wave per group of R consecutive member rows (rows are
// in cell order, so a group spans one or a few cells).  Work per wave is
// bounded by the group size, so crowded cells are spread over many waves.
// Each lane owns one home row of the group: its position, exclusions and
// running count live in that lane and are broadcast with readlane.  The
// candidates of the home cell's stencil are loaded straight into registers,
// K per lane per round (candidate q in lane q % 64), and every home row of
// the cell tests them there, so a candidate is read from memory once per cell
// and never through LDS.  Candidates are visited in stencil-slot order, each
// row's entries are appended in that order with a wave ballot.  Only
// wave-level synchronisation is used, so waves of one block may run different
// trip counts.  S is the stencil width of the grid the wave's rows belong to
// (3: cells of one list radius; 5: cells of half of it, fewer candidates per
// row and more cells per wave).
//
// Large launches are bound by vector issue, small ones by the chain of one
// wave, so the distance test is a filter in FP32: positions relative to the
// cell's first row (taken in FP64, nearest image, once per candidate and
// cell) are within 2^-24 of their size, and a squared distance outside
// [filter_lo, filter_hi] (GeomDev, an error bound around the list radius) is
// decided by it.  A distance inside (about one test in 10^5) is decided by
// the FP64 membership recipe, so the lists are those of that recipe.  The
// filter takes 8 vector instructions per test instead of 12, 3 lane reads
// per row instead of 6 and a third of the candidate registers (2 candidates:
// 64 or 70 vector registers and 7 to 8 waves per SIMD instead of 88 and 5).
// With the order and shapes of the launch (k_lists_wave, list_rows_per_wave)
// one build went from 106 to 70 us for the 98304-atom copolymer, 607 to 440
// for 256 replicas, 90 to 54 for 48000-atom hexane, 47.6 to 39.6 for 20480
// atoms at 14 A (graph replays of 10 builds).
// MolOnly: the only exclusions are the same-molecule ones.
template <int K, int S, bool MolOnly>
__device__ __forceinline__ void list_wave(const GridDev& g, int wv, int lw, bool site, int max_excl,
                                          const TopoDev& topo, const int* __restrict__ user2arow,
                                          int4* __restrict__ a_rec, int4* __restrict__ s_rec,
                                          Status* __restrict__ st, int* slot_base, int* slot_win,
                                          int* excl_lds)
{
    using St = Stencil<S>;
    const int lane = threadIdx.x & (kWave - 1);
    const double4* gpos = g.pos;      // read through load_member
    RELRES_GLOBAL const int* gstart = gbl(g.start);
    RELRES_GLOBAL const int* gnbr = gbl(g.nbr);
    RELRES_GLOBAL const int* grank = gbl(g.rank_of_lin);
    RELRES_GLOBAL int* glist = gbl(g.list);
    RELRES_GLOBAL const int* glor = gbl(g.lin_of_rank);
    // the system whose grid holds this wave's rows (wave-uniform; grids with
    // no rows have no waves)
    const int gs_lo = g.nsys > 1 ? __builtin_amdgcn_readfirstlane(g.wave_sys[lw]) : 0;
    const GeomDev& G = g.geom[gs_lo];
    // the grid's values are wave-uniform: readfirstlane keeps them in scalar
    // registers, where the compiler would otherwise hold them in vector ones
    const int n0 = __builtin_amdgcn_readfirstlane(G.n[0]);
    const int n1 = __builtin_amdgcn_readfirstlane(G.n[1]);
    const int n2 = __builtin_amdgcn_readfirstlane(G.n[2]);
    const double Lx = readfirst_d(G.box[0]), Ly = readfirst_d(G.box[1]), Lz = readfirst_d(G.box[2]);
    const double iLx = readfirst_d(G.inv_box[0]), iLy = readfirst_d(G.inv_box[1]),
                 iLz = readfirst_d(G.inv_box[2]);
    const float flo = readfirst_f(G.filter_lo), fhi = readfirst_f(G.filter_hi);
    // With enough cells per axis (S = 3: 5, S = 5: 7) every stencil cell is
    // less than half a box from the home cell's rows, so the difference of two
    // positions relative to one of those rows is their nearest image already.
    // (wave-uniform; readfirstlane makes the choice a scalar branch)
    constexpr int kDirect = S == 3 ? 5 : 7;
    const bool direct = __builtin_amdgcn_readfirstlane(n0 >= kDirect && n1 >= kDirect &&
                                                       n2 >= kDirect);
    const int R = g.rows_per_wave;
    const int r0 = __builtin_amdgcn_readfirstlane(G.row_base + (lw - G.wave_base) * R);
    const int r1 = __builtin_amdgcn_readfirstlane(min(G.row_base + G.members, r0 + R));
    const int cap = g.cap;
    const int* __restrict__ excl_off = topo.excl_off;
    const int* __restrict__ excl_idx = topo.excl_idx;
    const int same_mol = MolOnly ? 1 : topo.same_mol;
    // exclusion lists of the wave's home rows, staged once (kRowsPerWave x max_excl)
    int* my_excl = excl_lds + wv * kRowsPerWave * max_excl;

    // lane h < (r1 - r0) owns home row r0 + h
    const int nh = r1 - r0;
    const int myrow = r0 + lane;
    double mx = 0.0, my = 0.0, mz = 0.0;
    int mt = 0, mmol = 0;
    int mu = -1, marow = 0, mcell = -1, mcnt = 0;
    // The row's exclusions with itself: where they fill the index range
    // [mlo, mlo + mspan] (chains with their bonded neighbours excluded; a row
    // without exclusions, by itself), one unsigned compare tests them all and
    // mne is 0; otherwise mne of them are staged in LDS (the row itself is
    // tested by the range).
    int mlo = -1, mspan = 0, mne = 0;
    if (lane < nh) {
        uint32_t ment;
        load_member(gpos, myrow, mx, my, mz, ment, mmol);
        mu = (int)(ment & kIdxMask);
        mt = (int)(ment >> kIdxBits);
        mcell = gbl(g.row_cell)[myrow];
        if constexpr (!MolOnly) {
            mlo = mu;
            if (excl_off) {
                const int meb = excl_off[mu];
                const int ne = excl_off[mu + 1] - meb;
                if (ne > 0) {
                    const int first = min(mu, excl_idx[meb]), last = max(mu, excl_idx[meb + ne - 1]);
                    if (last - first == ne) {
                        mlo = first;
                        mspan = ne;
                    } else {
                        mne = ne;
                        for (int k = 0; k < ne; ++k) my_excl[lane * max_excl + k] = excl_idx[meb + k];
                    }
                }
            }
        }
        if (site) marow = user2arow[mu];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // The stencil slots a lane holds (slot `lane`, and `lane + 64` for the
    // 125-cell stencil) of a home cell: the slot's cell (rank, or -1), then
    // the first member and the end of its member range.  The next home cell's
    // reads are issued while this cell is processed (the ranks before this
    // cell's first candidate reads, the ranges at its first round), so the
    // dependent reads leave the per-cell critical path.  The range reads are
    // unconditional (lanes past the stencil and empty slots read a valid entry
    // and drop it at use), so no branch makes the compiler wait for them early.
    int next_rank[St::kPerLane];
    auto ranks_of = [&](int h) {
        const int c = readlane_i(mcell, h);
        if constexpr (S == 3) {
            next_rank[0] = gnbr[c * 27 + min(lane, 26)];
        } else {
            const int lin = __builtin_amdgcn_readfirstlane(glor[c]);
            const int cz = lin % n2, cy = (lin / n2) % n1, cx = lin / (n1 * n2);
#pragma unroll
            for (int u = 0; u < St::kPerLane; ++u)
                next_rank[u] = stencil_rank<S>(G, grank, cx, cy, cz, lane + kWave * u);
        }
    };
    auto no_ranks = [&]() {
#pragma unroll
        for (int u = 0; u < St::kPerLane; ++u) next_rank[u] = -1;
    };
    auto slot_valid = [&](int u) {
        return lane + kWave * u < St::kSlots && next_rank[u] >= 0;
    };
    if (nh > 0) ranks_of(0); else no_ranks();
    int next_lo[St::kPerLane], next_hi[St::kPerLane];
    auto range_of = [&]() {
#pragma unroll
        for (int u = 0; u < St::kPerLane; ++u) {
            int r = next_rank[u];
            // keeps the rank's first use here, after this cell's candidate
            // loads were issued: hoisted ahead of them, it would make the
            // wave wait for the rank read first
            asm volatile("" : "+v"(r));
            r = lane + kWave * u < St::kSlots && r >= 0 ? r : 0;
            next_lo[u] = gstart[r];
            next_hi[u] = gstart[r + 1];
        }
    };
    if (nh > 0) range_of();
    int h0 = 0;
    while (h0 < nh) {
        // rows h0 .. h1-1 share one cell
        const int c = readlane_i(mcell, h0);
        int h1 = h0 + 1;
        while (h1 < nh && readlane_i(mcell, h1) == c) ++h1;
        h1 = __builtin_amdgcn_readfirstlane(h1);   // wave-uniform: a scalar row loop
        int s0[St::kPerLane], cnt[St::kPerLane];
#pragma unroll
        for (int u = 0; u < St::kPerLane; ++u) {
            const bool ok = slot_valid(u);
            s0[u] = ok ? next_lo[u] : 0;
            cnt[u] = ok ? next_hi[u] - next_lo[u] : 0;
        }
        if (h1 < nh) ranks_of(h1); else no_ranks();
        // the cell's reference point and its rows relative to it (rows of one
        // cell: no image shift between them)
        const double rx = readlane_d(mx, h0), ry = readlane_d(my, h0), rz = readlane_d(mz, h0);
        const float ax = (float)(mx - rx), ay = (float)(my - ry), az = (float)(mz - rz);
        // first candidate of every slot: a wave scan of the counts in slot
        // order (slot lane, then slot lane + 64)
        int ncand = 0;
        int first[St::kPerLane];
#pragma unroll
        for (int u = 0; u < St::kPerLane; ++u) {
            const int pre = wave_inclusive_scan(cnt[u]);
            const int slot = lane + kWave * u;
            first[u] = ncand + pre - cnt[u];
            if (slot < St::kTab) {
                // member index of candidate q of this slot: slot_base + q
                slot_base[slot] = s0[u] - first[u];
            }
            ncand += __builtin_amdgcn_readlane(pre, kWave - 1);
        }
        int carry = -1;      // the slot of candidate cb - 1
        for (int cb = 0; cb < ncand; cb += kWave * K) {
            // The slot of each of the round's 64 K candidates (cb + p for p =
            // lane + 64 k): every non-empty slot marks its first candidate in
            // a window of the round (candidate cb + p at (p % 64) K + p / 64,
            // so a lane's K entries are one vector read), and a running
            // maximum in candidate order carries each mark over the slot's
            // other candidates.
#pragma unroll
            for (int k = 0; k < K; ++k) slot_win[lane * K + k] = -1;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int u = 0; u < St::kPerLane; ++u) {
                const int p = first[u] - cb;
                if (cnt[u] > 0 && p >= 0 && p < kWave * K)
                    slot_win[(p & (kWave - 1)) * K + (p >> 6)] = lane + kWave * u;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            int cslot[K];
#pragma unroll
            for (int k = 0; k < K; ++k) cslot[k] = slot_win[lane * K + k];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                cslot[k] = max(wave_inclusive_max(cslot[k]), carry);
                carry = __builtin_amdgcn_readlane(cslot[k], kWave - 1);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            double qx[K], qy[K], qz[K];
            int pi[K];          // member index of the candidate, -1: none
            uint32_t pe[K];     // the candidate's list entry
            int pm[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = cb + lane + kWave * k;
                qx[k] = qy[k] = qz[k] = 0.0;
                pe[k] = 0;
                pm[k] = 0;
                pi[k] = -1;
                if (q < ncand) {
                    pi[k] = slot_base[max(cslot[k], 0)] + q;
                    load_member(gpos, pi[k], qx[k], qy[k], qz[k], pe[k], pm[k]);
                }
            }
            // the next cell's member ranges (its stencil ranks were read at
            // this cell's start), issued after this cell's first candidate
            // reads and once per cell, outside the rows' loop
            if (cb == 0) range_of();
            // the candidates relative to the reference point, nearest image
            // (an empty slot lies at infinity: no test passes it)
            float px[K], py[K], pz[K];
            int pu[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double dx = qx[k] - rx, dy = qy[k] - ry, dz = qz[k] - rz;
                px[k] = pi[k] >= 0 ? (float)(dx - Lx * rint(dx * iLx)) : __builtin_inff();
                py[k] = (float)(dy - Ly * rint(dy * iLy));
                pz[k] = (float)(dz - Lz * rint(dz * iLz));
                pu[k] = (int)(pe[k] & kIdxMask);
            }
            // The conditions of a (row, candidate) pair are wave lane masks,
            // one per k, combined with scalar ANDs.  The rows' loop is
            // instantiated for differences that are the nearest image already
            // and for those that are not, so the choice is one scalar branch
            // per round and not a select per test.  Every cell has at least
            // one home row (h1 > h0): a loop that always runs, so no path
            // skips it with candidate reads pending.
            auto row_loop = [&](auto near) {
            constexpr bool kNear = decltype(near)::value;
            const float fLx = (float)Lx, fLy = (float)Ly, fLz = (float)Lz;
            int h = __builtin_amdgcn_readfirstlane(h0);
            do {
                const float xi = readlane_f(ax, h), yi = readlane_f(ay, h), zi = readlane_f(az, h);
                int hc = readlane_i(mcnt, h);
                RELRES_GLOBAL int* out =
                    glist + (size_t)__builtin_amdgcn_readfirstlane(r0 + h) * cap;
                uint64_t drop[K];
#pragma unroll
                for (int k = 0; k < K; ++k) drop[k] = 0ull;
                // the row's own atom shares its molecule: with the
                // same-molecule exclusion, one test drops both
                if (same_mol) {
                    const int moli = readlane_i(mmol, h);
#pragma unroll
                    for (int k = 0; k < K; ++k) drop[k] = __ballot(pm[k] == moli);
                }
                if constexpr (!MolOnly) {
                    const int lo = readlane_i(mlo, h), span = readlane_i(mspan, h);
                    const int ne = readlane_i(mne, h);
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        drop[k] |= __ballot((unsigned)(pu[k] - lo) <= (unsigned)span);
                    // scattered exclusions: each read once for all K
                    // candidates, four reads in flight (past the end, the
                    // last one again)
                    const int* hex = my_excl + h * max_excl;
                    for (int e = 0; e < ne; e += 4) {
                        int x[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) x[v] = hex[min(e + v, ne - 1)];
#pragma unroll
                        for (int v = 0; v < 4; ++v)
#pragma unroll
                            for (int k = 0; k < K; ++k) drop[k] |= __ballot(pu[k] == x[v]);
                    }
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (cb + kWave * k >= ncand) break;
                    float dx = px[k] - xi, dy = py[k] - yi, dz = pz[k] - zi;
                    if constexpr (!kNear) {
                        dx = fminf(fabsf(dx), fLx - fabsf(dx));
                        dy = fminf(fabsf(dy), fLy - fabsf(dy));
                        dz = fminf(fabsf(dz), fLz - fabsf(dz));
                    }
                    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
                    uint64_t mask = __ballot(!(r2 > fhi)) & ~drop[k];
                    const uint64_t open = mask & ~__ballot(r2 < flo);
                    if (__builtin_expect(open != 0ull, 0)) {
                        // too close to the list radius for the filter: the
                        // FP64 recipe on the members' own positions
                        bool in = false;
                        if (__builtin_amdgcn_inverse_ballot_w64(open) && pi[k] >= 0) {
                            double x, y, z;
                            uint32_t e;
                            int m;
                            load_member(gpos, pi[k], x, y, z, e, m);
                            in = member(make_double4(readlane_d(mx, h), readlane_d(my, h),
                                                     readlane_d(mz, h), 0.0),
                                        make_double4(x, y, z, 0.0), Lx, Ly, Lz, 0.5 * Lx, 0.5 * Ly,
                                        0.5 * Lz, G.rl2);
                        }
                        mask = (mask & ~open) | __ballot(in);
                    }
                    if (__builtin_amdgcn_inverse_ballot_w64(mask)) {
                        // 32-bit slot index: the store takes the row's scalar
                        // base and one lane offset
                        const uint32_t p = (uint32_t)(hc + lanes_below(mask));
                        if (p < (uint32_t)cap) out[p] = (int)pe[k];
                    }
                    hc += __popcll(mask);
                }
                if (lane == h) mcnt = hc;
            } while (++h < h1);
            };
            if (direct) row_loop(BoolC<true>());
            else row_loop(BoolC<false>());
        }
        if (ncand == 0) range_of();
        // the slot table is rewritten for the next cell
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        h0 = h1;
    }
    if (lane < nh) {
        gbl(g.nrow)[myrow] = mcnt;
        const int stored = min(mcnt, cap);
        const int ty = mt | (gs_lo << kTypeBits);
        if (site) s_rec[myrow] = make_int4(mu, ty, stored, marow);
        else a_rec[myrow] = make_int4(mu, ty, stored, topo.hybrid[mt]);
    }
    // only a row that outgrew its capacity touches the status word (rare), so
    // thousands of waves do not serialise on one address
    if (lane < nh && mcnt > cap) atomicMax(&st->max_row[site ? 1 : 0], mcnt);
}

// One launch for both grids; SA and SS are the stencil widths of the two
// grids.  The waves of the site list come first: their stencils hold two to
// three times the candidates of an atom wave's, and started last they ran on
// alone at the end of the launch (98304-atom copolymer: build 76 against 71
// us; 48000-atom hexane 69 against 61; 256 replicas 454 against 442).
template <int K, int SA, int SS, bool MolOnly>
__global__ __launch_bounds__(256, K == 2 ? (MolOnly ? 8 : 7) : 1) void k_lists_wave(const GridDev* __restrict__ grids,
                                                    int waves_a, int waves_total, int max_excl,
                                                    TopoDev topo,
                                                    const int* __restrict__ user2arow,
                                                    int4* __restrict__ a_rec,
                                                    int4* __restrict__ s_rec,
                                                    Status* __restrict__ st)
{
    __shared__ int slot_base[4][Stencil<(SA > SS ? SA : SS)>::kTab];
    __shared__ __align__(16) int slot_win[4][kWave * K];
    extern __shared__ int excl_lds[];
    // wave-uniform by construction; readfirstlane lets the compiler keep it
    // (and everything derived from it) in scalar registers
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int gw = blockIdx.x * 4 + wv;
    if (gw < waves_total) {                   // whole wave; no block barriers below
        const int waves_s = waves_total - waves_a;
        const bool site = gw < waves_s;
        const int lw = site ? gw : gw - waves_s;
        if (site)
            list_wave<K, SS, MolOnly>(grids[1], wv, lw, true, max_excl, topo, user2arow, a_rec,
                                      s_rec, st, slot_base[wv], slot_win[wv], excl_lds);
        else
            list_wave<K, SA, MolOnly>(grids[0], wv, lw, false, max_excl, topo, user2arow, a_rec,
                                      s_rec, st, slot_base[wv], slot_win[wv], excl_lds);
    }
    clear_bucket_counts(grids);   // last: the stores leave the start of the kernel alone
}

// Neighbour lists: one block per home cell (atom-grid cells first, then
// site-grid cells).  Rows are padded to the grid's capacity; the true count
// is stored even when it exceeds the capacity, so the host can regrow.
__global__ __launch_bounds__(kListBlock) void k_lists(const GridDev* __restrict__ grids,
                                                      int ncell_a, TopoDev topo,
                                                      const int* __restrict__ user2arow,
                                                      int4* __restrict__ a_rec,
                                                      int4* __restrict__ s_rec,
                                                      Status* __restrict__ st)
{
    __shared__ double4 c_pos[kChunk];
    __shared__ int2 c_meta[kChunk];
    __shared__ int c_user[kChunk];
    __shared__ int cell_start[27], cell_cnt[27], cell_pre[28];
    __shared__ int ncells_sh;
    __shared__ int home_cnt[kHomeMax];
    __shared__ int blk_max;
    __shared__ unsigned long long blk_sum;

    clear_bucket_counts(grids);
    const bool site = (int)blockIdx.x >= ncell_a;
    const GridDev& g = grids[site ? 1 : 0];
    const int c = site ? (int)blockIdx.x - ncell_a : (int)blockIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;

    if (threadIdx.x < 27) {
        // one lane per stencil slot: neighbour rank from the host-built table
        const int t = threadIdx.x;
        const int r = g.nbr[c * 27 + t];
        int cnt = -1, s0 = 0;
        if (r >= 0) {
            s0 = g.start[r];
            cnt = g.start[r + 1] - s0;
        }
        cell_start[t] = s0;
        cell_cnt[t] = cnt;
    }
    if (threadIdx.x == 0) {
        blk_max = 0;
        blk_sum = 0ull;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int k = 0, acc = 0;
        for (int t = 0; t < 27; ++t) {
            if (cell_cnt[t] < 0) continue;
            cell_start[k] = cell_start[t];
            cell_pre[k] = acc;
            acc += cell_cnt[t];
            ++k;
        }
        cell_pre[k] = acc;
        ncells_sh = k;
    }
    __syncthreads();
    const int ncells = ncells_sh;
    const int ncand = cell_pre[ncells];
    const int hb = g.start[c];
    const int he = g.start[c + 1];
    const GeomDev& G = g.geom[g.cell_sys[c]];
    const double Lx = G.box[0], Ly = G.box[1], Lz = G.box[2];
    const double hx = G.half[0], hy = G.half[1], hz = G.half[2];
    const double rl2 = G.rl2;
    const int cap = g.cap;

    for (int hg = hb; hg < he; hg += kHomeMax) {
        const int nh = min(kHomeMax, he - hg);
        for (int h = threadIdx.x; h < nh; h += blockDim.x) home_cnt[h] = 0;
        for (int cb = 0; cb < ncand; cb += kChunk) {
            const int clen = min(kChunk, ncand - cb);
            __syncthreads();
            for (int t = threadIdx.x; t < clen; t += blockDim.x) {
                const int q = cb + t;
                int k = 0;
                while (k + 1 < ncells && cell_pre[k + 1] <= q) ++k;
                const int src = cell_start[k] + (q - cell_pre[k]);
                c_pos[t] = g.pos[src];
                c_meta[t] = g.meta[src];
                c_user[t] = g.user[src];
            }
            __syncthreads();
            for (int h = wave; h < nh; h += nw) {
                const int row = hg + h;
                const double4 pi = g.pos[row];
                const int2 mi = g.meta[row];
                const int ui = g.user[row];
                int eb = 0, ne = 0;
                if (topo.excl_off) {
                    eb = topo.excl_off[ui];
                    ne = min(topo.excl_off[ui + 1] - eb, kWave);
                }
                const int myex = lane < ne ? topo.excl_idx[eb + lane] : -1;
                int cnt = home_cnt[h];
                int* out = g.list + (size_t)row * cap;
                for (int base = 0; base < clen; base += kWave) {
                    const int t = base + lane;
                    bool keep = false;
                    uint32_t entry = 0u;
                    if (t < clen) {
                        const int uj = c_user[t];
                        const int2 mj = c_meta[t];
                        keep = uj != ui && !(topo.same_mol && mj.y == mi.y);
                        for (int k = 0; k < ne; ++k)
                            if (__shfl(myex, k) == uj) keep = false;
                        if (keep) keep = member(pi, c_pos[t], Lx, Ly, Lz, hx, hy, hz, rl2);
                        entry = (uint32_t)uj | ((uint32_t)mj.x << kIdxBits);
                    }
                    const uint64_t mask = __ballot(keep);
                    if (keep) {
                        const int p = cnt + lanes_below(mask);
                        if (p < cap) out[p] = (int)entry;
                    }
                    cnt += __popcll(mask);
                }
                if (lane == 0) home_cnt[h] = cnt;
            }
        }
        __syncthreads();
        for (int h = threadIdx.x; h < nh; h += blockDim.x) {
            const int row = hg + h;
            const int cnt = home_cnt[h];
            g.nrow[row] = cnt;
            atomicMax(&blk_max, cnt);
            atomicAdd(&blk_sum, (unsigned long long)cnt);
            // packed row record for the force kernel: one load per row
            const int u = g.user[row];
            const int ty = g.meta[row].x;
            const int stored = min(cnt, cap);
            const int tys = ty | (g.cell_sys[c] << kTypeBits);
            if (site) s_rec[row] = make_int4(u, tys, stored, user2arow[u]);
            else a_rec[row] = make_int4(u, tys, stored, topo.hybrid[ty]);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && blk_max > cap) atomicMax(&st->max_row[site ? 1 : 0], blk_max);
}

// Exact list statistics on demand: entries (sum of row lengths) and the
// longest row of each grid (blockIdx.y), added to the cleared fields of *st.
// One thread per kStatRows rows, so that the rows of a large system are read by
// the whole chip: with one block per grid it took 1.3 ms on 256 replicas of 1.2
// million atoms and 105 us on 98304 atoms, now 21 and 4 us.
constexpr int kStatRows = 8;

__global__ void k_clear_stats(Status* st)
{
    if (threadIdx.x < 2) {
        st->entries[threadIdx.x] = 0ull;
        st->longest[threadIdx.x] = 0;
    }
}

__global__ __launch_bounds__(256) void k_list_stats(const GridDev* __restrict__ grids,
                                                    Status* __restrict__ st)
{
    __shared__ unsigned long long ssum[256 / kWave];
    __shared__ int smax[256 / kWave];
    const GridDev& g = grids[blockIdx.y];
    const int members = g.members;
    unsigned long long sum = 0ull;
    int mx = 0;
    RELRES_GLOBAL const int* gnrow = gbl(g.nrow);
#pragma unroll
    for (int u = 0; u < kStatRows; ++u) {
        const long long r = ((long long)blockIdx.x * kStatRows + u) * 256 + threadIdx.x;
        const int c = r < members ? gnrow[r] : 0;
        sum += (unsigned long long)c;
        mx = max(mx, c);
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o);
        mx = max(mx, __shfl_xor(mx, o));
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (lane == 0) {
        ssum[wave] = sum;
        smax[wave] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / kWave; ++w) {
            ssum[0] += ssum[w];
            smax[0] = max(smax[0], smax[w]);
        }
        if (ssum[0] > 0) {             // whole numbers: the order does not matter
            atomicAdd(&st->entries[blockIdx.y], ssum[0]);
            atomicMax(&st->longest[blockIdx.y], smax[0]);
        }
    }
}

// ---------------------------------------------------------------------------
// force kernel
// ---------------------------------------------------------------------------

// Coefficient table staged in LDS when it is small (ntypes <= kLdsTypes).
constexpr int kLdsTypes = 8;

// FP32 launches with energy and virial (Mixed) evaluate every term in FP64 and
// read the FP64 table only.
template <typename S, bool EW>
constexpr bool kMixed = EW && sizeof(S) != sizeof(double);

template <typename S, bool EW>
struct CoefLds {
    PairCoef<S> c[kMixed<S, EW> ? 1 : kLdsTypes * kLdsTypes];
    PairCoef<double> c64[kMixed<S, EW> ? kLdsTypes * kLdsTypes : 1];
};

// Distances per type pair, staged when they are not uniform (PC).
template <typename S, bool EW, bool PC>
struct CutLds {
    Cutoffs<S> c[PC && !kMixed<S, EW> ? kLdsTypes * kLdsTypes : 1];
    Cutoffs<double> c64[PC && sizeof(S) != sizeof(double) ? kLdsTypes * kLdsTypes : 1];
};

// The coefficient and distance rows of one row atom's type: pair-math
// coefficients, FP64 coefficients (energy and virial), and with per-pair
// distances (PC) the distance rows in both types.
template <typename S>
struct RowTab {
    const PairCoef<S>* c;
    const PairCoef<double>* c64;
    const Cutoffs<S>* cut;
    const Cutoffs<double>* cut64;
};

// A table of `count` T staged in LDS in two parts: stage_first reads word
// threadIdx.x (issued early, before the row record), stage_table writes it and
// copies any words beyond the first blockDim.x.
template <typename T>
__device__ __forceinline__ uint32_t stage_first(const T* __restrict__ src, int count)
{
    const int words = count * (int)(sizeof(T) / sizeof(uint32_t));
    return (int)threadIdx.x < words ? reinterpret_cast<const uint32_t*>(src)[threadIdx.x] : 0u;
}
template <typename T>
__device__ __forceinline__ void stage_table(T* dst, const T* __restrict__ src, int count,
                                            uint32_t first)
{
    const int words = count * (int)(sizeof(T) / sizeof(uint32_t));
    const uint32_t* s = reinterpret_cast<const uint32_t*>(src);
    uint32_t* d = reinterpret_cast<uint32_t*>(dst);
    if ((int)threadIdx.x < words) d[threadIdx.x] = first;
    for (int k = threadIdx.x + blockDim.x; k < words; k += blockDim.x) d[k] = s[k];
}

// Entries handled per lane per batch (see row_terms).
constexpr int kBatch = 2;
// ... and in forces-only launches of at least 8 entries per lane (issue-bound
// launches of large systems), where more gathers in flight per lane pay: the
// 256-replica batch's forces-only launch took 157 against 180 us, while every
// energy/virial launch and the launches of small systems were slower with 4.
constexpr int kBatchWide = 4;

constexpr uint32_t kNoEntry = 0xffffffffu;

// Periodic box of a system: edges and their reciprocals.
struct BoxV {
    double L[3], iL[3];
};

// The box of a wave whose rows all belong to system `sys`, in scalar registers.
__device__ __forceinline__ BoxV wave_box(const ForceArgs& a, int sys)
{
    BoxV b;
    if (a.nsys == 1) {
        for (int k = 0; k < 3; ++k) {
            b.L[k] = a.box[k];
            b.iL[k] = a.inv_box[k];
        }
    } else {
        for (int k = 0; k < 3; ++k) {
            b.L[k] = readfirst_d(a.boxes[6 * sys + k]);
            b.iL[k] = readfirst_d(a.boxes[6 * sys + 3 + k]);
        }
    }
    return b;
}

__device__ __forceinline__ BoxV row_box(const ForceArgs& a, int sys)
{
    BoxV b;
    if (a.nsys == 1) {
        for (int k = 0; k < 3; ++k) {
            b.L[k] = a.box[k];
            b.iL[k] = a.inv_box[k];
        }
    } else {
        for (int k = 0; k < 3; ++k) {
            b.L[k] = a.boxes[6 * sys + k];
            b.iL[k] = a.boxes[6 * sys + 3 + k];
        }
    }
    return b;
}

// Pair terms of one list entry, the FG part (CG = false, zero beyond r_s+) or
// the CG part (CG = true, zero beyond r_c+) of Eq. 20, with the neighbour's
// position already loaded.  Differences are taken in FP64 with the minimum
// image.  Force terms are evaluated in S and accumulated in TF; energy and
// virial terms are evaluated in FP64 and accumulated in FP64 (when they are
// requested, the FP32 force is rounded from the same FP64 terms).
template <bool CG, typename S, typename TF, bool EW, bool PC>
__device__ __forceinline__ void entry_terms(const BoxV& bx, const RowTab<S>& t,
                                            const Cutoffs<S>& cut_all,
                                            const Cutoffs<double>& cut64_all,
                                            double xi, double yi, double zi, uint32_t e,
                                            double px, double py, double pz,
                                            TF& fx, TF& fy, TF& fz, double* acc)
{
    if (e == kNoEntry) return;
    const int tj = (int)(e >> kIdxBits);
    const Cutoffs<double>& cut64 = PC ? t.cut64[tj] : cut64_all;
    const double rmax2 = CG ? cut64.rco2 : cut64.rso2;
    double dx = xi - px;
    double dy = yi - py;
    double dz = zi - pz;
    dx -= bx.L[0] * rint(dx * bx.iL[0]);
    dy -= bx.L[1] * rint(dy * bx.iL[1]);
    dz -= bx.L[2] * rint(dz * bx.iL[2]);
    const double r2d = dx * dx + dy * dy + dz * dz;
    if (!(r2d < rmax2)) return;
    if constexpr (sizeof(S) == sizeof(double) || EW) {
        // FP64 pair terms (full precision in FP64 mode; one Newton step when
        // they only feed energy/virial and FP32 forces)
        using M = MathF64<sizeof(S) == sizeof(double) ? 2 : 1>;
        double fpd, end;
        if constexpr (CG) cg_term<M>(t.c64[tj], cut64, r2d, fpd, end);
        else fg_term<M>(t.c64[tj], cut64, r2d, fpd, end);
        const double gx = fpd * dx, gy = fpd * dy, gz = fpd * dz;
        if constexpr (sizeof(TF) == sizeof(double)) {
            fx = fma(fpd, dx, fx);     // no rounding of the product
            fy = fma(fpd, dy, fy);
            fz = fma(fpd, dz, fz);
        } else {
            fx += (float)gx;
            fy += (float)gy;
            fz += (float)gz;
        }
        if constexpr (EW) {            // twice the sums: halved at the end
            acc[CG ? 1 : 0] += end;
            acc[2] += gx * dx;
            acc[3] += gy * dy;
            acc[4] += gz * dz;
            acc[5] += gx * dy;
            acc[6] += gx * dz;
            acc[7] += gy * dz;
        }
    } else {
        float fp, en;
        const Cutoffs<S>& cut = PC ? t.cut[tj] : cut_all;
        if constexpr (CG) cg_term<MathF32>(t.c[tj], cut, (float)r2d, fp, en);
        else fg_term<MathF32>(t.c[tj], cut, (float)r2d, fp, en);
        fx += fp * (float)dx;
        fy += fp * (float)dy;
        fz += fp * (float)dz;
    }
}

// Positions of a batch of entries (entry-less slots read atom 0, unused).
template <int B>
__device__ __forceinline__ void gather_batch(const ForceArgs& a, const uint32_t e[B],
                                             double px[B], double py[B], double pz[B])
{
#pragma unroll
    for (int u = 0; u < B; ++u) {
        const int uj = e[u] != kNoEntry ? (int)(e[u] & kIdxMask) : 0;
        px[u] = a.pos[3 * uj];
        py[u] = a.pos[3 * uj + 1];
        pz[u] = a.pos[3 * uj + 2];
    }
}

// Entries start, start + G, ... below cnt of one list row, B per lane at
// a time: their list loads, then their position gathers, are issued together
// before any pair term is computed.
template <bool CG, typename S, typename TF, bool EW, bool PC, int B>
__device__ __forceinline__ void row_terms(const ForceArgs& a, const BoxV& bx,
                                          const RowTab<S>& t,
                                          const Cutoffs<S>& cut, const Cutoffs<double>& cut64,
                                          double xi, double yi, double zi,
                                          const int* __restrict__ lst, int start, int cnt, int G,
                                          TF& fx, TF& fy, TF& fz, double* acc)
{
    for (int base = start; base < cnt; base += G * B) {
        uint32_t e[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int k = base + u * G;
            e[u] = k < cnt ? (uint32_t)lst[k] : kNoEntry;
        }
        double px[B], py[B], pz[B];
        gather_batch<B>(a, e, px, py, pz);
#pragma unroll
        for (int u = 0; u < B; ++u)
            entry_terms<CG, S, TF, EW, PC>(bx, t, cut, cut64, xi, yi, zi, e[u], px[u], py[u],
                                           pz[u], fx, fy, fz, acc);
    }
}


// ---------------------------------------------------------------------------
// Energy/virial reduction across the blocks of one force launch
// ---------------------------------------------------------------------------
// Each block's 8 partial sums (energy FG, CG, virial xx yy zz xy xz yz) are
// published as one record of 16 64-bit words: the high and low 32-bit halves
// of every double, each paired with a 32-bit launch tag.  64-bit stores are
// single-copy atomic, so a reader that sees the current tag in a word sees
// that word's payload; no store ever has to be waited for, and no atomic
// read-modify-write (which serialise on one address) is needed.  The tag is
// the device epoch + 1; the epoch advances once per launch.
//
// Launches of more than kEwDirect blocks: blocks b with b % 16 == g form group
// g (16 groups: fewer records for each group's waiting block to poll than with
// 8, and still one poll round for the 16 group records).  The highest-numbered
// block of each group waits for the records of the rest of its group and
// publishes the group sum; block nb-1 (the highest of all) then waits for the
// group records and writes energy and virial.  In smaller launches block nb-1
// waits for all the others itself, one wait in place of two: 1500 propane atoms
// (FP64, 128 blocks) 7.5 us a launch with two, 6.9 with one; at 200 blocks the
// two are even, and at 400 the records of one wait queue on one CU (1 us
// slower).  A launch with energy and virial is 2.5 to 4 us longer than one with
// forces only: about 0.8 for the block's sum and its record, the rest these
// waits, each a store and a load through the level all XCDs share.
//
// A waiting block only ever waits for blocks with lower numbers, which the
// hardware dispatched before it, so every wait ends; it is bounded anyway
// (a.spin_limit polls; a negative limit gives up at once), after which energy
// and virial are set to NaN and the status counts the failure, which the host
// reports (relres_sync, relres_check_lists).  Sums are taken in a fixed order:
// the result does not depend on which block finished when.
constexpr int kRecWords = 16;
constexpr int kEwDirect = 128;

// Writes one record: called by the whole block, `v` valid in threads 0..7
// (component threadIdx.x).  Lanes 0..15 of wave 0 store word threadIdx.x, so
// the record goes out as one contiguous 128-byte write, written through to
// the level all XCDs share.
__device__ __forceinline__ void put_record(unsigned long long* rec, double v, unsigned tag)
{
    if (threadIdx.x < 64) {
        const double c = __shfl(v, (int)(threadIdx.x >> 1));
        const unsigned long long bits = (unsigned long long)__double_as_longlong(c);
        const unsigned long long half = (threadIdx.x & 1) ? (bits & 0xffffffffull) : (bits >> 32);
        const unsigned long long word = ((unsigned long long)tag << 32) | half;
        if (threadIdx.x < kRecWords)
            __hip_atomic_store(rec + threadIdx.x, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Waits for `count` records (record m at rec + (first + stride*m) * 16 words)
// to carry `tag` and adds them up.  Sixteen consecutive lanes read the sixteen
// words of one record, so every load instruction covers whole records.  Returns,
// in the even ones of the first 16 lanes of each wave, the sum of component
// lane / 2 over the wave's records.  Sets *failed if a wait gave up.  (Two or
// three polls in flight, 80 to 270 ns apart, saw the records no sooner.)
template <int kPollBatch>      // records polled per thread at once
__device__ __forceinline__ double gather_records(const unsigned long long* rec, int first, int stride,
                                                 int count, unsigned tag, int spin_limit, int* failed)
{
    const int t = (int)threadIdx.x;
    const int word = t & (kRecWords - 1);
    double sum = 0.0;
    for (int base = 0; base < count; base += (kForceBlock / kRecWords) * kPollBatch) {
        // every slot loads on every poll (slots past `count` re-read the
        // first record), so all loads of a poll are in flight together; a
        // record already complete is final for this launch
        unsigned off[kPollBatch];
        bool valid[kPollBatch];
#pragma unroll
        for (int u = 0; u < kPollBatch; ++u) {
            const int m = base + t / kRecWords + (kForceBlock / kRecWords) * u;
            valid[u] = m < count;
            off[u] = (unsigned)(first + stride * (valid[u] ? m : 0)) * kRecWords + word;
        }
        unsigned long long w[kPollBatch];
        for (int it = 0;; ++it) {
#pragma unroll
            for (int u = 0; u < kPollBatch; ++u)
                w[u] = __hip_atomic_load(rec + off[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bool pending = spin_limit < 0;          // give up at once
#pragma unroll
            for (int u = 0; u < kPollBatch; ++u) pending |= valid[u] && (unsigned)(w[u] >> 32) != tag;
            if (!pending) break;
            if (it >= spin_limit) {
                *failed = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
#pragma unroll
        for (int u = 0; u < kPollBatch; ++u) {
            const unsigned lo = (unsigned)__shfl_down((unsigned)(w[u] & 0xffffffffull), 1);
            if (!(word & 1) && valid[u])
                sum += __longlong_as_double((long long)(((w[u] & 0xffffffffull) << 32) | lo));
        }
    }
    sum += __shfl_xor(sum, kRecWords);
    return sum + __shfl_xor(sum, 2 * kRecWords);
}

// Fixed-order block reduction of v[8]: result in threads 0..7 (component
// threadIdx.x) as the return value.
__device__ __forceinline__ double block_reduce8(const double v[8], double (*red)[kForceBlock / 64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double s = wave_sum8(v);
    if (lane < 8) red[wave_sum8_lane(lane)][wave] = s;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < 8)
        for (int w = 0; w < kForceBlock / 64; ++w) t += red[threadIdx.x][w];
    return t;
}

__device__ void ew_finish(const ForceArgs& a, const double acc[8], unsigned tag)
{
    __shared__ double red[8][kForceBlock / 64], red2[8][kForceBlock / 64];
    __shared__ int failed;
    const int nb = (int)gridDim.x;
    const int b = (int)blockIdx.x;
    const int lg = nb <= kEwDirect ? 0 : kEwLogGroups;
    const int groups = 1 << lg;
    const int g = b & (groups - 1);

    if (threadIdx.x == 0) failed = 0;
    const double mine = block_reduce8(acc, red);
    // records: blocks [0, nb), groups [nb, nb + kEwGroups)
    unsigned long long* grec = a.ew_rec + (size_t)nb * kRecWords;
    if (b + groups < nb) {               // not the last of its group
        put_record(a.ew_rec + (size_t)b * kRecWords, mine, tag);
        return;
    }
    // group g: members g, g + groups, ..., b - groups (in that order), then this block
    // records per thread per poll: as few loads as cover the group in one
    // round (a poll's loads queue on this one CU's memory pipeline, so extra
    // slots that re-read a record cost time: 16 per thread took 0.5 us more
    // than 8 for 71 records)
    const int count = b >> lg;
    constexpr int kSlots = kForceBlock / kRecWords;      // records per load instruction
    double v;
    if (count <= 2 * kSlots)
        v = gather_records<2>(a.ew_rec, g, groups, count, tag, a.spin_limit, &failed);
    else if (count <= 4 * kSlots)
        v = gather_records<4>(a.ew_rec, g, groups, count, tag, a.spin_limit, &failed);
    else if (count <= 8 * kSlots)
        v = gather_records<8>(a.ew_rec, g, groups, count, tag, a.spin_limit, &failed);
    else
        v = gather_records<16>(a.ew_rec, g, groups, count, tag, a.spin_limit, &failed);
    const int lane = (int)threadIdx.x & (kWave - 1);
    if (lane < kRecWords && !(lane & 1)) red2[lane >> 1][threadIdx.x / kWave] = v;
    __syncthreads();
    double gsum = mine;
    if (threadIdx.x < 8) {
        double t = 0.0;
        for (int w = 0; w < kForceBlock / kWave; ++w) t += red2[threadIdx.x][w];
        gsum = t + mine;
    }
    if (b != nb - 1) {
        put_record(grec + (size_t)g * kRecWords, failed ? __builtin_nan("") : gsum, tag);
        if (threadIdx.x == 0 && failed) atomicAdd(a.ew_failed, 1u);
        return;
    }
    // final block.  One group: its sum.  Else the group sums in group order: the other groups' records
    // are gathered (groups 0..ngroups-1 except g, which is this block's own);
    // to keep the order fixed, the own group's sum is slotted in at its place.
    __shared__ double gred[kEwGroups][8];
    if (threadIdx.x < 8) gred[g][threadIdx.x] = gsum;
    if (groups > 1) {
        const int t = (int)threadIdx.x;
        const int q = t / kRecWords, word = t & (kRecWords - 1);
        const bool other = q < groups && q != g;
        unsigned long long w = 0;
        if (other) {
            for (int it = 0;; ++it) {
                w = __hip_atomic_load(grec + (size_t)q * kRecWords + word, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
                if ((unsigned)(w >> 32) == tag && a.spin_limit >= 0) break;
                if (it >= a.spin_limit) {
                    failed = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
        }
        const unsigned lo = (unsigned)__shfl_down((unsigned)(w & 0xffffffffull), 1);
        if (other && !(word & 1))
            gred[q][word >> 1] = __longlong_as_double((long long)(((w & 0xffffffffull) << 32) | lo));
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const bool bad = failed != 0;
    double val = 0.0;
    if (threadIdx.x < 8) {
        for (int q = 0; q < groups; ++q) val += gred[q][threadIdx.x];
        if (bad) val = __builtin_nan("");
        if (threadIdx.x < 2 && a.energy) a.energy[1 + threadIdx.x] = val;
        if (threadIdx.x >= 2 && a.virial) a.virial[threadIdx.x - 2] = val;
    }
    const double e_cg = __shfl_down(val, 1);
    if (threadIdx.x == 0) {
        if (bad) atomicAdd(a.ew_failed, 1u);
        if (a.energy) a.energy[0] = val + e_cg;
        __hip_atomic_store(a.epoch, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// What the half kick of atom i, component c, needs besides the pair forces.
template <typename TF>
__device__ __forceinline__ void kick_read(const MdKick& k, int i, int c, double& v, TF& f, double& m)
{
    v = k.vel[3 * i + c];
    f = ((const TF*)k.bonded)[3 * i + c];
    m = k.mass[i];
}

// The rows of a wave belong to one system (with several systems a table says
// which), so the box stays in scalar registers; a box per lane held 12 vector
// registers.  At least 6 waves per SIMD: the launches of large systems wait
// for their list entries and gathers, and 80 registers against 87 (5 waves)
// took the energy/virial launch of 256 replicas from 214.6 to 203.0 us, of the
// 98304-atom copolymer from 22.1 to 19.3, of 80000 atoms at 14 A from 62.5 to
// 58.9 (72 and 64 registers spill: no faster, and 30 to 70 % slower).  Energy and
// virial with distances per type pair read from memory need 90.
// Kick: the half kick of a dynamics step follows.  What it needs is read under
// the pair terms, in launches with energy and virial (no registers left for it)
// after them.
// Packed: rows of several systems share a wave, each lane with its row's box
// (forces-only launches of many small systems, ForceArgs::packed).
template <typename S, typename TF, bool EW, bool LDS, bool PC, int B, bool Kick, bool Packed>
__global__ __launch_bounds__(kForceBlock, B == kBatchWide ? 1 : (EW && PC && !LDS) || Packed ? 5 : 6) void k_forces(
    ForceArgs a, Cutoffs<S> cut, Cutoffs<double> cut64)
{
    const bool rb = (int)blockIdx.x >= a.blocks_a;
    const int lb = rb ? (int)blockIdx.x - a.blocks_a : (int)blockIdx.x;
    const int nb = rb ? a.blocks_b : a.blocks_a;
    // Consecutive workgroups are dealt round-robin to the 8 XCDs; give each XCD
    // a contiguous run of rows (neighbouring cells) so they share its L2.
    const int per = nb >> 3;
    const int logical = (lb & 7) * per + (lb >> 3);
    const int lg = rb ? a.log_lanes_b : a.log_lanes_a;
    const int G = 1 << lg;
    const int sub = (int)threadIdx.x & (G - 1);
    // wave of this kind, and its rows
    const int lw = __builtin_amdgcn_readfirstlane(logical * (kForceBlock / kWave) +
                                                  (int)threadIdx.x / kWave);
    int row = ((int)threadIdx.x & (kWave - 1)) >> lg, rows = kWave >> lg, sys = 0;
    const bool plain = Packed || a.nsys == 1;
    if (plain) {
        rows = min(rows, (rb ? a.n_srow : a.n_arow) - (lw << (6 - lg)));
    } else {
        int4 w = make_int4(0, 0, 0, 0);
        if (lw < a.n_waves[rb ? 1 : 0]) w = a.waves_tab[rb ? 1 : 0][lw];
        rows = w.y;
        sys = __builtin_amdgcn_readfirstlane(w.z);
        row += w.x;
    }
    const bool live = ((int)threadIdx.x & (kWave - 1)) >> lg < rows;
    if (plain) row += lw << (6 - lg);

    // the first words of the LDS tables are read before the row record, so
    // the two reads overlap (written to LDS once the record is in)
    const PairCoef<S>* coef_g = (const PairCoef<S>*)(sizeof(S) == 8 ? a.coef64 : a.coef32);
    const Cutoffs<S>* pcut_g = (const Cutoffs<S>*)(sizeof(S) == 8 ? (const void*)a.pcut64
                                                                   : (const void*)a.pcut32);
    const int np = a.ntypes * a.ntypes;
    uint32_t stg[4] = {0u, 0u, 0u, 0u};
    if constexpr (LDS) {
        if constexpr (kMixed<S, EW>) stg[1] = stage_first((const PairCoef<double>*)a.coef64, np);
        else stg[0] = stage_first(coef_g, np);
        if constexpr (PC) {
            if constexpr (!kMixed<S, EW>) stg[2] = stage_first(pcut_g, np);
            if constexpr (sizeof(S) != sizeof(double)) stg[3] = stage_first(a.pcut64, np);
        }
    }

    unsigned tag = 0;
    if constexpr (EW) {
        // tag 0 is never used: it marks a cleared record.  The epoch is an
        // ordinary load: only the previous launch wrote it (this launch writes
        // it after every block has published, i.e. after every block read
        // it), and the kernel boundary makes that write visible.  A
        // device-coherent atomic load from every wave cost 0.2 us per launch.
        tag = a.epoch[0] + 1u;
        tag += tag == 0u;
    }
    // The row's own list (the atom list for rows of ordinary atoms, the site
    // list for rows of hybrid atoms) does not depend on the row record, so its
    // first entries are loaded together with the record.  Slots past the row's
    // count read the row's padding (in bounds) and are dropped once the count
    // is known.
    const int* own_list = rb ? a.s_list + (size_t)row * a.s_cap : a.a_list + (size_t)row * a.a_cap;
    const int own_cap = rb ? a.s_cap : a.a_cap;
    uint32_t e_own[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
        const int k = sub + u * G;
        e_own[u] = (live && k < own_cap) ? (uint32_t)own_list[k] : kNoEntry;
    }
    int4 rec = make_int4(-1, 0, 0, 1);
    if (live) rec = rb ? a.s_rec[row] : a.a_rec[row];
    // FG entries: for a hybrid row they sit in the atom-list row named by the
    // record (loaded together with that row's count)
    uint32_t e_fg[B];
    int cnt_a = rec.z;
    if (rb) {
#pragma unroll
        for (int u = 0; u < B; ++u) e_fg[u] = kNoEntry;
        cnt_a = 0;
        if (live) {
            const int* fl = a.a_list + (size_t)rec.w * a.a_cap;
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int k = sub + u * G;
                if (k < a.a_cap) e_fg[u] = (uint32_t)fl[k];
            }
            cnt_a = a.a_rec[rec.w].z;
        }
    } else {
#pragma unroll
        for (int u = 0; u < B; ++u) e_fg[u] = e_own[u];
    }

    const PairCoef<S>* coef;
    const PairCoef<double>* coef64;
    const Cutoffs<S>* pcut = nullptr;
    const Cutoffs<double>* pcut64 = nullptr;
    if constexpr (LDS) {
        __shared__ CoefLds<S, EW> tab;
        __shared__ CutLds<S, EW, PC> ctab;
        if constexpr (kMixed<S, EW>)
            stage_table(tab.c64, (const PairCoef<double>*)a.coef64, np, stg[1]);
        else
            stage_table(tab.c, coef_g, np, stg[0]);
        if constexpr (PC) {
            if constexpr (!kMixed<S, EW>) stage_table(ctab.c, pcut_g, np, stg[2]);
            if constexpr (sizeof(S) != sizeof(double)) stage_table(ctab.c64, a.pcut64, np, stg[3]);
        }
        __syncthreads();
        coef = tab.c;
        if constexpr (kMixed<S, EW>) coef64 = tab.c64;
        else coef64 = (const PairCoef<double>*)tab.c;
        if constexpr (PC) {
            pcut = ctab.c;
            if constexpr (sizeof(S) != sizeof(double)) pcut64 = ctab.c64;
            else pcut64 = (const Cutoffs<double>*)ctab.c;
        }
    } else {
        coef = coef_g;
        coef64 = (const PairCoef<double>*)a.coef64;
        if constexpr (PC) {
            pcut = pcut_g;
            pcut64 = a.pcut64;
        }
    }

    TF fx = TF(0), fy = TF(0), fz = TF(0);
    // dynamics: velocity, bonded force (component sub) and mass of the row's
    // atom for the half kick, read under the pair terms
    double kv = 0.0, km = 1.0;
    TF kf = TF(0);
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const bool own = rb ? rec.x >= 0 : (rec.x >= 0 && rec.w == 0);   // hybrid atom rows belong to the site range
    if (own) {
        const int ui = rec.x, ti = rec.y & ((1 << kTypeBits) - 1);
        const int cnt_s = rb ? rec.z : 0;
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int k = sub + u * G;
            if (k >= cnt_a) e_fg[u] = kNoEntry;
            if (k >= cnt_s) e_own[u] = kNoEntry;
        }
        const double xi = a.pos[3 * ui], yi = a.pos[3 * ui + 1], zi = a.pos[3 * ui + 2];
        // the first batches of both parts: all gathers before any arithmetic
        double fxp[B], fyp[B], fzp[B], sxp[B], syp[B], szp[B];
        gather_batch<B>(a, e_fg, fxp, fyp, fzp);
        if (rb) gather_batch<B>(a, e_own, sxp, syp, szp);
        if constexpr (Kick && !EW)
            if (sub < 3) kick_read<TF>(a.kick, ui, sub, kv, kf, km);
        // the box (several systems: a read) after the gathers, so the wave does
        // not wait for it before issuing them
        const BoxV bx = Packed ? row_box(a, rec.y >> kTypeBits) : wave_box(a, sys);
        const int ro = ti * a.ntypes;
        const RowTab<S> rt{coef + ro, coef64 + ro, PC ? pcut + ro : nullptr,
                           PC ? pcut64 + ro : nullptr};
#pragma unroll
        for (int u = 0; u < B; ++u)
            entry_terms<false, S, TF, EW, PC>(bx, rt, cut, cut64, xi, yi, zi, e_fg[u], fxp[u],
                                              fyp[u], fzp[u], fx, fy, fz, acc);
        if (rb) {
#pragma unroll
            for (int u = 0; u < B; ++u)
                entry_terms<true, S, TF, EW, PC>(bx, rt, cut, cut64, xi, yi, zi, e_own[u],
                                                 sxp[u], syp[u], szp[u], fx, fy, fz, acc);
        }
        // the rest of both rows
        const int ar = rb ? rec.w : row;
        const int rest = sub + B * G;
        row_terms<false, S, TF, EW, PC, B>(a, bx, rt, cut, cut64, xi, yi, zi,
                                        a.a_list + (size_t)ar * a.a_cap, rest, cnt_a, G, fx, fy,
                                        fz, acc);
        if (rb)
            row_terms<true, S, TF, EW, PC, B>(a, bx, rt, cut, cut64, xi, yi, zi,
                                           a.s_list + (size_t)row * a.s_cap, rest, cnt_s, G, fx,
                                           fy, fz, acc);
    }
    fx = group_sum(fx, G);
    fy = group_sum(fy, G);
    fz = group_sum(fz, G);
    if constexpr (Kick) {
        // one component per lane of the row (all by the first lanes of a
        // narrower group), then the block's kinetic sum
        __shared__ double kred[kForceBlock / kWave];
        double ke = 0.0;
        if (own) {
            const double h = 0.5 * a.kick.st->dt;
            for (int c = sub; c < 3; c += G) {
                if (EW || c != sub) kick_read<TF>(a.kick, rec.x, c, kv, kf, km);
                const TF ft = (c == 0 ? fx : c == 1 ? fy : fz) + kf;
                ((TF*)a.forces)[3 * rec.x + c] = ft;
                const double v = kv + h * (a.kick.ftm2v / km) * (double)ft;
                a.kick.vel[3 * rec.x + c] = v;
                ke += km * v * v;
            }
        }
        ke = wave_sum(ke);                 // complete in lane 63
        if (((int)threadIdx.x & (kWave - 1)) == kWave - 1) kred[threadIdx.x / kWave] = ke;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < kForceBlock / kWave; ++w) t += kred[w];
            a.kick.partial[blockIdx.x] = t;
        }
    } else if (own && sub == 0) {
        TF* F = (TF*)a.forces;
        F[3 * rec.x] = fx;
        F[3 * rec.x + 1] = fy;
        F[3 * rec.x + 2] = fz;
    }
    if constexpr (EW) {
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] *= 0.5;
        if (a.nsys == 1) {
            ew_finish(a, acc, tag);
        } else {
            // several systems: a wave's rows belong to one of them, and it
            // writes their sums; a second kernel adds each system's waves
            const int lane = (int)threadIdx.x & (kWave - 1);
            const size_t wrec = (rb ? (size_t)a.blocks_a * (kForceBlock / kWave) : 0) + (size_t)lw;
            const double ws = wave_sum8(acc);
            if (lane < 8) a.wave_ew[8 * wrec + wave_sum8_lane(lane)] = ws;
        }
    }
}


// The wave tables of several systems, one thread per entry, one grid row per
// kind and lane count.
__global__ __launch_bounds__(256) void k_wave_tables(WaveTabs t)
{
    const int kind = (int)blockIdx.y / kLaneCounts, lg = (int)blockIdx.y % kLaneCounts;
    const int w = (int)(blockIdx.x * 256 + threadIdx.x);
    if (w >= t.n[kind][lg]) return;
    const int stride = t.nsys + 1;
    const int* rows = t.first + (size_t)kind * stride;
    const int* first = t.first + (size_t)(2 + kind * kLaneCounts + lg) * stride;
    // the last system whose waves start at or before w (systems without rows
    // start where the next one does)
    int lo = 0, hi = t.nsys - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= w) lo = mid;
        else hi = mid - 1;
    }
    const int row = rows[lo] + ((w - first[lo]) << (6 - lg));
    t.waves[t.at[kind][lg] + w] = make_int4(row, min(kWave >> lg, rows[lo + 1] - row), lo, 0);
}

__global__ void k_zero_outputs(double* energy, double* virial, int nsys)
{
    for (int t = threadIdx.x; t < 6 * nsys; t += blockDim.x) {
        if (energy && t < 3 * nsys) energy[t] = 0.0;
        if (virial) virial[t] = 0.0;
    }
}

// Energy and virial of every system (one block per system): the sums of the
// system's atom waves, then of its site waves, each thread in wave order, then
// a fixed-order block sum, so results are deterministic.  kSysLoads waves per
// thread per round are requested before any is added.
constexpr int kSysLoads = 4;

__global__ __launch_bounds__(256) void k_reduce_sys_ew(ForceArgs a, double* __restrict__ energy,
                                                       double* __restrict__ virial)
{
    __shared__ double red[8][4];
    const int sy = (int)blockIdx.x;
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int wa = a.sys_wave[0][sy], na = a.sys_wave[0][sy + 1] - wa;
    int ws = 0, ns = 0;
    if (a.n_srow > 0) {
        ws = a.sys_wave[1][sy];
        ns = a.sys_wave[1][sy + 1] - ws;
    }
    const size_t woff1 = (size_t)a.blocks_a * (kForceBlock / kWave) + (size_t)ws;
    const int total = na + ns;
    for (int jb = (int)threadIdx.x; jb < total; jb += 256 * kSysLoads) {
        double4 q[kSysLoads][2];
#pragma unroll
        for (int u = 0; u < kSysLoads; ++u) {
            const int j = min(jb + 256 * u, total - 1);
            const size_t wg = j < na ? (size_t)(wa + j) : woff1 + (size_t)(j - na);
            const double4* p = reinterpret_cast<const double4*>(a.wave_ew + 8 * wg);
            q[u][0] = p[0];
            q[u][1] = p[1];
        }
#pragma unroll
        for (int u = 0; u < kSysLoads; ++u) {
            if (jb + 256 * u < total) {
                v[0] += q[u][0].x; v[1] += q[u][0].y; v[2] += q[u][0].z; v[3] += q[u][0].w;
                v[4] += q[u][1].x; v[5] += q[u][1].y; v[6] += q[u][1].z; v[7] += q[u][1].w;
            }
        }
    }
    {
        const double s = wave_sum8(v);
        const int lane = (int)threadIdx.x & 63;
        if (lane < 8) red[wave_sum8_lane(lane)][threadIdx.x >> 6] = s;
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        const int k = threadIdx.x;
        const double t = red[k][0] + red[k][1] + red[k][2] + red[k][3];
        if (k < 2 && energy) energy[3 * sy + 1 + k] = t;
        if (k >= 2 && virial) virial[6 * sy + k - 2] = t;
        red[k][0] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0 && energy) energy[3 * sy] = red[0][0] + red[1][0];
}

template <typename S>
Cutoffs<S> cut_as(const double* c64)
{
    Cutoffs<S> c;
    c.rsi = (S)c64[0]; c.rso = (S)c64[1]; c.rci = (S)c64[2]; c.rco = (S)c64[3];
    c.rsi2 = (S)c64[4]; c.rso2 = (S)c64[5]; c.rci2 = (S)c64[6]; c.rco2 = (S)c64[7];
    return c;
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

hipError_t launch_bin(int n, const double* pos, TopoDev topo, GridDev* grids_dev, double4* wpos,
                      int2* key_a, int2* key_s, Status* st, bool check_moved, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    if (topo.sys)
        hipLaunchKernelGGL(k_bin<true>, dim3((n + 255) / 256), dim3(256), 0, s, n, pos, topo,
                           grids_dev, wpos, key_a, key_s, st, check_moved ? 1 : 0);
    else
        hipLaunchKernelGGL(k_bin<false>, dim3((n + 255) / 256), dim3(256), 0, s, n, pos, topo,
                           grids_dev, wpos, key_a, key_s, st, check_moved ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_moved(int n, const double* pos, TopoDev topo, const GridDev* grids_dev,
                        const double4* wpos, Status* st, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_moved, dim3((n + 255) / 256), dim3(256), 0, s, n, pos, topo, grids_dev,
                       wpos, st);
    return hipGetLastError();
}

int scan_segments(int ncell) { return (ncell + kScanSeg - 1) / kScanSeg; }

hipError_t launch_scan(GridDev* grids_dev, int ngrids, int ncell_a, int ncell_s, int* seg_tot,
                       hipStream_t s)
{
    const int nseg0 = scan_segments(ncell_a), nseg1 = ngrids > 1 ? scan_segments(ncell_s) : 0;
    if (nseg0 <= 1 && nseg1 <= 1) {
        hipLaunchKernelGGL(k_scan, dim3(ngrids), dim3(kScanThreads), 0, s, grids_dev);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_totals, dim3(nseg0 + nseg1), dim3(kScanThreads), 0, s, grids_dev,
                       nseg0, seg_tot);
    hipLaunchKernelGGL(k_scan_segments, dim3(nseg0 + nseg1), dim3(kScanThreads), 0, s, grids_dev,
                       nseg0, seg_tot);
    return hipGetLastError();
}

hipError_t launch_scatter(int n, GridDev* grids_dev, const int2* key_a, const int2* key_s,
                          hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter, dim3((n + 255) / 256), dim3(256), 0, s, n, grids_dev, key_a,
                       key_s);
    return hipGetLastError();
}

hipError_t launch_cellsort(GridDev* grids_dev, int ncell_a, int ncell_total, long long members,
                           const double4* wpos, TopoDev topo, int* user2arow, hipStream_t s)
{
    // a few members per cell (mean below 8): 4 cells per wave
    const bool small = (long long)members < 8LL * ncell_total;
    const int waves_per_block = 4;
    const int cells_per_block = waves_per_block * (small ? 4 : 1);
    int blocks = (ncell_total + cells_per_block - 1) / cells_per_block;
    if (blocks > 65535) blocks = 65535;
    if (blocks < 1) blocks = 1;
    if (small)
        hipLaunchKernelGGL(k_cellsort<16>, dim3(blocks), dim3(64 * waves_per_block), 0, s,
                           grids_dev, ncell_a, ncell_total, wpos, topo, user2arow);
    else
        hipLaunchKernelGGL(k_cellsort<64>, dim3(blocks), dim3(64 * waves_per_block), 0, s,
                           grids_dev, ncell_a, ncell_total, wpos, topo, user2arow);
    return hipGetLastError();
}

int place_segments(int ncell) { return (ncell + kPlaceSeg - 1) / kPlaceSeg; }

hipError_t launch_place(GridDev* grids_dev, int ncell_a, int ncell_s, long long members, int n,
                        const int2* key_a, const int2* key_s, const double4* wpos, TopoDev topo,
                        int* user2arow, int* seg_tot, hipStream_t s)
{
    // a few members per cell (mean below 8): 4 cells per wave, as k_cellsort
    const bool small = members < 8LL * (ncell_a + ncell_s);
    const int cells = (kPlaceThreads / kWave) * (small ? 4 : 1);
    const int blocks_a = (ncell_a + cells - 1) / cells, blocks_s = (ncell_s + cells - 1) / cells;
    if (blocks_a + blocks_s == 0) return hipSuccess;
    const int nseg_a = place_segments(ncell_a);
    if (ncell_a + ncell_s > kPlaceMaxCells) {
        hipLaunchKernelGGL(k_place_totals, dim3(nseg_a + place_segments(ncell_s)),
                           dim3(kPlaceThreads), 0, s, grids_dev, nseg_a, seg_tot);
    } else {
        seg_tot = nullptr;
    }
    if (small)
        hipLaunchKernelGGL(k_place<16>, dim3(blocks_a + blocks_s), dim3(kPlaceThreads), 0, s,
                           grids_dev, blocks_a, seg_tot, nseg_a, n, key_a, key_s, wpos, topo,
                           user2arow);
    else
        hipLaunchKernelGGL(k_place<64>, dim3(blocks_a + blocks_s), dim3(kPlaceThreads), 0, s,
                           grids_dev, blocks_a, seg_tot, nseg_a, n, key_a, key_s, wpos, topo,
                           user2arow);
    return hipGetLastError();
}

int list_candidates(int total_waves, int cand, double stencil_members)
{
    if (cand == 2 || cand == 4) return cand;
    // RELRES_LIST_CANDIDATES=2|4 overrides the automatic choice (tuning runs)
    if (const char* e = std::getenv("RELRES_LIST_CANDIDATES")) {
        if (e[0] == '2' && e[1] == 0) return 2;
        if (e[0] == '4' && e[1] == 0) return 4;
    }
    // 4 per lane needs the registers of 5 waves per SIMD, 2 those of 7 or 8:
    // worth it in a launch of at most 4 waves per SIMD (24000-atom hexane,
    // 4000 waves: build 34.4 against 38.5 us; 48000-atom hexane, 8000 waves:
    // 56.7 against 53.4 us), or where a stencil takes many rounds of 128
    // candidates (80000 atoms at 14 A, 1700 candidates: 117 against 127 us;
    // the hexane's site stencils, 750 candidates, do not).
    return total_waves <= 256 * 4 * 4 || stencil_members > kCrowdedStencil ? 4 : 2;
}

hipError_t launch_lists(GridDev* grids_dev, int ncell_a, int ncell_s, int waves_a, int waves_s,
                        TopoDev topo, const int* user2arow, int4* a_rec, int4* s_rec, Status* st,
                        bool per_wave, int cand, double stencil_members, int stencil_a,
                        int stencil_s, hipStream_t s)
{
    if (per_wave || stencil_a != 3 || stencil_s != 3) {
        const int total = waves_a + waves_s;
        if (total == 0) return hipSuccess;
        const int mx = topo.excl_off ? topo.max_excl : 0;
        const size_t dyn = sizeof(int) * 4 * kRowsPerWave * (size_t)mx;
        const bool k4 = list_candidates(total, cand, stencil_members) == 4;
        const dim3 grid((total + 3) / 4), block(256);
        const bool mol_only = topo.same_mol && !topo.excl_off;
#define RELRES_LISTS(K, SA, SS)                                                                   \
        do {                                                                                      \
            if (mol_only)                                                                         \
                hipLaunchKernelGGL((k_lists_wave<K, SA, SS, true>), grid, block, dyn, s,          \
                                   grids_dev, waves_a, total, mx, topo, user2arow, a_rec, s_rec,  \
                                   st);                                                           \
            else                                                                                  \
                hipLaunchKernelGGL((k_lists_wave<K, SA, SS, false>), grid, block, dyn, s,         \
                                   grids_dev, waves_a, total, mx, topo, user2arow, a_rec, s_rec,  \
                                   st);                                                           \
        } while (0)
        const int sel = (k4 ? 4 : 0) | (stencil_a == 5 ? 2 : 0) | (stencil_s == 5 ? 1 : 0);
        switch (sel) {
        case 0: RELRES_LISTS(2, 3, 3); break;
        case 1: RELRES_LISTS(2, 3, 5); break;
        case 2: RELRES_LISTS(2, 5, 3); break;
        case 3: RELRES_LISTS(2, 5, 5); break;
        case 4: RELRES_LISTS(4, 3, 3); break;
        case 5: RELRES_LISTS(4, 3, 5); break;
        case 6: RELRES_LISTS(4, 5, 3); break;
        default: RELRES_LISTS(4, 5, 5); break;
        }
#undef RELRES_LISTS
        return hipGetLastError();
    }
    if (ncell_a + ncell_s == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lists, dim3(ncell_a + ncell_s), dim3(kListBlock), 0, s, grids_dev,
                       ncell_a, topo, user2arow, a_rec, s_rec, st);
    return hipGetLastError();
}

// One force launch; forces-only launches of wide rows take kBatchWide entries
// per lane per batch.
template <typename S, typename TF, bool EW, bool LDS, bool PC>
void launch_force_kernel(const ForceArgs& a, const double* cut64, dim3 grid, dim3 block,
                         hipStream_t s)
{
#define RELRES_FORCES(B, KICK, PACKED)                                                           \
    hipLaunchKernelGGL((k_forces<S, TF, EW, LDS, PC, B, KICK, PACKED>), grid, block, 0, s, a,    \
                       cut_as<S>(cut64), cut_as<double>(cut64))
    if constexpr (EW) {
        if (a.kick.vel) RELRES_FORCES(kBatch, true, false);
        else RELRES_FORCES(kBatch, false, false);
    } else if (a.kick.vel) {
        if (a.wide_batch) RELRES_FORCES(kBatchWide, true, false);
        else RELRES_FORCES(kBatch, true, false);
    } else if (a.packed) {
        RELRES_FORCES(kBatch, false, true);
    } else {
        if (a.wide_batch) RELRES_FORCES(kBatchWide, false, false);
        else RELRES_FORCES(kBatch, false, false);
    }
#undef RELRES_FORCES
}

hipError_t launch_forces(const ForceArgs& a, const double* cut64, bool per_pair, int pair_math,
                         int precision, bool ew, hipStream_t s)
{
    const dim3 grid(a.blocks_a + a.blocks_b), block(kForceBlock);
    const bool lds = a.ntypes <= kLdsTypes;
#define RELRES_LAUNCH_PC(S, TF, EW, PC)                                                          \
    do {                                                                                         \
        if (lds)                                                                                 \
            launch_force_kernel<S, TF, EW, true, PC>(a, cut64, grid, block, s);                  \
        else                                                                                     \
            launch_force_kernel<S, TF, EW, false, PC>(a, cut64, grid, block, s);                 \
    } while (0)
#define RELRES_LAUNCH(S, TF, EW)                                                                 \
    do {                                                                                         \
        if (per_pair) RELRES_LAUNCH_PC(S, TF, EW, true);                                         \
        else RELRES_LAUNCH_PC(S, TF, EW, false);                                                 \
    } while (0)
    if (precision == 64) {
        if (ew) RELRES_LAUNCH(double, double, true); else RELRES_LAUNCH(double, double, false);
    } else if (pair_math == 64) {
        if (ew) RELRES_LAUNCH(double, float, true); else RELRES_LAUNCH(double, float, false);
    } else {
        if (ew) RELRES_LAUNCH(float, float, true); else RELRES_LAUNCH(float, float, false);
    }
#undef RELRES_LAUNCH
#undef RELRES_LAUNCH_PC
    return hipGetLastError();
}

hipError_t launch_list_stats(GridDev* grids_dev, int ngrids, int most_rows, Status* st, hipStream_t s)
{
    const int blocks = (most_rows + 256 * kStatRows - 1) / (256 * kStatRows);
    hipLaunchKernelGGL(k_clear_stats, dim3(1), dim3(64), 0, s, st);
    hipLaunchKernelGGL(k_list_stats, dim3(blocks > 0 ? blocks : 1, ngrids), dim3(256), 0, s, grids_dev, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// backward (adjoint) pass
// ---------------------------------------------------------------------------
// J = e_bar E + sum_i g_i . F_i.  Per ordered pair (i, j) of a list row, with
// d = x_i - x_j, fpair = -u~'(r)/r (F_i gets fpair d) and
// hc = (d fpair/dr)/r:
//   dJ/dx_i += -e_bar fpair d + fpair (g_i - g_j) + hc ((g_i - g_j) . d) d
//   dJ/dP_{t_i t_j} += e_bar u~_P / 2 + (g_i . d) fpair_P
// where u~_P, fpair_P are the pair terms evaluated with the derivative record
// of parameter P (the terms are linear in the record's coefficients).  Each
// unordered pair appears in both rows, hence the half energy weight.

// The terms are linear in eps, so the record of the eps derivative (unit eps)
// gives the pair's own terms too: fpair = eps f_eps, hc = eps h_eps.  A pair
// is evaluated with the eps and the sigma records only, which share r and its
// powers.
//
// Terms of one pair from a record: fpair, energy and h = (d fpair/dr)/r.
struct PairTerms {
    double f, e, h;
};

// LJ region: q = {c12, c6, e12, e6}
__device__ __forceinline__ PairTerms lj_terms(const double* q, double r2i, double r6i, double shift)
{
    return {r6i * (q[0] * r6i - q[1]) * r2i, r6i * (q[2] * r6i - q[3]) - shift,
            r2i * r2i * r6i * (8.0 * q[1] - 14.0 * q[0] * r6i)};
}

// A quartic zone: g = {gamma_0 .. gamma_4}, d = r - r_-
__device__ __forceinline__ PairTerms zone_terms(double g0, double g1, double g2, double g3,
                                                double g4, double d, double ir, double shift)
{
    const double dp = g1 + d * (2.0 * g2 + d * (3.0 * g3 + d * (4.0 * g4)));
    const double dpp = 2.0 * g2 + d * (6.0 * g3 + d * (12.0 * g4));
    const double f = -dp * ir;
    return {f, g0 + d * (g1 + d * (g2 + d * (g3 + d * g4))) - shift, (-dpp - f) * ir * ir};
}

// The eps and sigma terms of one pair, FG part (r2 < r_s+^2) or CG part
// (r2 < r_c+^2); T is the pair's table.
template <bool CG>
__device__ __forceinline__ void back_terms(const double* T, double r2, PairTerms& te, PairTerms& ts)
{
    using M = MathF64<2>;
    const Cutoffs<double>& cut = *reinterpret_cast<const Cutoffs<double>*>(T + kTabCut);
    const double* E = T + (CG ? kTabCgE : kTabFgE);
    const double* S = T + (CG ? kTabCgS : kTabFgS);
    // CG fields: 4 LJ, gamma_0+, gamma_3+, gamma_4+, 5 of f_c-, Gamma_c-', Gamma_c-
    if (r2 < (CG ? cut.rci2 : cut.rsi2)) {
        if (CG && r2 < cut.rso2) {
            if (r2 < cut.rsi2) {
                te = {0.0, E[4] - E[13], 0.0};
                ts = {0.0, S[4] - S[13], 0.0};
                return;
            }
            double r, ir;
            M::root(r2, r, ir);
            const double d = r - cut.rsi;
            te = zone_terms(E[4], 0.0, 0.0, E[5], E[6], d, ir, E[13]);
            ts = zone_terms(S[4], 0.0, 0.0, S[5], S[6], d, ir, S[13]);
            return;
        }
        const double r2i = M::recip(r2);
        const double r6i = r2i * r2i * r2i;
        te = lj_terms(E, r2i, r6i, CG ? E[12] : E[9]);
        ts = lj_terms(S, r2i, r6i, CG ? S[12] : S[9]);
    } else {
        double r, ir;
        M::root(r2, r, ir);
        const double d = r - (CG ? cut.rci : cut.rsi);
        constexpr int g = CG ? 7 : 4;
        te = zone_terms(E[g], E[g + 1], E[g + 2], E[g + 3], E[g + 4], d, ir, CG ? E[12] : E[9]);
        ts = zone_terms(S[g], S[g + 1], S[g + 2], S[g + 3], S[g + 4], d, ir, CG ? S[12] : S[9]);
    }
}

// Entries sub, sub + G, ... of one list row (FG part when CG is false, CG
// part when true), two per lane at a time: their list loads, then their
// position and gradient gathers, are issued together; `e` holds the first two
// (read with the row record).  TM bounds the number of types.  acc[q]: the eps
// and sigma sums of entries of type q.
template <bool CG, int TM>
__device__ __forceinline__ void back_row(const BackArgs& b, const BoxV& bx, const double* T,
                                         double xi, double yi, double zi, double gix, double giy,
                                         double giz, double ebar, const int* __restrict__ lst,
                                         int cnt, int sub, int G, uint32_t e[2], double gp[3],
                                         double acc[TM][2])
{
    const ForceArgs& a = b.f;
    for (int base = sub; base < cnt; base += 2 * G) {
        double px[2], py[2], pz[2], gx[2], gy[2], gz[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = base + u * G;
            if (base != sub) e[u] = k < cnt ? (uint32_t)lst[k] : kNoEntry;
            else if (k >= cnt) e[u] = kNoEntry;
        }
        gather_batch<2>(a, e, px, py, pz);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            gx[u] = gy[u] = gz[u] = 0.0;
            if (b.gforce) {
                const int uj = e[u] != kNoEntry ? (int)(e[u] & kIdxMask) : 0;
                gx[u] = b.gforce[3 * uj];
                gy[u] = b.gforce[3 * uj + 1];
                gz[u] = b.gforce[3 * uj + 2];
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (e[u] == kNoEntry) continue;
            const int tj = (int)(e[u] >> kIdxBits);
            double dx = xi - px[u];
            double dy = yi - py[u];
            double dz = zi - pz[u];
            dx -= bx.L[0] * rint(dx * bx.iL[0]);
            dy -= bx.L[1] * rint(dy * bx.iL[1]);
            dz -= bx.L[2] * rint(dz * bx.iL[2]);
            const double r2 = dx * dx + dy * dy + dz * dz;
            const double* Tj = T + tj * kBackTab;
            const Cutoffs<double>& cut = *reinterpret_cast<const Cutoffs<double>*>(Tj + kTabCut);
            if (!(r2 < (CG ? cut.rco2 : cut.rso2))) continue;
            PairTerms te, ts;
            back_terms<CG>(Tj, r2, te, ts);
            const double eps = Tj[kTabEps + (CG ? 1 : 0)];
            const double fp = eps * te.f, hc = eps * te.h;
            const double wx = gix - gx[u], wy = giy - gy[u], wz = giz - gz[u];
            const double hd = hc * (dx * wx + dy * wy + dz * wz) - ebar * fp;
            gp[0] += fp * wx + hd * dx;
            gp[1] += fp * wy + hd * dy;
            gp[2] += fp * wz + hd * dz;
            const double gd = gix * dx + giy * dy + giz * dz, he = 0.5 * ebar;
            const double ve = he * te.e + gd * te.f;
            const double vs = he * ts.e + gd * ts.f;
#pragma unroll
            for (int q = 0; q < TM; ++q) {
                acc[q][0] += q == tj ? ve : 0.0;
                acc[q][1] += q == tj ? vs : 0.0;
            }
        }
    }
}

// One launch over the rows of the force kernel.  What bounds it is the chain
// row record -> list entries -> gathers -> pair terms of its waves and the
// FP64 issue of the terms.  The tables are staged in LDS (read per pair from
// memory before), two entries per lane are in flight, a pair takes two record
// evaluations instead of three, and a block leaves one partial per bin, with
// the blocks of a bin side by side for k_reduce_bins (one per wave, a whole
// record apart, before).  98304-atom copolymer, four types: 35 us in the kernel
// trace, 72.7 us before.
template <int TM>
__global__ __launch_bounds__(kForceBlock, TM == 4 ? 4 : 1) void k_backward(BackArgs b)
{
    extern __shared__ __align__(16) double back_lds[];
    const ForceArgs& a = b.f;
    const bool rb = (int)blockIdx.x >= a.blocks_a;
    const int lb = rb ? (int)blockIdx.x - a.blocks_a : (int)blockIdx.x;
    const int nb = rb ? a.blocks_b : a.blocks_a;
    const int per = nb >> 3;
    const int logical = (lb & 7) * per + (lb >> 3);
    const int lg = rb ? a.log_lanes_b : a.log_lanes_a;
    const int G = 1 << lg;
    const int row = logical * (kForceBlock >> lg) + ((int)threadIdx.x >> lg);
    const int sub = (int)threadIdx.x & (G - 1);
    const int nt = a.ntypes, np = nt * nt;
    double* tab = back_lds;                              // [np][kBackTab]
    double* red = back_lds + np * kBackTab;              // [4 waves][nt][nt][4]

    // the packed tables' first words before the row record, so the two reads
    // overlap (written to LDS once the row's own reads are issued)
    typedef double double2v __attribute__((ext_vector_type(2)));
    RELRES_GLOBAL const double2v* ptab = (RELRES_GLOBAL const double2v*)b.table;
    const int words = np * kBackTab / 2;
    const double2v t_first = ptab[min((int)threadIdx.x, words - 1)];
    // the first entries of the row's own list, whatever its length (slots past
    // the end are dropped once it is known)
    const bool live = rb ? row < a.n_srow : row < a.n_arow;
    uint32_t e_own[2], e_fg[2] = {kNoEntry, kNoEntry};
    {
        const int* lst = rb ? a.s_list + (size_t)row * a.s_cap : a.a_list + (size_t)row * a.a_cap;
        const int cap = rb ? a.s_cap : a.a_cap;
#pragma unroll
        for (int u = 0; u < 2; ++u)
            e_own[u] = live && sub + u * G < cap ? (uint32_t)lst[sub + u * G] : kNoEntry;
    }
    int4 rec = make_int4(-1, 0, 0, 1);
    if (live) rec = rb ? a.s_rec[row] : a.a_rec[row];
    const bool own = rb ? rec.x >= 0 : (rec.x >= 0 && rec.w == 0);
    int cnt_a = rec.z;
    double xi = 0.0, yi = 0.0, zi = 0.0, gix = 0.0, giy = 0.0, giz = 0.0;
    if (own) {
        const int ui = rec.x;
        if (rb) {
            const int* lst = a.a_list + (size_t)rec.w * a.a_cap;
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (sub + u * G < a.a_cap) e_fg[u] = (uint32_t)lst[sub + u * G];
            cnt_a = a.a_rec[rec.w].z;
        }
        xi = a.pos[3 * ui];
        yi = a.pos[3 * ui + 1];
        zi = a.pos[3 * ui + 2];
        if (b.gforce) {
            gix = b.gforce[3 * ui];
            giy = b.gforce[3 * ui + 1];
            giz = b.gforce[3 * ui + 2];
        }
    }
    const int sy = rec.x >= 0 ? rec.y >> kTypeBits : 0;
    const double ebar = b.genergy ? b.genergy[sy] : 0.0;
    const BoxV bx = row_box(a, sy);
    {
        double2v* t2 = (double2v*)tab;
        if ((int)threadIdx.x < words) t2[threadIdx.x] = t_first;
        for (int k = (int)threadIdx.x + kForceBlock; k < words; k += kForceBlock) t2[k] = ptab[k];
    }
    for (int k = (int)threadIdx.x; k < 4 * 4 * np; k += kForceBlock) red[k] = 0.0;
    __syncthreads();
    double afg[TM][2] = {}, acg[TM][2] = {};
    double gp[3] = {0.0, 0.0, 0.0};
    const int ti = rec.y & ((1 << kTypeBits) - 1);
    if (own) {
        const int ar = rb ? rec.w : row;
        const double* T = tab + ti * nt * kBackTab;
        back_row<false, TM>(b, bx, T, xi, yi, zi, gix, giy, giz, ebar,
                            a.a_list + (size_t)ar * a.a_cap, cnt_a, sub, G, rb ? e_fg : e_own, gp,
                            afg);
        if (rb)
            back_row<true, TM>(b, bx, T, xi, yi, zi, gix, giy, giz, ebar,
                               a.s_list + (size_t)row * a.s_cap, rec.z, sub, G, e_own, gp, acg);
    }
    for (int c = 0; c < 3; ++c) gp[c] = group_sum(gp[c], G);
    if (own && sub == 0) {
        b.gpos[3 * rec.x] = gp[0];
        b.gpos[3 * rec.x + 1] = gp[1];
        b.gpos[3 * rec.x + 2] = gp[2];
    }
    // per-wave sums per (row type, entry type, parameter) of the types the
    // wave's rows have, then the block's waves in order
    const int wave = (int)(threadIdx.x >> 6);
    for (int t = 0; t < nt; ++t) {
        if (__ballot(own && ti == t) == 0ull) continue;
        double v[2 * TM];
        double* out = red + ((size_t)wave * nt + t) * 4 * nt;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            if (part == 1 && !rb) break;
#pragma unroll
            for (int q = 0; q < TM; ++q)
#pragma unroll
                for (int P = 0; P < 2; ++P)
                    v[2 * q + P] = own && ti == t ? (part ? acg[q][P] : afg[q][P]) : 0.0;
            const int lane = (int)threadIdx.x & (kWave - 1);
#pragma unroll
            for (int k = 0; k < 2 * TM; k += 8) {
                double w[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = k + j < 2 * TM ? v[k + j] : 0.0;
                const double s = wave_sum8(w);
                const int comp = k + wave_sum8_lane(lane & 7);     // 2 q + P
                if (lane < 8 && (comp >> 1) < nt) out[4 * (comp >> 1) + 2 * part + (comp & 1)] = s;
            }
        }
    }
    __syncthreads();
    for (int k = (int)threadIdx.x; k < 4 * np; k += kForceBlock)
        b.partial[(size_t)k * gridDim.x + blockIdx.x] =
            ((red[k] + red[4 * np + k]) + red[8 * np + k]) + red[12 * np + k];
}

// dJ/dP[a][b] = sum over blocks of the partial sums, in a fixed order; one
// block per bin, whose partials lie side by side.
__global__ __launch_bounds__(256) void k_reduce_bins(const double* __restrict__ partial, int blocks,
                                                     int nt, double* __restrict__ grad_pair)
{
    __shared__ double red[4];
    const int bin = (int)blockIdx.x;             // (t * nt + q) * 4 + P
    const double* p = partial + (size_t)bin * blocks;
    double s = 0.0;
    // four loads of a thread in flight (past the end, the last one again, dropped)
    for (int w = (int)threadIdx.x; w < blocks; w += 1024) {
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = p[min(w + 256 * u, blocks - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) s += w + 256 * u < blocks ? x[u] : 0.0;
    }
    const double v = wave_sum(s);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int P = bin & 3, tq = bin >> 2;
        grad_pair[(size_t)P * nt * nt + tq] = red[0] + red[1] + red[2] + red[3];
    }
}

hipError_t launch_backward(const BackArgs& b, double* grad_pair, hipStream_t s)
{
    const int nt = b.f.ntypes;
    const int blocks = b.f.blocks_a + b.f.blocks_b;
    if (blocks > 0) {
        const dim3 grid(blocks), block(kForceBlock);
        const size_t lds = sizeof(double) * (size_t)nt * nt * (kBackTab + 16);
        if (nt <= 2)
            hipLaunchKernelGGL(k_backward<2>, grid, block, lds, s, b);
        else if (nt <= 4)
            hipLaunchKernelGGL(k_backward<4>, grid, block, lds, s, b);
        else
            hipLaunchKernelGGL(k_backward<8>, grid, block, lds, s, b);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_reduce_bins, dim3(4 * nt * nt), dim3(256), 0, s, b.partial, blocks, nt,
                       grad_pair);
    return hipGetLastError();
}

// Chain rule from pair-table gradients to per-type parameters: for type t and
// family f (FG, CG), dJ/d eps_t = sum over ordered pairs (t, b) and (a, t) of
// dJ/d eps_ab times d eps_ab/d eps_t, and dJ/d sigma_t likewise through
// eps_ab and sigma_ab.  jac[(f * nt^2 + q) * 6] holds, for pair q = a*nt + b,
// the derivatives of (eps_ab, eps_ab, sigma_ab) with respect to (eps_a,
// sigma_a, sigma_a), then those with respect to type b's values.  Eight lanes
// per output (kBackwardTypes), lane b with the pairs (t, b) and (b, t), summed
// in a fixed order: one round of reads, where a thread per output waited for
// each of its 2 nt pairs (4.4 us for four types, now 3.8).
__global__ __launch_bounds__(4 * kBackwardTypes * kBackwardTypes) void k_type_grad(
    const double* __restrict__ gpair, const double* __restrict__ jac, int nt,
    double* __restrict__ gtype)
{
    const int o = (int)threadIdx.x / kBackwardTypes, b = (int)threadIdx.x % kBackwardTypes;
    const bool in = o < 4 * nt && b < nt;
    const int P = o / nt, t = o % nt;
    double s = 0.0;
    if (in) {
        const int f = P >> 1, y = P & 1;          // family, 0 = eps / 1 = sigma
        const size_t np = (size_t)nt * nt;
        const double* ge = gpair + (size_t)(2 * f) * np;       // dJ/d eps_ab of the family
        const double* gs = gpair + (size_t)(2 * f + 1) * np;   // dJ/d sigma_ab
        const double* J = jac + (size_t)f * np * 6;
        const size_t q = (size_t)t * nt + b, r = (size_t)b * nt + t;
        // type t is the first of the pair, then the second
        s = y == 0 ? ge[q] * J[6 * q] : ge[q] * J[6 * q + 1] + gs[q] * J[6 * q + 2];
        s += y == 0 ? ge[r] * J[6 * r + 3] : ge[r] * J[6 * r + 4] + gs[r] * J[6 * r + 5];
    }
    s = group_sum(s, kBackwardTypes);
    if (in && b == 0) gtype[o] = s;
}

hipError_t launch_type_grad(const double* gpair, const double* jac, int nt, double* gtype,
                            hipStream_t s)
{
    hipLaunchKernelGGL(k_type_grad, dim3(1), dim3(4 * kBackwardTypes * kBackwardTypes), 0, s, gpair,
                       jac, nt, gtype);
    return hipGetLastError();
}

// Energy/virial scratch of relres_forces_noalloc, for callers that cannot
// allocate: the launch epoch in its first 256 bytes, then the block and group
// records of the force kernel.  One copy per GPU, zero at load, shared by
// every call on that GPU (calls that overlap on one GPU race).  Host code
// reaches it only through the address scratch_address() returns.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

hipError_t scratch_address(void** out)
{
    return hipGetSymbolAddress(out, HIP_SYMBOL(scratch));
}

__global__ void k_clear_words(unsigned long long* p, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

hipError_t launch_clear_words(unsigned long long* p, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_clear_words, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_wave_tables(const WaveTabs& t, hipStream_t s)
{
    int most = 1;
    for (int kind = 0; kind < 2; ++kind)
        for (int lg = 0; lg < kLaneCounts; ++lg) most = t.n[kind][lg] > most ? t.n[kind][lg] : most;
    hipLaunchKernelGGL(k_wave_tables, dim3((most + 255) / 256, 2 * kLaneCounts), dim3(256), 0, s, t);
    return hipGetLastError();
}

hipError_t launch_zero_outputs(double* energy, double* virial, int nsys, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_outputs, dim3(1), dim3(256), 0, s, energy, virial, nsys);
    return hipGetLastError();
}

hipError_t launch_reduce_sys_ew(const ForceArgs& a, double* energy, double* virial, hipStream_t s)
{
    hipLaunchKernelGGL(k_reduce_sys_ew, dim3(a.nsys), dim3(256), 0, s, a, energy, virial);
    return hipGetLastError();
}

}  // namespace relres
