"""Which stream a call uses, and where the parameter gradients arrive."""
import numpy as np
import pytest

import workloads as w
from _util import make_relres

pytestmark = pytest.mark.gpu


def test_calls_follow_the_current_stream():
    import torch
    from paper_2104_10231_amd.relres import _stream
    side = torch.cuda.Stream()
    assert _stream(None) == torch.cuda.current_stream().cuda_stream
    assert _stream(side) == side.cuda_stream
    with torch.cuda.stream(side):
        assert _stream(None) == side.cuda_stream
    s = w.propane_liquid(2, n_mol=200)
    rr = make_relres(s, 64)
    pos = torch.from_numpy(s.pos).cuda()
    rr.build_lists(pos, s.box)
    want = rr.forces(pos)[0].cpu()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        moved = pos.clone() + 5.0                 # on the side stream, like the call behind it
        got = rr.forces(moved - 5.0)[0]
    side.synchronize()
    assert torch.allclose(got.cpu(), want, rtol=1e-9, atol=1e-9)
    rr.close()


@pytest.mark.parametrize("devices", ["cpu", "cuda", "mixed"])
def test_parameter_gradients_arrive_on_their_devices(devices):
    import torch
    from paper_2104_10231_amd.autograd import energy_forces
    s = w.propane_liquid(3, n_mol=200)
    rr = make_relres(s, 64)
    pos = torch.from_numpy(s.pos).cuda()
    rr.build_lists(pos, s.box)
    where = {"cpu": ["cpu"] * 4, "cuda": ["cuda"] * 4, "mixed": ["cpu", "cuda", "cuda", "cpu"]}[devices]
    theta = [torch.tensor(np.asarray(getattr(s, k), np.float64), device=d, requires_grad=True)
             for k, d in zip(("eps_fg", "sig_fg", "eps_cg", "sig_cg"), where)]
    F, E = energy_forces(rr, pos.requires_grad_(True), *theta)
    grads = torch.autograd.grad((F * F).sum() + E, theta)
    up = (2.0 * F).detach()
    ref = rr.backward_types(pos.detach(), up, torch.ones(1, dtype=torch.float64, device="cuda"))[1].cpu()
    for k, g in enumerate(grads):
        assert g.device.type == where[k] and torch.equal(g.cpu(), ref[k])
    grads[0].add_(1.0)                            # the gradients do not share memory
    assert torch.equal(grads[3].cpu(), ref[3])
    rr.close()
