"""The reverse step on grids around its 16x16 tile (smaller than the tile and
its rings, whole tiles, ragged ones) against autograd of the CPU twin, and a
recorded segment over both ways of replaying it."""
import numpy as np
import pytest
import torch

import oracle
from oracle import torch_step
from paper_1907_13415_amd import inputs
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

P = (0.9, 2.72, 0.06, 0.31, 0.7, 1.3)


def _twin(f, q5, af, aq, steps):
    ft = torch.tensor(f[:, 0], requires_grad=True)
    qt = torch.tensor(q5[:, 0], requires_grad=True)
    s = [torch.tensor(P[k], dtype=torch.float64, requires_grad=True) for k in (1, 2, 3)]
    f1, q1 = ft, qt
    for _ in range(steps):
        f1, q1 = torch_step.step(f1, q1, P[0], s[0], s[1], s[2], P[4], P[5])
    ((torch.tensor(af[:, 0]) * f1).sum() + (torch.tensor(aq[:, 0]) * q1).sum()).backward()
    return ft.grad.numpy(), qt.grad.numpy(), np.array([v.grad.item() for v in s])


# one step to 1e-12 (1e-11 in the parameters) as the reverse step's other test
# holds; three chained steps to three times that
@pytest.mark.parametrize("nx,ny,steps", [(1, 1, 1), (3, 2, 1), (16, 16, 1), (17, 33, 1), (24, 24, 1), (40, 21, 3),
                                         (33, 48, 3), (700, 240, 2)])
def test_reverse_step_at_tile_edges(nx, ny, steps):
    require_gpu()
    from paper_1907_13415_amd import lc
    print("reverse step %dx%d, %d steps" % (nx, ny, steps), flush=True)
    shape = (1, ny, nx)
    rng = np.random.default_rng(nx + 1000 * ny)
    q5 = inputs.random_q5(shape, rng, amp=0.12)
    f = oracle.rest_populations(oracle.D2Q9, shape, rel=inputs.random_rel(9, shape, rng, amp=2e-3))
    af, aq = rng.normal(size=(9,) + shape), rng.normal(size=(5,) + shape)
    wf, wq, wp = _twin(f, q5, af, aq, steps)
    s = lc.Solver("D2Q9", "fp64", shape, P)
    dev = s.device
    fd, qd, afd, aqd = (torch.tensor(a, device=dev).contiguous() for a in (f, q5, af, aq))
    dp = torch.zeros(3, dtype=torch.float64, device=dev)
    if steps == 1:
        lc.lc_vjp_step(s.ctx, fd.data_ptr(), qd.data_ptr(), afd.data_ptr(), aqd.data_ptr(), dp.data_ptr())
    else:
        hist = torch.empty(lc.lc_vjp_history_bytes(s.grid, steps), dtype=torch.uint8, device=dev)
        lc.lc_vjp_segment(s.ctx, fd.data_ptr(), qd.data_ptr(), steps, hist.data_ptr(), afd.data_ptr(), aqd.data_ptr(),
                          dp.data_ptr())
    s.stream.synchronize()
    ef = np.abs(afd.cpu().numpy()[:, 0] - wf).max() / np.abs(wf).max()
    eq = np.abs(aqd.cpu().numpy()[:, 0] - wq).max() / np.abs(wq).max()
    ep = np.abs(dp.cpu().numpy() - wp) / np.maximum(np.abs(wp), 1e-12)
    print("f %.1e Q %.1e params %s" % (ef, eq, ep), flush=True)
    assert ef < 1e-12 * steps and eq < 1e-12 * steps
    if nx * ny > 1:  # a single site has no gradients: dK is a sum of zeros
        assert ep.max() < 1e-11 * steps
