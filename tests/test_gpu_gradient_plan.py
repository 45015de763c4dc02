"""The checkpointed sweep on the library's own tile shapes.

Until a tuning is set, lbm_batch_forward_ckpt chooses the shapes of the
forward, recompute and reverse launches itself.  Every node-update rounds alike
on any of them, so the final state and dL/df(0) are those of a set tuning, bit
for bit.  The rate gradients are sums over nodes and steps in another order:
at most 4e5 terms of either sign, whose orders differ by 4e5 * 1.1e-16 of the
sum of their magnitudes, some 20 times the largest rate: 1e-9 of it.
"""
import numpy as np
import pytest
import torch

from paper_1802_02369_amd import lbm

pytestmark = pytest.mark.gpu


def _sweep(lens, nsteps, ckpt, stride, eq, tuned, kernel=0):
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    b = lbm.Batch(off, [lbm.Params(s_e=1.3 + 0.01 * i, eq_kind=eq,
                                   source_on=0 if eq == 2 else 1)
                        for i in range(len(lens))])
    if tuned:
        b.set_tuning(**tuned)
    b.set_recompute_stride(stride)
    b.set_adjoint_kernel(kernel)
    g = torch.Generator().manual_seed(11)
    rho = (1 + 0.01 * torch.rand(n, generator=g, dtype=torch.float64)).cuda()
    J = (0.01 * torch.rand(n, generator=g, dtype=torch.float64)).cuda()
    zeta = torch.zeros_like(rho)
    ws = b.adjoint_workspace(nsteps, ckpt)
    f = b.equilibrium(rho, J, zeta)
    b.forward_ckpt(f, nsteps, ckpt, ws)
    _, fbar = b.loss(f, None, ws)
    rates = b.adjoint(ws, nsteps, ckpt, fbar, use_graph=False)
    return f, fbar, rates.cpu().numpy()


CASES = [
    # one lattice, one node per lane in the reverse kernel: shorter than a
    # tile, as long as its output, one node more, several tiles
    ([40], 23, 7, 1, 0), ([72], 34, 34, 1, 0), ([73], 34, 34, 1, 0),
    ([208], 41, 20, 1, 0), ([1000], 40, 13, 1, 0), ([8192], 40, 25, 1, 0),
    # eight wavefronts of one node, and two nodes per lane
    ([50021], 8, 6, 1, 0), ([150001], 2, 2, 1, 0),
    # ragged lattices, some shorter than the mirror lanes
    ([5, 16, 17, 63, 64, 65, 300, 1023, 4097], 37, 10, 1, 0),
    # every second state stored: odd and even segments, one-step segments
    ([5, 64, 379, 380, 381, 2000], 37, 9, 2, 0), ([3001], 24, 8, 2, 0),
    ([333, 77], 5, 1, 2, 0), ([333, 77], 5, 1, 1, 0),
    # linear and fluid equilibria
    ([700, 41], 20, 8, 1, 1), ([700, 41], 20, 8, 2, 2),
]


@pytest.mark.parametrize("lens, nsteps, ckpt, stride, eq", CASES)
def test_own_shapes_match_a_tuning(lens, nsteps, ckpt, stride, eq):
    tuned = dict(nodes_per_lane=2, steps_per_launch=4, waves_per_group=2)
    f0, fb0, r0 = _sweep(lens, nsteps, ckpt, stride, eq, tuned)
    f1, fb1, r1 = _sweep(lens, nsteps, ckpt, stride, eq, None)
    assert torch.isfinite(fb0).all()
    assert torch.equal(f0, f1)
    assert torch.equal(fb0, fb1)
    assert np.abs(r0 - r1).max() <= 1e-9 * np.abs(r0).max()


def test_own_shapes_with_one_step_reverse():
    tuned = dict(nodes_per_lane=2, steps_per_launch=4, waves_per_group=2)
    lens = [40, 1000, 777]
    plain = lbm.KERNEL_PLAIN
    f0, fb0, r0 = _sweep(lens, 21, 10, 1, 0, tuned, plain)
    f1, fb1, r1 = _sweep(lens, 21, 10, 1, 0, None, plain)
    assert torch.equal(f0, f1)
    assert torch.equal(fb0, fb1)
    assert np.abs(r0 - r1).max() <= 1e-9 * np.abs(r0).max()


def test_setting_the_tuning_in_force_keeps_the_workspace():
    """A workspace sized before the tuning is set explicitly to what it
    already was is large enough after it."""
    b = lbm.Batch(np.array([0, 3000, 5000]), [lbm.Params()] * 2)
    ws = b.adjoint_workspace(40, 10)
    f = b.equilibrium(*(torch.full((5000,), v, dtype=torch.float64, device="cuda")
                        for v in (1.0, 0.0, 0.0)))
    b.forward_ckpt(f, 40, 10, ws)
    t = b.get_tuning()
    b.set_tuning(t["nodes_per_lane"], t["steps_per_launch"], t["waves_per_group"])
    b.forward_ckpt(f, 40, 10, ws)
    _, fbar = b.loss(f, None, ws)
    b.adjoint(ws, 40, 10, fbar)


@pytest.mark.parametrize("lens, nsteps, ckpt", [
    # a last segment shorter and longer than a launch, of one step, one
    # segment alone; two and eight wavefronts' shapes
    ([300, 65], 31, 10), ([300, 65], 30, 10), ([300, 65], 9, 20),
    ([2000], 120, 119), ([2000], 301, 150), ([45001], 26, 25), ([45001], 60, 25),
    # two nodes per lane, joined and not
    ([100003], 5, 2), ([95001], 35, 17), ([180001], 31, 15),
])
def test_joined_launches_repeat_and_capture(lens, nsteps, ckpt):
    """Recompute and reverse in the same launches: a second sweep, a captured
    one and its replay give the bits of the first."""
    tuned = dict(nodes_per_lane=2, steps_per_launch=4, waves_per_group=2)
    f0, fb0, r0 = _sweep(lens, nsteps, ckpt, 1, 0, tuned)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    f1, fb1, r1 = _sweep(lens, nsteps, ckpt, 1, 0, None)
    assert torch.equal(f0, f1) and torch.equal(fb0, fb1)
    assert np.abs(r0 - r1).max() <= 1e-9 * np.abs(r0).max()
    b = lbm.Batch(off, [lbm.Params(s_e=1.3 + 0.01 * i) for i in range(len(lens))])
    b.set_recompute_stride(1)
    g = torch.Generator().manual_seed(11)
    n = int(off[-1])
    rho = (1 + 0.01 * torch.rand(n, generator=g, dtype=torch.float64)).cuda()
    J = (0.01 * torch.rand(n, generator=g, dtype=torch.float64)).cuda()
    ws = b.adjoint_workspace(nsteps, ckpt)
    f = b.equilibrium(rho, J, torch.zeros_like(rho))
    b.forward_ckpt(f, nsteps, ckpt, ws)
    _, seed = b.loss(f, None, ws)
    fbar = seed.clone()
    for _ in range(4):
        fbar.copy_(seed)
        rates = b.adjoint(ws, nsteps, ckpt, fbar, use_graph=True).cpu().numpy()
        assert torch.equal(fbar, fb1)
        assert np.array_equal(rates, r1)
