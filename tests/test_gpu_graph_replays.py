"""use_graph = 1 on the same buffers again and again: the first call enqueues
directly, the second captures and launches, the later ones replay.  Every one of
them gives the bits of direct launches, with eager work and synchronisations in
between, for each kind of launch sequence: tiles, resident lattices beside tiles
(fork and join), shape groups on their streams, checks, copies back after an odd
number of launches, and the reverse sweeps with and without a second stream."""
import numpy as np
import pytest

from parity_util import gpu_params, oracle_params, random_fields

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# resident on any plan and tuning, tiles alone (too short, too long)
LENGTHS = [700, 41, 3, 15, 2000, 9000, 300, 5953, 64]


def _batch(seed, flags=0, lens=LENGTHS):
    from paper_1802_02369_amd import lbm
    rng = np.random.default_rng(seed)
    params = [oracle_params("paper", s_e=1.2 + 0.05 * i) for i in range(len(lens))]
    fields = [random_fields(rng, L, p, amp=0.02, u=0.01, ds=0.02)
              for L, p in zip(lens, params)]
    ps = [gpu_params(p) for p in params]
    for p in ps:
        p.flags = flags
    b = lbm.Batch(np.concatenate([[0], np.cumsum(lens)]), ps)
    return b, [torch.from_numpy(np.concatenate(c)).cuda() for c in zip(*fields)]


RUNS = {
    "plan": dict(),
    "tiles": dict(tuning=(2, 8, 4), resident=0),
    "resident beside tiles": dict(tuning=(2, 8, 4)),
    "resident alone": dict(lens=[700, 41, 16, 2000, 5952]),
    "one node per lane, copy back": dict(tuning=(1, 1, 1), resident=0),
    "groups": dict(groups=[(8, 40, 4), (4, 16, 4), (2, 8, 1)]),
    "checked": dict(flags=1),
}


@pytest.mark.parametrize("what", RUNS)
def test_runs_replayed(what):
    how = RUNS[what]
    b, x = _batch(3, how.get("flags", 0), how.get("lens", LENGTHS))
    if "tuning" in how:
        b.set_tuning(*how["tuning"])
    if "resident" in how:
        b.set_resident(how["resident"])
    if "groups" in how:
        b.set_groups(how["groups"], np.arange(len(LENGTHS)) % len(how["groups"]))
    f0 = b.equilibrium(*x)
    want = {}
    for steps in (33, 1, 34):
        f = f0.clone()
        b.run(f, steps, use_graph=False)
        assert torch.isfinite(f).all()
        want[steps] = f
    bufs = f0.clone(), f0.clone()
    # four calls alike, then others in between, and the first again
    for steps, k in [(33, 0)] * 4 + [(1, 0)] * 4 + [(33, 1)] * 3 + [
            (34, 1), (33, 1), (34, 1), (34, 1), (34, 1), (33, 0), (33, 0), (33, 0)]:
        f = bufs[k]
        f.copy_(f0)
        _ = (f * 2).sum().item()
        b.run(f, steps, use_graph=True)
        torch.cuda.synchronize()
        assert torch.equal(f, want[steps]), (steps, k)


SWEEPS = {
    "plan": dict(),
    "second stream": dict(tuning=(2, 4, 2)),
    "one node per lane": dict(tuning=(1, 5, 1)),
    "stride 2": dict(stride=2),
    "stride 2, tuning": dict(tuning=(2, 8, 4), stride=2),
    "one step per launch": dict(kernel=1),
}


@pytest.mark.parametrize("what", SWEEPS)
@pytest.mark.parametrize("nsteps, ckpt", [(31, 7), (12, 12)])
def test_sweeps_replayed(what, nsteps, ckpt):
    from paper_1802_02369_amd import lbm
    how = SWEEPS[what]
    b, x = _batch(4)
    if "tuning" in how:
        b.set_tuning(*how["tuning"])
    b.set_recompute_stride(how.get("stride", 1))
    b.set_adjoint_kernel(lbm.KERNEL_PLAIN if how.get("kernel") else 0)
    ws = b.adjoint_workspace(nsteps, ckpt)
    f = b.equilibrium(*x)
    b.forward_ckpt(f, nsteps, ckpt, ws)
    _, seed = b.loss(f, None, ws)
    want = seed.clone()
    rates = b.adjoint(ws, nsteps, ckpt, want, use_graph=False).clone()
    assert torch.isfinite(want).all() and torch.isfinite(rates).all()
    fbar = seed.clone()
    L = lbm.lib()
    rbar = torch.empty_like(rates)
    for _ in range(4):
        fbar.copy_(seed)
        rbar.zero_()
        _ = (fbar * 2).sum().item()
        lbm.check(L.lbm_batch_adjoint(b._h, ws.data_ptr(), ws.numel() * 8, nsteps,
                                      ckpt, fbar.data_ptr(), rbar.data_ptr(), 1))
        torch.cuda.synchronize()
        assert torch.equal(fbar, want)
        assert torch.equal(rbar, rates)
