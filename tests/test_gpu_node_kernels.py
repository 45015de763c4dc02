"""Node-wise kernels of a batch (blocks of 1024 nodes over the concatenated
lattices) and the per-lattice sums over tiles, at lattice boundaries on, next
to and inside the blocks: the fields equal those of each lattice alone bit for
bit; the loss equals the sum of its terms."""
import math

import numpy as np
import pytest

import oracle
from parity_util import gpu_params, oracle_params, random_fields, random_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = {
    "one": [5],
    "block": [1024],
    "block_and_one": [1025, 3],
    "aligned": [1024, 2048, 512, 512, 1024],
    "ragged": [3, 1020, 4, 1021, 252, 253, 251, 2500, 7, 64],
    "tiny": [3 + i % 5 for i in range(700)],
    "long": [70001, 3, 505, 100000],
}


def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("which", list(LENGTHS))
def test_node_kernels_match_each_lattice_alone(which):
    from paper_1802_02369_amd import lbm
    lens = LENGTHS[which]
    rng = np.random.default_rng(len(lens) + lens[0])
    names = ("paper", "odd", "linear", "fluid")
    params = [oracle_params(names[i % 4], s_e=float(s))
              for i, s in enumerate(rng.uniform(1.1, 1.8, len(lens)))]
    offsets = np.concatenate([[0], np.cumsum(lens)])
    gps = [gpu_params(p) for p in params]
    b = lbm.Batch(offsets, gps)
    fields = [np.concatenate(x) for x in zip(*[
        random_fields(rng, L, p, amp=0.1, u=0.05, ds=0.1)
        for L, p in zip(lens, params)])]
    rho, J, zeta = [torch.from_numpy(x).to(dev()) for x in fields]
    mbar = torch.from_numpy(rng.normal(size=(6, offsets[-1]))).to(dev())
    target = torch.from_numpy(rng.uniform(0.9, 1.1, offsets[-1])).to(dev())
    f = b.equilibrium(rho, J, zeta)
    m = b.moments(f)
    aws = b.adjoint_workspace(0, 1)
    b.forward_ckpt(f, 0, 1, aws)
    fbar = b.moments_adjoint(mbar, aws)
    adj = b.equilibrium_adjoint(rho, J, zeta, fbar, aws)
    loss, lbar = b.loss(f, target, aws)
    loss0, _ = b.loss(f, None, aws)
    checked = range(len(lens)) if len(lens) < 20 else rng.integers(0, len(lens), 12)
    for i in checked:
        s = slice(int(offsets[i]), int(offsets[i + 1]))
        lat = lbm.Lattice(lens[i], gps[i])
        one = [x[s].contiguous() for x in (rho, J, zeta)]
        g = lat.equilibrium(*one)
        assert torch.equal(g, f[:, s]), i
        assert torch.equal(lat.moments(g), m[:, s]), i
        ws = lat.adjoint_workspace(0, 1)
        lat.forward_ckpt(g, 0, 1, ws)
        gbar = lat.moments_adjoint(mbar[:, s].contiguous(), ws)
        assert torch.equal(gbar, fbar[:, s]), i
        for x, y in zip(lat.equilibrium_adjoint(*one, gbar, ws), adj):
            assert torch.equal(x, y[s]), i
        # rho at the nodes as the library sums it; positive terms, summed in
        # blocks of 252 and then over blocks: well below 100 roundings each
        d = m[0, s].cpu().numpy() - target[s].cpu().numpy()
        want = math.fsum(0.5 * x * x for x in d)
        assert abs(loss[i].item() - want) <= 100 * 2.0 ** -53 * want, i
        d = m[0, s].cpu().numpy() - params[i].rho0
        want = math.fsum(0.5 * x * x for x in d)
        assert abs(loss0[i].item() - want) <= 100 * 2.0 ** -53 * want, i
        wl, gl = lat.loss(g, target[s].contiguous(), ws)
        assert wl == loss[i].item() and torch.equal(gl, lbar[:, s]), i


@pytest.mark.parametrize("n", [300, 70001])
def test_rate_gradients_over_many_tiles(n):
    """The rate partials of a lattice of few and of many reverse tiles against
    the oracle's one-step adjoint."""
    from paper_1802_02369_amd import lbm
    po = oracle_params("paper", s_e=1.4)
    rng = np.random.default_rng(n)
    f0 = random_state(rng, n, po, amp=0.1, u=0.05, ds=0.1)
    fb = rng.normal(size=(6, n))
    _, want = oracle.step_adjoint(f0, fb, po)
    lat = lbm.Lattice(n, gpu_params(po))
    ws = lat.adjoint_workspace(1, 1)
    f = torch.from_numpy(f0).to(dev())
    lat.forward_ckpt(f, 1, 1, ws)
    got = lat.adjoint(ws, 1, 1, torch.from_numpy(fb).to(dev()))
    # each partial is a sum of n terms of either sign: held against the size
    # of the terms, as in the one-step adjoint test (1e-11 of the largest)
    assert np.abs(np.array(got) - want).max() <= 1e-11 * max(np.abs(want).max(), math.sqrt(n))
