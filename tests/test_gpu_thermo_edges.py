"""The equation of state's logarithm and exponential where their range
reductions change: densities next to powers of two and to sqrt(1/2) 2^k (the
two ends of the logarithm's mantissa), temperatures next to half-integer powers
of two (the ends of the exponential's fraction), and non-positive densities."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_params, oracle_params

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def around(x, steps=3):
    """x and its nearest doubles on both sides."""
    out = [x]
    lo = hi = x
    for _ in range(steps):
        lo, hi = np.nextafter(lo, 0.0), np.nextafter(hi, np.inf)
        out += [lo, hi]
    return out


def equilibrium_both(rho, s, po):
    from paper_1802_02369_amd import lbm
    rho = np.array(rho)
    zeta = rho * np.array(s)
    J = 0.01 * rho
    lat = lbm.Lattice(len(rho), gpu_params(po))
    got = lat.equilibrium(*[torch.from_numpy(x).to(dev()) for x in (rho, J, zeta)])
    return got.cpu().numpy(), oracle.init(rho, J, zeta, po)


def per_node(got, want):
    scale = np.abs(want).max(axis=0)
    return (np.abs(got - want) / scale).max()


# X = ln(T/T0) carries a few ulp of ln rho and s; T and its products a few
# more, all relative to the node's largest population: 5e-14 is the bar of the
# wide-range equilibrium test, kept here.
@pytest.mark.parametrize("pname", ["paper", "odd"])
def test_log_reduction_edges(pname):
    po = oracle_params(pname)
    rho = []
    for k in range(-8, 9):
        for m in (1.0, np.sqrt(0.5),
                  np.frombuffer(np.uint64(0x3fe6a09e00000000).tobytes())[0],
                  np.frombuffer(np.uint64(0x3fe6a09effffffff).tobytes())[0],
                  np.frombuffer(np.uint64(0x3fe6a09f00000000).tobytes())[0]):
            rho += around(m * 2.0 ** k * po.rho0)
    got, want = equilibrium_both(rho, [0.1 * po.cp] * len(rho), po)
    assert per_node(got, want) < 5e-14


@pytest.mark.parametrize("pname", ["paper", "odd"])
def test_exp_reduction_edges(pname):
    po = oracle_params(pname)
    s = []
    for half in range(-16, 17):  # log2(T/T0) = half / 2 at rho = rho0
        s += around(po.s0 + half / 2 * np.log(2.0) * po.cp / po.gamma)
    got, want = equilibrium_both([po.rho0] * len(s), s, po)
    assert per_node(got, want) < 5e-14


@pytest.mark.parametrize("bad", [0.0, -0.0, -0.3, -1.0, -5e3, np.inf, np.nan])
@pytest.mark.parametrize("shape", [(1, 4, 1), (8, 4, 4), None])
def test_non_positive_density_is_nan(bad, shape):
    """One node of density `bad` makes its own f0 (which does not stream) NaN
    after a step, in the tile kernels and in the one-step kernel."""
    from paper_1802_02369_amd import lbm
    po = oracle_params("paper")
    n = 300
    f = torch.zeros((6, n), dtype=torch.float64, device=dev())
    f[:3] = 1.0 / 3.0
    f[0, 100] = bad - 2.0 / 3.0
    lat = lbm.Lattice(n, gpu_params(po))
    if shape is None:
        lat.set_tuning(kernel=lbm.KERNEL_PLAIN)
    else:
        lat.set_tuning(nodes_per_lane=shape[0], steps_per_launch=shape[1],
                       waves_per_group=shape[2])
    lat.step(f, 1)
    assert torch.isnan(f[0, 100])
    assert torch.isfinite(f[:, :97]).all() and torch.isfinite(f[:, 104:]).all()
