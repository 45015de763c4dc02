"""The diagnostics of a lattice's first call (sums combined in the workspace)
are those of the later ones (sums in pinned memory), bit for bit."""
import numpy as np
import pytest
import torch

from paper_1802_02369_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 255, 257, 65537, 262145])
def test_first_and_later_diagnostics(n):
    lat = lbm.Lattice(n)
    g = torch.Generator().manual_seed(n)
    rho = (1 + 0.1 * torch.rand(n, generator=g, dtype=torch.float64)).cuda()
    f = lat.equilibrium(rho, 0.1 * rho, 0.2 * rho)
    d = [lat.diagnostics(f) for _ in range(4)]
    assert np.isfinite(d[0]).all() and d[0][6] == 0 and d[0][7] == 0
    for x in d[1:]:
        assert np.array_equal(x, d[0])
