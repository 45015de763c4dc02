"""Large batches of mixed kinds of equilibria on the library's own plan, four
and eight nodes per lane: bitwise the run on a tuning of two."""
import numpy as np
import pytest
import torch

from paper_1802_02369_amd import lbm

pytestmark = pytest.mark.gpu

KINDS = [dict(), dict(eq_kind=1, u0_lin=0.15, s0_lin=0.2),
         dict(eq_kind=2, source_on=0),
         dict(eq_kind=3, source_on=0, u0_lin=0.2, alpha=-0.5)]


@pytest.mark.parametrize("lens", [
    [int(1024 * 8 ** (i / 511)) for i in range(512)],  # (4, 4, 1) tiles
    [1 << 22, (1 << 22) + 1],                          # (8, 4, 1)
])
def test_mixed_plan_matches_a_tuning(lens):
    n = sum(lens)
    g = torch.Generator().manual_seed(2)
    rho = (1 + 0.01 * torch.rand(n, generator=g, dtype=torch.float64)).cuda()
    out = []
    for tuned in (False, True):
        b = lbm.Batch(np.concatenate([[0], np.cumsum(lens)]),
                      [lbm.Params(s_e=1.3, s_psi=1.2, **KINDS[i % len(KINDS)])
                       for i in range(len(lens))])
        if tuned:
            b.set_tuning(2, 8, 1)
        f = b.equilibrium(rho, 0.1 * (rho - 1), 0.1 * (rho - 1))
        b.run(f, 41, use_graph=False)
        aws = b.adjoint_workspace(6, 3)
        b.forward_ckpt(f, 6, 3, aws)
        out.append(f)
    assert torch.isfinite(out[0]).all()
    assert torch.equal(*out)
