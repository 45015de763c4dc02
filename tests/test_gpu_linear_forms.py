"""Batches of the thermal scheme, alone and with section 7's equilibria: the
kernels for linear equilibria round as the one that selects them per lattice
(the same lattices beside one of another kind), bit for bit, on the library's
own plan and on tunings."""
import numpy as np
import pytest

from parity_util import gpu_params, oracle_params, random_fields

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [40, 65, 300, 1023, 5000]


@pytest.mark.parametrize("shape", [None, (1, 5, 1), (4, 5, 4), (8, 5, 2)])
@pytest.mark.parametrize("names", [("thermal",), ("thermal_odd", "linear")])
def test_linear_forms_match_mixed_kinds(names, shape):
    from paper_1802_02369_amd import lbm
    rng = np.random.default_rng(9)
    params = [oracle_params(names[i % len(names)], s_e=1.2 + 0.1 * i)
              for i in range(len(LENGTHS))]
    other = oracle_params("paper", s_e=1.4)
    fields = [random_fields(rng, L, p, amp=0.02, u=0.01, ds=0.02)
              for L, p in zip(LENGTHS + [50], params + [other])]

    def run(lens, ps):
        b = lbm.Batch(np.concatenate([[0], np.cumsum(lens)]),
                      [gpu_params(p) for p in ps])
        if shape:
            b.set_tuning(*shape)
        f = b.equilibrium(*[torch.from_numpy(np.concatenate(c)).cuda()
                            for c in zip(*fields[:len(lens)])])
        b.run(f, 23, use_graph=False)
        aws = b.adjoint_workspace(9, 4)
        b.forward_ckpt(f, 9, 4, aws)
        return f

    one = run(LENGTHS, params)
    mixed = run(LENGTHS + [50], params + [other])
    assert torch.isfinite(one).all()
    assert torch.equal(one, mixed[:, :sum(LENGTHS)])
