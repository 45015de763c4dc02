"""Kernels compiled for linear or fluid equilibria alone round as the ones that
select the equilibria per lattice, bit for bit: a batch of one kind against the
same lattices beside one of another kind, and each lattice alone, on the
library's own plan and on every tuning's tile shape."""
import numpy as np
import pytest

from parity_util import gpu_params, oracle_params, random_fields

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [64, 65, 300, 1023, 5000]
# nodes per lane, wavefronts per workgroup, steps per launch
SHAPES = [None, (1, 1, 5), (2, 1, 5), (2, 2, 5), (2, 4, 5), (2, 8, 5), (4, 1, 5),
          (4, 2, 5), (4, 4, 5), (4, 8, 5), (8, 1, 5), (8, 2, 5), (8, 4, 5), (8, 8, 5)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("name", ["linear", "fluid"])
def test_one_kind_matches_mixed_kinds(name, shape):
    from paper_1802_02369_amd import lbm
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(5)
    params = [oracle_params(name, s_e=1.2 + 0.1 * i) for i in range(len(LENGTHS))]
    fields = [random_fields(rng, L, p, amp=0.02, u=0.01, ds=0.02)
              for L, p in zip(LENGTHS, params)]
    other = oracle_params("paper", s_e=1.4)
    fields.append(random_fields(rng, 50, other, amp=0.02, u=0.01, ds=0.02))

    def run(lens, ps):
        b = lbm.Batch(np.concatenate([[0], np.cumsum(lens)]),
                      [gpu_params(p) for p in ps])
        if shape:
            b.set_tuning(nodes_per_lane=shape[0], waves_per_group=shape[1],
                         steps_per_launch=shape[2])
        else:
            b.prepare()
        x = [torch.from_numpy(np.concatenate(c)).cuda()
             for c in zip(*fields[:len(lens)])]
        f = b.equilibrium(*x)
        b.run(f, 23)
        return f

    n = sum(LENGTHS)
    one = run(LENGTHS, params)
    mixed = run(LENGTHS + [50], params + [other])
    assert torch.isfinite(one).all()
    assert torch.equal(one, mixed[:, :n])
    o = 0
    for L, p, x in zip(LENGTHS, params, fields):
        lat = lbm.Lattice(L, gpu_params(p))
        if shape:
            lat.set_tuning(nodes_per_lane=shape[0], waves_per_group=shape[1],
                           steps_per_launch=shape[2])
        f = lat.equilibrium(*[torch.from_numpy(c).cuda() for c in x])
        lat.step(f, 23)
        assert torch.equal(f, one[:, o:o + L])
        o += L
