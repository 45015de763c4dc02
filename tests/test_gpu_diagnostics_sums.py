"""Diagnostics over one block, several, a full tree of blocks and more nodes
than blocks cover at once: sums to the rounding of a tree of at most 2^-52 (n /
2^18 + 20) of the sum of magnitudes, minima and counts exactly, and the same
bits again in a second call and on a second thread's call."""
import math
import threading

import numpy as np
import pytest

from parity_util import gpu_params, oracle_params, random_fields

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [3, 255, 256, 257, 511, 65535, 65536, 65537,
                               130817, 262143, 262144, 262145, 700001])
def test_sums_minima_counts(n):
    from paper_1802_02369_amd import lbm
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = oracle_params("paper", s_e=1.4)
    lat = lbm.Lattice(n, gpu_params(p))
    rng = np.random.default_rng(n)
    x = [torch.from_numpy(a).cuda()
         for a in random_fields(rng, n, p, amp=0.1, u=0.05, ds=0.1)]
    f = lat.equilibrium(*x)
    m = lat.moments(f).cpu().numpy()
    got = lat.diagnostics(f)
    bound = 2.0 ** -52 * (n / 2 ** 18 + 20)
    for k in range(3):
        assert abs(got[k] - math.fsum(m[k])) <= bound * math.fsum(np.abs(m[k]))
    assert got[4] == m[0].min()
    assert got[6:] == [0.0, 0.0]
    others = []
    workers = [threading.Thread(target=lambda: others.append(lat.diagnostics(f)))
               for _ in range(4)]
    for w in workers:
        w.start()
    for w in workers:
        w.join()
    assert all(o == got for o in others)
    # the last node's density is not finite
    f[0, n - 1] = float("inf")
    bad = lat.diagnostics(f)
    assert bad[6] == 1.0 and bad[4] == (m[0][:-1].min() if n > 1 else math.inf)
