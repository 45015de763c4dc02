"""Diagnostics again and again, and of more lattices at once than there is
pinned memory for: the same bits every time."""
import threading

import numpy as np
import pytest
import torch

from paper_1802_02369_amd import lbm

pytestmark = pytest.mark.gpu


def _state(n):
    lat = lbm.Lattice(n)
    g = torch.Generator().manual_seed(n)
    rho = (1 + 0.1 * torch.rand(n, generator=g, dtype=torch.float64)).cuda()
    return lat, lat.equilibrium(rho, 0.1 * rho, 0.2 * rho)


@pytest.mark.parametrize("n", [3, 255, 257, 65537, 262145])
def test_repeated_diagnostics(n):
    lat, f = _state(n)
    d = [lat.diagnostics(f) for _ in range(4)]
    assert np.isfinite(d[0]).all() and d[0][6] == 0 and d[0][7] == 0
    for x in d[1:]:
        assert np.array_equal(x, d[0])


def test_diagnostics_of_many_lattices_at_once():
    """Sixteen threads, each behind the steps of its own lattice: those without
    pinned memory combine the sums on the device."""
    sizes = [70001 + 4099 * i for i in range(16)]
    states = [_state(n) for n in sizes]
    for lat, f in states:
        lat.workspace()
    want = [lat.diagnostics(f) for lat, f in states]
    got = [[] for _ in sizes]
    ready = threading.Barrier(len(sizes))

    def call(i):
        lat, f = states[i]
        for _ in range(5):
            ready.wait()
            g = f.clone()
            lat.step(g, 200)
            got[i].append(lat.diagnostics(f))

    threads = [threading.Thread(target=call, args=(i,)) for i in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for w, g in zip(want, got):
        assert len(g) == 5 and np.isfinite(w).all()
        for x in g:
            assert np.array_equal(x, w)
