"""What the library launches, seen through a recorded HIP runtime (no GPU)."""
import ctypes
import shutil

import numpy as np
import pytest

from launch_util import Memory, run_recorded

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def recorded(function, *args):
    run_recorded("test_launches_host", function, *args)


class Null:
    cuda_stream = 0


def make_batch(lens, kinds=(0,)):
    from paper_1802_02369_amd import lbm
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    return lbm.Batch(off, [lbm.Params(s_e=1.3, eq_kind=int(k), source_on=int(k < 2),
                                      s_psi=1.3)
                           for k in np.resize(kinds, len(lens))], stream=Null())


# ------------------------------------ a refused forward leaves the sweep --

def set_tuning(L, h, shape=None):
    """The tuning (P, K, wavefronts), or the one in force."""
    from paper_1802_02369_amd import lbm
    t = lbm.CTuning()
    assert L.lbm_batch_get_tuning(h, ctypes.byref(t)) == 0
    if shape:
        t.nodes_per_lane, t.steps_per_launch, t.waves_per_group = shape
    assert L.lbm_batch_set_tuning(h, ctypes.byref(t)) == 0


def sweep_calls(rec, tuned, between):
    """Return codes of the calls that use a checkpointed forward's tables, and
    the calls they made, pointers as buffer and offset; `between` runs after
    the forward."""
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    b = make_batch([3000, 20000, 770])
    h, n, T, C = b._h, 23770, 20, 7
    if tuned:
        set_tuning(L, h, tuned)
    ws = Memory(L.lbm_batch_adjoint_workspace_bytes(h, T, C))
    f, fbar, aux = Memory(48 * n), Memory(48 * n), Memory(48 * n)
    assert L.lbm_batch_forward_ckpt(h, f.ptr, ws.ptr, ws.nbytes, T, C) == 0
    between(L, h, f, ws, T, C)
    rec.clear()
    codes = [
        L.lbm_batch_loss(h, f.ptr, None, ws.ptr, ws.nbytes, aux.ptr, fbar.ptr),
        L.lbm_batch_moments_adjoint(h, aux.ptr, fbar.ptr, ws.ptr, ws.nbytes),
        L.lbm_batch_equilibrium_adjoint(h, aux.ptr, aux.ptr, aux.ptr, fbar.ptr,
                                        aux.ptr, aux.ptr, aux.ptr, ws.ptr,
                                        ws.nbytes),
        L.lbm_batch_adjoint(h, ws.ptr, ws.nbytes, T, C, fbar.ptr, aux.ptr, 0)]
    buffers = {"ws": ws, "f": f, "fbar": fbar, "aux": aux}

    def name(word):
        if not word.startswith("0x"):
            return word
        p = int(word, 16)
        return next((f"{k}+{p - m.ptr}" for k, m in buffers.items()
                     if m.ptr <= p < m.ptr + m.nbytes), "host")
    return codes, [" ".join(map(name, x.split())) for x in rec.log()]


def too_small(L, h, f, ws, T, C):
    set_tuning(L, h)
    assert L.lbm_batch_forward_ckpt(h, f.ptr, ws.ptr, 64, T, C) == -3


def overlapping(L, h, f, ws, T, C):
    set_tuning(L, h)
    assert L.lbm_batch_forward_ckpt(h, ws.ptr + 64, ws.ptr, ws.nbytes, T, C) == -1


def misaligned(L, h, f, ws, T, C):
    set_tuning(L, h)
    assert L.lbm_batch_forward_ckpt(h, f.ptr + 4, ws.ptr, ws.nbytes, T, C) == -1


def other_steps(L, h, f, ws, T, C):
    assert L.lbm_batch_forward_ckpt(h, f.ptr, ws.ptr, 64, 3 * T, C + 2) == -3


def other_stride(L, h, f, ws, T, C):
    assert L.lbm_batch_set_recompute_stride(h, 2) == 0
    assert L.lbm_batch_forward_ckpt(h, f.ptr, ws.ptr, 64, T, C) == -3


def other_shape(L, h, f, ws, T, C):
    set_tuning(L, h, (4, 16, 2))


def refused_forward(rec, how, tuned, sweeps):
    want, plain = sweep_calls(rec, tuned, lambda *a: None)
    assert want == [0] * 4
    got, calls = sweep_calls(rec, tuned, globals()[how])
    assert got == [0, 0, 0, 0 if sweeps else -1], got
    if not sweeps:
        plain = plain[:len(calls)]
    assert calls == plain, [x for x in zip(calls, plain) if x[0] != x[1]][:3]


@pytest.mark.parametrize("how, tuned, sweeps", [
    ("too_small", None, True), ("overlapping", None, True),
    ("misaligned", None, True), ("other_steps", None, True),
    # settings the sweep was not resolved for: the reverse sweep is refused
    # until the next forward_ckpt, the other calls take the tables there are
    ("other_stride", (2, 8, 1), False), ("other_shape", (2, 8, 1), False)])
def test_refused_forward_leaves_the_sweep(how, tuned, sweeps):
    """A forward_ckpt that is refused, also after the tuning in force was set,
    changes nothing about the sweep of the forward before it: the launches are
    the same, on the same tables of the workspace."""
    recorded("refused_forward", how, tuned, sweeps)


# --------------------------------------- arguments no forward was run with --

def adjoint_of_no_forward(rec, ckpt, after):
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    lat = lbm.Lattice(100, stream=Null())
    ws, f, fbar = Memory(1 << 20), Memory(4800), Memory(4800)
    if after:
        assert L.lbm_forward_ckpt(lat._h, f.ptr, ws.ptr, ws.nbytes, 9, 3) == 0
    rec.clear()
    rates = (ctypes.c_double * 3)()
    assert L.lbm_adjoint(lat._h, ws.ptr, ws.nbytes, 9, ckpt, fbar.ptr, rates, 0) == -1
    assert rec.log() == []


@pytest.mark.parametrize("ckpt", [0, -1, 4])
@pytest.mark.parametrize("after", [False, True])
def test_adjoint_refuses_other_checkpoints(ckpt, after):
    """lbm_adjoint with a ckpt_every that no forward was run with, 0 among
    them, is refused before it does anything."""
    recorded("adjoint_of_no_forward", ckpt, after)


# ------------------------------------------------- kernels of one kind --

def kinds_of_kernels(rec, kinds, want):
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    b = make_batch([3000, 700, 90, 41], kinds)
    h, n = b._h, 3831
    f = Memory(48 * n)
    for tuned in (None, (4, 16, 4)):
        if tuned:
            set_tuning(L, h, tuned)
        ws = Memory(L.lbm_batch_workspace_bytes(h, 0))
        assert L.lbm_batch_prepare(h, ws.ptr, ws.nbytes) == 0
        rec.clear()
        assert L.lbm_batch_run(h, f.ptr, ws.ptr, ws.nbytes, 40, 0) == 0
        aws = Memory(L.lbm_batch_adjoint_workspace_bytes(h, 10, 5))
        assert L.lbm_batch_forward_ckpt(h, f.ptr, aws.ptr, aws.nbytes, 10, 5) == 0
        # k_batch_tile<P, W, M, EQ, false>
        eq = {x.split("k_batch_tileI")[1].split("EEE")[0].split("E")[3]
              for x in rec.launches("k_batch_tile")}
        assert eq == {want}, eq


@pytest.mark.parametrize("kinds, want", [
    ((0,), "Li0"), ((1,), "Li1"), ((2,), "Li2"),
    # the thermal scheme's equilibria are linear
    ((3,), "Li1"), ((1, 3), "Li1"),
    ((0, 1), "Lin1"), ((2, 3), "Lin1")])
def test_kernels_of_one_kind_of_equilibria(kinds, want):
    """Batches whose lattices have equilibria of one form run the kernels
    compiled for it, others the one that selects them per lattice."""
    recorded("kinds_of_kernels", kinds, want)


# ------------------------------------------------------ the tuning cache --

def run_of(rec, n, batch, cache=None, tuned=None, steps=50):
    """The tile launches of `steps` steps of one lattice of n nodes (as a batch
    of one with resident lattices off, or alone) after an autotune with the
    cache, with a tuning, or with neither."""
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    if batch:
        b, pre = make_batch([n]), "lbm_batch_"
        assert L.lbm_batch_set_resident(b._h, 0) == 0
    else:
        b, pre = lbm.Lattice(n, stream=Null()), "lbm_"
    call = lambda name, *a: getattr(L, pre + name)(b._h, *a)
    f = Memory(48 * n)
    if cache:
        ws = Memory(call("workspace_bytes", lbm.WS_TUNE))
        assert call("autotune", f.ptr, ws.ptr, ws.nbytes, 32, cache.encode(),
                    None) == 0
    if tuned:
        t = lbm.CTuning(lbm.KERNEL_BLOCKED, *tuned)
        assert call("set_tuning", ctypes.byref(t)) == 0
    ws = Memory(call("workspace_bytes", lbm.WS_STEP))
    if batch:
        assert call("prepare", ws.ptr, ws.nbytes) == 0
    rec.clear()
    if batch:
        assert call("run", f.ptr, ws.ptr, ws.nbytes, steps, 0) == 0
    else:
        assert call("step", f.ptr, ws.ptr, ws.nbytes, steps) == 0
    return [tuple(x.split()[1:4]) for x in rec.log() if x.startswith("launch")]


def cached_plan(rec, tmp, batch):
    import json
    cache = tmp + "/tune.json"
    rec.prefer("ELi8ELi0E")  # eight mirror lanes: only the plan has them
    small = run_of(rec, 16000, batch, cache)
    assert small == run_of(rec, 16000, batch)
    assert len(json.load(open(cache))) == 1
    # the same class of sizes, another default tuning: the plan, not that of
    # the default of 16000 nodes
    large = run_of(rec, 17000, batch, cache)
    assert len(json.load(open(cache))) == 1
    assert large == run_of(rec, 17000, batch)
    assert large != run_of(rec, 17000, batch, tuned=(1, 13, 1))


def cached_shape(rec, tmp, batch):
    import json
    cache = tmp + "/tune.json"
    kernel = "k_batch_tile" if batch else "k_step_tile"
    run_of(rec, 1500000, batch, cache)
    (key, entry), = json.load(open(cache)).items()
    # a set shape won there; it is the default tuning of the larger size
    with open(cache, "w") as fp:
        json.dump({key: {"kernel": entry["kernel"], "P": 8, "K": 40, "W": 4,
                         **({"resident": 0} if batch else {})}}, fp)
    got = run_of(rec, 2500000, batch, cache)
    assert len(json.load(open(cache))) == 1
    assert got == run_of(rec, 2500000, batch, tuned=(8, 40, 4))
    assert got != run_of(rec, 2500000, batch)
    assert all(kernel in x[0] for x in got)


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("what", ["cached_plan", "cached_shape"])
def test_tuning_cache_across_defaults(tmp_path, what, batch):
    """An entry of the tuning cache means the same at every size of its class:
    the library's own plan, or a shape."""
    recorded(what, str(tmp_path), batch)


# ------------------------------------------------ host memory of diagnostics --

def diagnose(rec, lat, n):
    """What one call of lbm_diagnostics asks for: host memory, launches."""
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    out = (ctypes.c_double * 8)()
    f = Memory(48 * n)
    ws = Memory(L.lbm_workspace_bytes(lat._h, lbm.WS_STEP))
    rec.clear()
    assert L.lbm_diagnostics(lat._h, f.ptr, ws.ptr, ws.nbytes, out) == 0
    names = [x.split("k_diag_")[1][:5] for x in rec.launches()]
    return [x for x in rec.log() if x.startswith("host")], names


def diagnostics_memory(rec):
    from paper_1802_02369_amd import lbm
    lats = {n: lbm.Lattice(n, stream=Null()) for n in (3, 257, 100003)}
    first = True
    for _ in range(3):
        for n, lat in lats.items():
            got = diagnose(rec, lat, n)
            assert got == (["host_malloc 65536"] if first else [], ["parti"]), got
            first = False
    # handles that come and go one by one, and the last one
    rec.clear()
    for n in (3, 1000):
        lat = lbm.Lattice(n, stream=Null())
        assert diagnose(rec, lat, n) == ([], ["parti"])
    del lat
    rec.clear()
    lats.clear()
    assert rec.log() == []


def test_diagnostics_share_pinned_memory():
    """Calls one after another share one buffer of pinned memory, whatever
    their handles; making and destroying handles takes and frees none."""
    recorded("diagnostics_memory")


def diagnostics_without_pinned(rec):
    from paper_1802_02369_amd import lbm
    lat = lbm.Lattice(1000, stream=Null())
    rec.refuse_host_memory(True)
    for _ in range(20):
        assert diagnose(rec, lat, 1000) == (["host_malloc 65536"], ["parti", "final"])
    rec.refuse_host_memory(False)
    assert diagnose(rec, lat, 1000) == (["host_malloc 65536"], ["parti"])
    assert diagnose(rec, lat, 1000) == ([], ["parti"])


def test_diagnostics_go_on_without_pinned_memory():
    """Where pinned memory cannot be had, the sums are combined in the
    workspace."""
    recorded("diagnostics_without_pinned")


def diagnostics_at_once(rec):
    import threading
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    lats = [lbm.Lattice(500, stream=Null()) for _ in range(12)]
    rec.hold(True)  # every call waits until all have come
    codes = []

    def call(lat):
        out = (ctypes.c_double * 8)()
        f, ws = Memory(48 * 500), Memory(L.lbm_workspace_bytes(lat._h, lbm.WS_STEP))
        codes.append(L.lbm_diagnostics(lat._h, f.ptr, ws.ptr, ws.nbytes, out))

    rec.clear()
    threads = [threading.Thread(target=call, args=(lat,)) for lat in lats]
    for t in threads:
        t.start()
    rec.wait_for(12)
    rec.hold(False)
    for t in threads:
        t.join()
    assert codes == [0] * 12
    log = [x.split()[0] for x in rec.log()]
    assert log.count("host_malloc") == 8 and log.count("launch") == 12 + 4
    rec.clear()
    del threads
    lats.clear()
    assert rec.log() == ["host_free"] * 7


def test_diagnostics_at_once_are_bounded():
    """Twelve calls at once: eight buffers, the others do without; all but one
    go back with the last handle."""
    recorded("diagnostics_at_once")


# -------------------------------------------------- plans of mixed batches --

def mixed_plan(rec, lens, eight):
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    n = sum(lens)
    shapes = {}
    for kinds in ((0, 1), (0,), (1, 3)):
        b = make_batch(lens, kinds)
        assert L.lbm_batch_set_resident(b._h, 0) == 0
        f = Memory(48 * n)
        ws = Memory(L.lbm_batch_workspace_bytes(b._h, lbm.WS_STEP))
        assert L.lbm_batch_prepare(b._h, ws.ptr, ws.nbytes) == 0
        aws = Memory(L.lbm_batch_adjoint_workspace_bytes(b._h, 4, 4))
        rec.clear()
        assert L.lbm_batch_run(b._h, f.ptr, ws.ptr, ws.nbytes, 40, 0) == 0
        assert L.lbm_batch_forward_ckpt(b._h, f.ptr, aws.ptr, aws.nbytes, 4, 4) == 0
        names = {x.split("k_batch_tileI")[1].split("EEE")[0]
                 for x in rec.launches("k_batch_tile")}
        shapes[kinds] = {tuple(int(v[2:]) for v in x.split("E")[:3]) for x in names}
    # nodes per lane, wavefronts, mirror lanes
    wide = {(4, 4, 2), (4, 8, 2), (4, 12, 2)}
    assert not shapes[(0, 1)] & wide, shapes
    assert all((8, 4, 1) in shapes[k] for k in eight), shapes
    assert all((8, 4, 1) not in shapes[k] for k in shapes if k not in eight), shapes
    # one form of equilibria: the plan does not depend on which
    assert shapes[(0,)] == shapes[(1, 3)], shapes


@pytest.mark.parametrize("lens, eight", [
    ([700, 90, 41], []), ([2000] * 40, []), ([4096] * 400, []),
    ([int(1024 * 8 ** (i / 511)) for i in range(512)], [(0,), (1, 3)]),
    ([int(512 * 32 ** (i / 1023)) for i in range(1024)], []),
    # long lattices: eight nodes per lane by their small halo on either
    ([1 << 22] * 2, [(0, 1), (0,), (1, 3)])])
def test_plans_of_mixed_batches(lens, eight):
    """The plan of a batch whose kernels select the equilibria per lattice has
    the shapes that suit those kernels; eight: the kinds that run at eight nodes
    per lane."""
    recorded("mixed_plan", lens, eight)


# ------------------------------------------------------------------ graphs --

def captures(rec, tuned):
    """What a call does: "direct", "capture" (and launch) or "replay"."""
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    b = make_batch([3000, 700, 90, 41])
    h, n = b._h, 3831
    if tuned:
        set_tuning(L, h, tuned)
    f, g, r = Memory(48 * n), Memory(48 * n), Memory(96)
    ws = Memory(L.lbm_batch_workspace_bytes(h, lbm.WS_STEP))
    aws = Memory(L.lbm_batch_adjoint_workspace_bytes(h, 20, 7))
    assert L.lbm_batch_prepare(h, ws.ptr, ws.nbytes) == 0
    assert L.lbm_batch_forward_ckpt(h, f.ptr, aws.ptr, aws.nbytes, 20, 7) == 0

    def did(call):
        rec.clear()
        assert call() == 0
        log = [x.split()[0] for x in rec.log()]
        if "capture" in log:
            assert log[0] == "capture" and log.count("graph") == 1
            assert log[-1] == "graph" and "launch" in log
            return "capture"
        if "graph" in log:
            assert log == ["graph"]
            return "replay"
        return "direct"

    run = lambda m, k: did(lambda: L.lbm_batch_run(h, m.ptr, ws.ptr, ws.nbytes, k, 1))
    sweep = lambda m: did(lambda: L.lbm_batch_adjoint(
        h, aws.ptr, aws.nbytes, 20, 7, m.ptr, r.ptr, 1))
    assert [run(f, 20) for _ in range(4)] == ["direct", "capture", "replay", "replay"]
    assert [run(f, 21), run(f, 20), run(g, 20)] == ["direct"] * 3
    assert [run(g, 20), run(g, 20)] == ["capture", "replay"]
    assert [sweep(f) for _ in range(4)] == ["direct", "capture", "replay", "replay"]
    assert [sweep(g), sweep(f), sweep(f)] == ["direct", "direct", "capture"]


@pytest.mark.parametrize("tuned", [None, (2, 8, 2), (2, 8, 4)])
def test_second_call_alike_is_captured(tuned):
    """A run or reverse sweep whose arguments come a second time in a row is
    captured, later ones are replayed, and others enqueue directly."""
    recorded("captures", tuned)
