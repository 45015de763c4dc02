"""A workspace sized once stays large enough when the choice of shapes moves
between the library's own plan and the tuning in force (recorded HIP runtime,
no GPU)."""
import shutil

import pytest

from launch_util import Memory, run_recorded
from test_launches_host import make_batch, set_tuning

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

LENGTHS = [[8000], [16384], [3, 16, 17, 5000], [100003], [600] * 40]


def plan_and_tuning(rec, lens):
    from paper_1802_02369_amd import lbm
    L = lbm.lib()
    n = sum(lens)
    f = Memory(48 * n)

    def calls(h, ws, aws):
        assert L.lbm_batch_prepare(h, ws.ptr, ws.nbytes) == 0
        assert L.lbm_batch_run(h, f.ptr, ws.ptr, ws.nbytes, 20, 0) == 0
        assert L.lbm_batch_forward_ckpt(h, f.ptr, aws.ptr, aws.nbytes, 20, 7) == 0

    def sizes(h):
        return (Memory(L.lbm_batch_workspace_bytes(h, lbm.WS_STEP)),
                Memory(L.lbm_batch_adjoint_workspace_bytes(h, 20, 7)))

    # sized on the plan, then the tuning in force is set
    b = make_batch(lens)
    mem = sizes(b._h)
    calls(b._h, *mem)
    set_tuning(L, b._h)
    calls(b._h, *mem)
    # sized on that tuning, then the autotuner goes back to the plan
    b = make_batch(lens)
    set_tuning(L, b._h)
    mem = sizes(b._h)
    tune = Memory(L.lbm_batch_workspace_bytes(b._h, lbm.WS_TUNE))
    rec.prefer("k_batch_resident" if lens[0] == 600 else
               "ELi8ELi0E" if n < 50000 else "Li1ELi12ELi8E")
    assert L.lbm_batch_autotune(b._h, f.ptr, tune.ptr, tune.nbytes, 32, None,
                                None) == 0
    rec.clear()
    calls(b._h, *mem)


@pytest.mark.parametrize("lens", LENGTHS)
def test_workspace_holds_for_plan_and_tuning(lens):
    run_recorded("test_workspace_host", "plan_and_tuning", lens)
