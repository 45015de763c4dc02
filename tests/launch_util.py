"""Runs a function of a test file in a process whose HIP runtime is
hip_recorder.cpp (no GPU): the library's host side is real, its kernels are
written down instead of run."""
import atexit
import ctypes
import functools
import os
import shutil
import subprocess
import sys
import tempfile

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@functools.lru_cache(None)
def build():
    tmp = tempfile.mkdtemp()
    atexit.register(shutil.rmtree, tmp)
    so = os.path.join(tmp, "hip_recorder.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC",
                    os.path.join(HERE, "hip_recorder.cpp"), "-o", so], check=True)
    return so


def run_recorded(module, function, *args):
    """Calls module.function(recorder, *args) in the recorded process; the
    child's assertions end it with a failure."""
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {HERE!r}]\n"
            f"from launch_util import Recorder\nr = Recorder({build()!r})\n"
            f"import {module} as m\nm.{function}(r, *{args!r})\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, f"status {r.returncode}\n{r.stdout}{r.stderr}"


class Recorder:
    def __init__(self, so):
        # the library's references to HIP find these definitions first
        self._l = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self._l.rec_log.restype = ctypes.c_char_p
        self._l.rec_prefer.argtypes = [ctypes.c_char_p]

    def clear(self):
        self._l.rec_clear()

    def prefer(self, kernel: str):
        """Launches of kernels named so take a thousandth of the time."""
        self._l.rec_prefer(kernel.encode())

    def refuse_host_memory(self, on: bool):
        """hipHostMalloc fails from now on, or works again."""
        self._l.rec_refuse_host_memory(int(on))

    def hold(self, on: bool):
        """Synchronising a stream waits while on."""
        self._l.rec_hold(int(on))

    def wait_for(self, calls: int):
        """Waits until so many calls synchronise a stream."""
        assert self._l.rec_wait_for(calls) == 0

    def log(self):
        return self._l.rec_log().decode().splitlines()

    def launches(self, part=""):
        """The kernels launched whose name holds `part`."""
        return [x.split()[1] for x in self.log()
                if x.startswith("launch ") and part in x.split()[1]]


class Memory:
    """`nbytes` of device memory, 256-byte aligned."""

    def __init__(self, nbytes):
        self._a = np.zeros(nbytes + 256, dtype=np.uint8)
        self.ptr = (self._a.ctypes.data + 255) & ~255
        self.nbytes = nbytes
