"""Host programs over the library's own sources (tests/host/*.cpp), built with
the host compiler."""
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

import torch

from paper_2609_33252_amd import workload as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_33252_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def available():
    return bool(shutil.which("g++")) and os.path.exists(
        os.path.join(ROCM, "include", "hip", "hip_runtime.h"))


def build(name, out, *args):
    """Compiles tests/host/<name>.cpp: the HIP headers' host half only, no device
    code and no HIP library."""
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC,
                        "-isystem", os.path.join(ROCM, "include"), *args,
                        os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


def run(name, tmp_path, *args):
    r = subprocess.run([build(name, str(tmp_path / name), *args)], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


@functools.lru_cache(maxsize=None)
def _plan_lib():
    with tempfile.TemporaryDirectory() as tmp:
        return ctypes.CDLL(build("plan", os.path.join(tmp, "plan.so"), "-shared", "-fPIC"))


# the tiles a (row alignment, second tile list) pair of batch_plan stands for
_TILES = {(256, 0): "256", (128, 0): "128", (64, 1): "128", (64, 2): "64 by rows",
          (128, 3): "64", (128, 4): "160"}


def tiles(wl, pairs):
    """Rows of the tiles that run a batch of `pairs` pairs of workload wl ("64 by
    rows": the bf16 list ordered by rows) on this device, or one of 256 compute
    units."""
    c = wl.cfg
    n_cu = 256
    if torch.cuda.is_available():
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    wk = {W.FP8: 1, W.MXFP4: 2}.get(c["w"], 0)
    a, l = ctypes.c_int(), ctypes.c_int()
    _plan_lib().plan(wk, int(pairs), c["E"], c["I"], n_cu, ctypes.byref(a), ctypes.byref(l))
    return _TILES[a.value, l.value]
