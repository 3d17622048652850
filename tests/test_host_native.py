"""Host-side programs over the library's own sources (tests/host/*.cpp), built
with the host compiler and run on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_33252_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def _run(tmp_path, name, *args):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("host compiler or HIP headers missing")
    exe = str(tmp_path / name)
    # the HIP headers' host half only: no device code, no HIP library
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC,
                        "-isystem", os.path.join(ROCM, "include"), *args,
                        os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_row_scale_loads_stay_in_their_buffer(tmp_path):
    _run(tmp_path, "row_scales")


def test_layer_order_and_retry(tmp_path):
    # the runtime over a model of HIP's streams: layers back to back under random
    # policies and stream counts, and launches that fail at each of their steps
    _run(tmp_path, "layer_order", "-w", "-x", "c++")
