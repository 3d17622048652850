"""Checks of the library's host code and of its layouts on the CPU, by programs
over its own sources (tests/host/*.cpp)."""
import pytest

from . import _native

pytestmark = pytest.mark.skipif(not _native.available(),
                                reason="host compiler or HIP headers missing")


def test_row_scale_loads_stay_in_their_buffer(tmp_path):
    _native.run("row_scales", tmp_path)


def test_layer_order_and_retry(tmp_path):
    # the runtime over a model of HIP's streams: layers back to back under random
    # policies and stream counts, and launches that fail at each of their steps
    _native.run("layer_order", tmp_path, "-w", "-x", "c++")
