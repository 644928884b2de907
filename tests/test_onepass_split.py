"""Where the one-pass expert backward runs and how it spreads its hidden tiles (csrc/onepass_split.h), compiled for the host."""
import ctypes
import functools
import os
import subprocess
import tempfile

import pytest

SRC = r"""
#include "onepass_split.h"
using namespace slicemoe;
extern "C" int waves(int ds, int He) { return onepass_waves(ds, He); }
extern "C" int passes(int ds, int He) { return onepass_passes(ds, He); }
extern "C" int pass_tiles(int ds, int He) { return onepass_pass_tiles(ds, He); }
extern "C" int chosen(int ds, int He, int E, long long units, long long cus) { return onepass_chosen(ds, He, E, units, cus); }
extern "C" int chunk(int He) { return rows_chunk(He); }
"""


@functools.lru_cache(maxsize=None)
def split():
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04286_amd", "csrc")
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "split.cpp"), os.path.join(tmp, "split.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, src, "-o", so])
        lib = ctypes.CDLL(so)
    lib.chosen.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong]
    return lib


@pytest.mark.parametrize("ds", [24, 48, 96])
def test_every_hidden_tile_is_in_one_pass(ds):
    s = split()
    for He in range(32, 8192, 32):
        n, per, w = s.passes(ds, He), s.pass_tiles(ds, He), s.waves(ds, He)
        assert per % 2 == 0 and per <= w, He
        assert (n - 1) * per < He // 16 <= n * per, He   # the last pass has tiles, and no pass follows it


@pytest.mark.parametrize("He,E,small,large", [(192, 16, None, None), (224, 16, 256, 2560), (384, 64, 256, 2560), (416, 16, 256, 3072), (576, 16, 256, 3072),
                                              (608, 16, 256, 4096), (672, 16, 192, 4096), (672, 15, 224, 4096), (768, 16, 192, 4096), (768, 32, 192, 4096), (768, 33, 256, 4096),
                                              (704, 16, 256, 4096), (800, 16, 0, 5120), (1536, 16, 0, 8192)])
def test_the_choice_at_width_96(He, E, small, large):
    """At 256 compute units: one pass up to `small` units of 32 rows and from `large` on, the two kernels between."""
    s = split()
    for units in (1, 100, 191, 192, 193, 223, 224, 225, 255, 256, 257, 1000, 2559, 2560, 3071, 3072, 4095, 4096, 5119, 5120, 8191, 8192, 100000):
        assert s.chosen(96, He, E, units, 256) == (1 if small is None or units <= small or units >= large else 0), units


def test_the_hidden_tiles_streamed_at_a_time():
    for He in range(32, 4096, 32):
        assert split().chunk(He) == max(c for c in range(1, 8) if He // 32 % c == 0), He


def test_the_choice_at_the_other_widths():
    for ds, want in ((24, 1), (48, 1), (64, 0), (128, 0), (192, 0)):
        assert all(split().chosen(ds, He, 16, units, 256) == want for He in (32, 256, 3072) for units in (1, 512, 100000))
