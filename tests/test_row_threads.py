"""How many threads copy a row of the cache (csrc/commit_device.h), compiled for the host."""
import ctypes
import subprocess

import pytest

from paper_2602_00523_amd import build

SOURCE = """
#include "commit_device.h"
extern "C" int threads_of(long pieces, int most) { return 1 << sage::closing::row_shift(pieces, most); }
"""


def test_a_row_takes_one_turn_while_there_are_threads(tmp_path):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    (tmp_path / "rows.hip").write_text(SOURCE)
    subprocess.run([hipcc, "-O2", "-std=c++20", "-fPIC", "-shared", "--cuda-host-only", "-I", build.CSRC, "-I", build.ROOT + "/include",
                    str(tmp_path / "rows.hip"), "-o", str(tmp_path / "rows.so")], check=True, capture_output=True)
    threads = ctypes.CDLL(str(tmp_path / "rows.so")).threads_of
    threads.argtypes = [ctypes.c_long, ctypes.c_int]
    for most in (128, 256, 512, 1024):
        for pieces in [1, 4, 127, 128, 129, 255, 256, 257, 512, 513, 1000, 1024, 1025, 4096, 1 << 40]:
            t = threads(pieces, most)
            assert 128 <= t <= most and t & (t - 1) == 0
            assert t >= min(pieces, most)                   # every piece has a thread
            assert t == 128 or t < 2 * pieces               # no more threads than that takes
