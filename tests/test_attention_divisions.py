"""The divisions with which the attention kernels cut a call (csrc/split_divisions.h), compiled for the host: the code itself, with a
reciprocal that may be one unit in the last place off either way."""
import ctypes
import subprocess

import numpy as np
import pytest

from paper_2602_00523_amd import build

SOURCE = """
#include "split_divisions.h"
extern "C" void quotients(const int* x, const int* y, const float* reciprocal, int n, int* out) {
    for (int i = 0; i < n; ++i)
        out[i] = sage::div_floor(x[i], y[i], [&](int a, int) { return sage::by_reciprocal(a, reciprocal[i]); });
}
extern "C" int group_share(int x, int groups) { return sage::per_group(x, groups); }
extern "C" void products(const int* x, int n, int y, int* out) {
    for (int i = 0; i < n; ++i) out[i] = sage::by_product(x[i], sage::inverse(y));
}
extern "C" void up_by_cost(const int* x, int n, int cost, int* out) {
    for (int i = 0; i < n; ++i) out[i] = sage::div_up_by_cost(x[i], cost);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("divisions")
    (d / "divisions.hip").write_text(SOURCE)
    subprocess.run([hipcc, "-O2", "-std=c++20", "-fPIC", "-shared", "--cuda-host-only", "-I", build.CSRC, str(d / "divisions.hip"), "-o",
                    str(d / "divisions.so")], check=True, capture_output=True)
    return ctypes.CDLL(str(d / "divisions.so"))


@pytest.mark.parametrize("off", [-1, 0, 1])
@pytest.mark.parametrize("most", [(1 << 21) - 1, (1 << 31) - 1])
def test_division_by_reciprocal(lib, most, off):
    g = np.random.default_rng(7)
    y = np.concatenate([np.arange(1, 600), g.integers(1, 1 << 21, 4000)]).astype(np.int64)
    r = np.float32(1) / y.astype(np.float32)
    if off:
        r = np.nextafter(r, np.float32(np.inf if off > 0 else 0), dtype=np.float32)
    for k in (0, 1, 2, 3, 31, 32, 255, 4095, 1 << 20):            # just below, at and above multiples, the largest among them
        for d in (-1, 0, 1):
            q = np.minimum(k, most // y)
            for x in (q * y + d, most // y * y + d, most + 0 * y, np.clip(q * y + d, 1 << 21, None)):
                x = np.ascontiguousarray(np.clip(x, 0, most), np.int32)
                yi, got = y.astype(np.int32), np.empty_like(x)
                lib.quotients(*(a.ctypes.data_as(ctypes.c_void_p) for a in (x, yi, r)), len(x), got.ctypes.data_as(ctypes.c_void_p))
                np.testing.assert_array_equal(got, x // y)


def test_division_by_column_groups(lib):
    for groups in (1, 2, 3, 4):
        assert [lib.group_share(x, groups) for x in range(257)] == [x // groups for x in range(257)]


def test_division_by_product(lib):
    k = np.random.default_rng(8).integers(0, 1 << 24, 20000)
    for y in range(2, 257):
        x = np.concatenate([np.arange(1025), (k // y)[:, None].repeat(3, 1).ravel() * y + np.tile([-1, 0, 1], len(k)), (1 << 24) - 1 - np.arange(300)])
        x = np.ascontiguousarray(np.clip(x, 0, (1 << 24) - 1), np.int32)
        got = np.empty_like(x)
        lib.products(*(a.ctypes.data_as(ctypes.c_void_p) if isinstance(a, np.ndarray) else a for a in (x, len(x), y, got)))
        np.testing.assert_array_equal(got, x // y)


def test_division_by_cost(lib):
    top = (1 << 31) - 8
    x = np.concatenate([np.arange(5000), top - np.arange(5000), np.random.default_rng(9).integers(0, top, 200000)]).astype(np.int32)
    for cost in (1, 3, 4):
        got = np.empty_like(x)
        lib.up_by_cost(*(a.ctypes.data_as(ctypes.c_void_p) if isinstance(a, np.ndarray) else a for a in (x, len(x), cost, got)))
        np.testing.assert_array_equal(got, -(-x.astype(np.int64) // cost))
