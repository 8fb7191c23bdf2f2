"""The attention kernels' divisions of small numbers (div_floor, per_group in tree_attention_bf16.hip), with the arithmetic that the
device does: fp32, and a reciprocal that may be one unit in the last place off either way."""
import numpy as np
import pytest


@pytest.mark.parametrize("off", [-1, 0, 1])
def test_division_by_reciprocal(off):
    g = np.random.default_rng(7)
    y = np.concatenate([np.arange(1, 600), g.integers(1, 1 << 21, 4000)]).astype(np.int64)
    for k in (0, 1, 2, 3, 31, 32, 255, 4095):                     # just below, at and above multiples, the largest among them
        for d in (-1, 0, 1):
            q = np.minimum(k, ((1 << 21) - 2) // y)
            for x in (q * y + d, ((1 << 21) - 2) // y * y + d):
                x = np.clip(x, 0, (1 << 21) - 1)
                r = np.float32(1) / y.astype(np.float32)
                if off:
                    r = np.nextafter(r, np.float32(np.inf if off > 0 else 0), dtype=np.float32)
                got = ((x.astype(np.float32) + np.float32(0.5)) * r).astype(np.int64)
                np.testing.assert_array_equal(got, x // y)


def test_division_by_column_groups():
    x = np.arange(257)
    np.testing.assert_array_equal((x * 171) >> 9, x // 3)
