"""Inline assembly of the device code: what the compiler does not check inside such a statement."""
import os
import re
import subprocess

import pytest

from paper_2602_00523_amd import build

SOURCE = """
#include "sage_internal.h"
__global__ void unconditional(const unsigned char* const* p, unsigned char* out) {
    __shared__ unsigned char lds[1024];
    sage::lds_direct_load16(p[threadIdx.x], threadIdx.x * 16u, (__attribute__((address_space(3))) unsigned char*)lds);
    out[threadIdx.x] = lds[threadIdx.x];
}
__global__ void conditional(const unsigned char* const* p, unsigned char* out) {
    __shared__ unsigned char lds[1024];
    sage::lds_direct_load16_if(out[threadIdx.x], p[threadIdx.x], threadIdx.x * 16u, (__attribute__((address_space(3))) unsigned char*)lds);
    out[threadIdx.x] = lds[threadIdx.x];
}
"""


def test_scalar_base_of_a_load_has_its_wait_states(tmp_path):
    """Five wait states between a vector instruction that writes a scalar register and a vector-memory instruction that reads it."""
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    (tmp_path / "k.hip").write_text(SOURCE)
    cmd = [hipcc, *build.COMMON, "--cuda-device-only", "-S", str(tmp_path / "k.hip"), "-o", str(tmp_path / "k.s")]
    subprocess.run(cmd, check=True, capture_output=True)
    checked = 0
    states, writer = 100, None                               # since a vector instruction last wrote a scalar register
    for line in (tmp_path / "k.s").read_text().splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        if re.match(r"v_read(first)?lane", line):
            states, writer = 0, line
        elif line.startswith("global_load_lds"):
            assert "s[" in line and states >= 5, f"{states} wait states between {writer!r} and {line!r}"
            checked += 1
        else:
            states += 1 + (int(line.split()[1], 0) if line.startswith("s_nop") else 0)
    assert checked == 2
