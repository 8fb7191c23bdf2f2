"""Waits that the hardware leaves to the code and that the compiler does not, or not always, put in, in the generated assembly."""
import os
import re
import subprocess

import pytest

from paper_2602_00523_amd import build

SOURCE = """
#include "sage_internal.h"
__global__ void load(const unsigned char* const* p, unsigned char* out) {
    __shared__ unsigned char lds[1024];
    sage::lds_direct_load16(p[threadIdx.x], threadIdx.x * 16u, (__attribute__((address_space(3))) unsigned char*)lds);
    out[threadIdx.x] = lds[threadIdx.x];
}
"""


def assembly(source, out, flags=()):
    """The lines of the assembly of a source as the library is built, without comments and directives."""
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    subprocess.run([hipcc, *build.COMMON, *flags, "--cuda-device-only", "-S", str(source), "-o", str(out)], check=True, capture_output=True)
    lines = (line.split(";")[0].strip() for line in out.read_text().splitlines())
    return [line for line in lines if line.endswith(":") or (line and not line.startswith("."))]


def operands(line):
    return line.split(None, 1)[1].split(",") if " " in line or "\t" in line else []


def wait_states(line):
    return 1 + (int(operands(line)[0], 0) if line.startswith("s_nop") else 0)


def test_scalar_base_of_a_load_has_its_wait_states(tmp_path):
    """Five wait states between a vector instruction that writes a scalar register and a vector-memory instruction that reads it."""
    (tmp_path / "k.hip").write_text(SOURCE)
    checked = 0
    states, writer = 100, None                               # since a vector instruction last wrote a scalar register
    for line in assembly(tmp_path / "k.hip", tmp_path / "k.s"):
        if line.endswith(":"):
            continue
        if re.match(r"v_read(first)?lane", line):
            states, writer = 0, line
        elif line.startswith("global_load_lds"):
            assert "s[" in line and states >= 5, f"{states} wait states between {writer!r} and {line!r}"
            checked += 1
        else:
            states += wait_states(line)
    assert checked == 1


def vector_registers(operand):
    m = re.match(r"[-|]*([va])\[(\d+):(\d+)\]", operand.strip())
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"[-|]*([va])(\d+)\b", operand.strip())
    return {(m[1], int(m[2]))} if m else set()


# wait states between an MFMA and another instruction that reads or overwrites its result: passes + 3, of more than two + 4
MFMA_WAIT_STATES = {"32x32x16": 12, "4x4x4": 5}


def early_reads(lines):
    """Pairs of an MFMA and an instruction that touches its result too early on some path, and the wait states between them."""
    labels = {line[:-1]: i for i, line in enumerate(lines) if line.endswith(":")}
    found, checked = [], 0
    for at, line in enumerate(lines):
        if not line.startswith("v_mfma"):
            continue
        need = MFMA_WAIT_STATES[re.match(r"v_mfma_f32_(\d+x\d+x\d+)", line)[1]]
        result = vector_registers(operands(line)[0])
        assert result
        checked += 1
        paths, best = [(at + 1, 0)], {}
        while paths:
            i, states = paths.pop()
            while i < len(lines) and states < need and best.get(i, need) > states:
                best[i] = states
                other = lines[i]
                i += 1
                if other.endswith(":"):
                    continue
                if other.startswith("s_endpgm"):
                    break
                if other.startswith(("s_branch", "s_cbranch")):
                    target = labels[operands(other)[0].strip()]
                    if other.startswith("s_branch"):
                        i = target
                    else:
                        paths.append((target, states + 1))
                elif other.startswith("v_mfma"):
                    d, a, b, c = (vector_registers(x) for x in operands(other))
                    if (a | b) & result:
                        found.append((line, other, states))
                    if d & result:                           # accumulates further: another result, which is looked at by itself
                        break
                elif other.startswith(("v_", "ds_", "global_", "flat_", "buffer_", "scratch_")):
                    if any(vector_registers(x) & result for x in operands(other)):
                        found.append((line, other, states))
                        break
                states += wait_states(other)
    assert checked
    return found


@pytest.mark.parametrize("name", ["tree_attention_bf16.hip", "lm_head_topk.hip", "lm_head_rows.hip"])
def test_mfma_results_have_their_wait_states(tmp_path, name):
    """The compiler counts these, but not always along the shortest of the paths that join ahead of the reader."""
    assert early_reads(assembly(os.path.join(build.CSRC, name), tmp_path / "k.s", build.EXTRA.get(name, []))) == []


def test_early_reads_are_found():
    """The check itself: a read past a branch, and one that comes late enough on the shortest path."""
    mfma = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], a[0:3], v[0:15]"
    text = [mfma, "s_cbranch_scc1 .L1", "s_nop 15", ".L1:", "s_nop 9", "v_max_f32_e32 v20, v3, v4", "s_endpgm"]
    assert [states for _, _, states in early_reads(text)] == [11]
    text[4] = "s_nop 10"
    assert early_reads(text) == []
    assert early_reads([mfma, "v_mfma_f32_32x32x16_bf16 v[32:47], v[4:7], a[0:3], 0", "s_endpgm"])


STORE_SOURCE = """
#include "sage_internal.h"
__global__ void overwritten(unsigned char* p, const unsigned* x) {
    sage::Store16 v = {x[0], x[1], x[2], x[3]};
    asm volatile("" : "+v"(v));
    sage::store_through16<0>(p + threadIdx.x * 32, v);
    v = v * 3u;
    asm volatile("" : "+v"(v));
    sage::store_through16<16>(p + threadIdx.x * 32, v);
}
"""


def early_overwrites(lines):
    """Pairs of a 16-byte store and a vector instruction that overwrites its data less than two wait states later on some path,
    and the wait states between them; the number of stores that were looked at."""
    labels = {line[:-1]: i for i, line in enumerate(lines) if line.endswith(":")}
    found, checked = [], 0
    for at, line in enumerate(lines):
        if not line.startswith("global_store_dwordx4"):
            continue
        data = vector_registers(operands(line)[1])
        assert len(data) == 4, line
        checked += 1
        paths = [(at + 1, 0)]
        while paths:
            i, states = paths.pop()
            while i < len(lines) and states < 2 and not lines[i].startswith("s_endpgm"):
                other = lines[i]
                i += 1
                if other.endswith(":"):
                    continue
                if other.startswith("s_branch"):
                    i = labels[operands(other)[0].strip()]
                elif other.startswith("s_cbranch"):
                    paths.append((labels[operands(other)[0].strip()], states + 1))
                elif other.startswith("v_") and vector_registers(operands(other)[0]) & data:
                    found.append((line, other, states))
                    break
                states += wait_states(other)
    return found, checked


def test_data_of_a_store_has_its_wait_states(tmp_path):
    """Two wait states between a store of more than 8 bytes and a vector instruction that overwrites its data: the statement's own,
    where nothing else stands between the two, and all of the attention kernels'."""
    (tmp_path / "k.hip").write_text(STORE_SOURCE)
    assert early_overwrites(assembly(tmp_path / "k.hip", tmp_path / "k.s")) == ([], 2)
    name = "tree_attention_bf16.hip"
    found, checked = early_overwrites(assembly(os.path.join(build.CSRC, name), tmp_path / "a.s", build.EXTRA[name]))
    assert found == [] and checked >= 36


def test_early_overwrites_are_found():
    store = "global_store_dwordx4 v[4:5], v[0:3], off sc1"
    assert early_overwrites([store, "s_nop 0", "v_mov_b32_e32 v3, 0", "s_endpgm"])[0][0][2] == 1
    assert early_overwrites([store, "s_cbranch_scc1 .L1", "s_nop 1", ".L1:", "v_mov_b32_e32 v0, 0", "s_endpgm"])[0][0][2] == 1
    assert early_overwrites([store, "s_nop 1", "v_mov_b32_e32 v3, 0", "s_endpgm"]) == ([], 1)
    assert early_overwrites([store, "v_mov_b32_e32 v4, 0", "s_nop 0", "v_mov_b32_e32 v2, 0", "s_endpgm"]) == ([], 1)


def test_attention_has_no_generic_stores(tmp_path):
    """A store to a generic address also counts on the LDS counter: reads of LDS between such stores wait for each of them."""
    name = "tree_attention_bf16.hip"
    text = assembly(os.path.join(build.CSRC, name), tmp_path / "k.s", build.EXTRA[name])
    assert any(line.startswith("global_store_dwordx4") for line in text)
    assert [line for line in text if line.startswith("flat_store")] == []
