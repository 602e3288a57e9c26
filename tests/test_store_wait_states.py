"""Stores of 16 bytes whose offset stands in a scalar register, in the assembly of the library's kernels (no GPU): two wait
states, by an s_nop, before anything overwrites the registers that they store.  The compiler leaves none there, and the GPU then
stores the new value now and then."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WITHIN = 8   # instructions behind a store among which its s_nop stands


def vector_registers(operand):
    span = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if span:
        return set(range(int(span[1]), int(span[2]) + 1))
    one = re.fullmatch(r"v(\d+)", operand)
    return {int(one[1])} if one else set()


def unprotected(instructions):
    """Numbers of all such stores, and those of them that can be overtaken."""
    stores, bad = 0, []
    for i, text in enumerate(instructions):
        m = re.match(r"buffer_store_dwordx[34] (\S+), \S+, \S+, s\d+ ", text)
        if not m:
            continue
        stores += 1
        data = vector_registers(m[1])
        for after in instructions[i + 1:i + 1 + WITHIN]:
            name, _, operands = after.partition(" ")
            if name == "s_nop":
                if int(operands) < 1:
                    bad.append((text, after))
                break
            if name.startswith("v_") and vector_registers(operands.split(",")[0].strip()) & data:
                bad.append((text, after))
                break
        else:
            bad.append((text, "no s_nop"))
    return stores, bad


def test_what_counts_as_unprotected():
    store = "buffer_store_dwordx4 v[4:7], v1, s[4:7], s9 offen nt"
    assert unprotected([store, "s_nop 1", "v_mov_b32_e32 v4, 0"]) == (1, [])
    assert unprotected([store, "v_mov_b32_e32 v8, 0", "s_nop 1"]) == (1, [])
    assert unprotected(["buffer_store_dwordx4 v[4:7], v1, s[4:7], 0 offen nt", "v_mov_b32_e32 v4, 0"]) == (0, [])
    for behind in (["v_cndmask_b32_e64 v4, 0, 1, s[30:31]", "s_nop 1"], ["s_nop 0"], ["v_add_f32_e32 v[6:7], v0, v1"], ["s_endpgm"]):
        assert len(unprotected([store, *behind])[1]) == 1, behind


def test_wide_stores_have_their_wait_states(tmp_path):
    from paper_1712_02679_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which("hipcc")):
        pytest.skip("no hipcc")
    out = str(tmp_path / "kernels.s")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall", "-Wextra")]
    res = subprocess.run([hipcc, *flags, "-I" + os.path.join(ROOT, "include"), "-I" + build.CSRC, "--cuda-device-only", "-S", "-o", out,
                          os.path.join(build.CSRC, "adacomp_kernels.hip")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    with open(out) as f:
        lines = [line.split(";")[0].strip() for line in f if line.startswith("\t")]
    stores, bad = unprotected([line for line in lines if line and not line.startswith(".")])
    assert stores > 100   # k_pack and the unpack kernels with the optimizer's step
    assert not bad, (len(bad), stores, bad[:5])
