"""Registers of the kernels with 1024 threads, from the compiler's own remarks (no GPU): two of their workgroups fit a compute
unit with at most 64 vector registers and 80 scalar ones (a wave with more is given 112 of a SIMD's 800)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_two_workgroups_of_1024_threads_fit_a_compute_unit():
    from paper_1712_02679_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which("hipcc")):
        pytest.skip("no hipcc")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall", "-Wextra")]
    res = subprocess.run([hipcc, *flags, "-I" + os.path.join(ROOT, "include"), "-I" + build.CSRC, "--cuda-device-only", "-c",
                          "-Rpass-analysis=kernel-resource-usage", "-o", os.devnull, os.path.join(build.CSRC, "adacomp_kernels.hip")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    seen = set()
    for name, body in re.findall(r"Function Name: (\S+)(.*?)(?=Function Name|\Z)", res.stderr, re.S):
        if not re.search(r"k_fusedILi\d+ELi16E|k_packILb\dELi\dELi16E", name):   # 16 waves
            continue
        seen.add("k_fused" if "k_fused" in name else "k_pack")
        scalar, vector = (int(re.search(r" %s: (\d+)" % what, body)[1]) for what in ("TotalSGPRs", "VGPRs"))
        assert scalar <= 80 and vector <= 64, (name, scalar, vector)
    assert seen == {"k_fused", "k_pack"}
