"""What the unpack kernels ask of a launch and of a compute unit, from the compiler's assembly (no GPU): bytes of arguments, and
registers where they decide how many workgroups are resident."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name with its template arguments: {directive: value}}"""
    from paper_1712_02679_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which("hipcc")):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "kernels.s")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall", "-Wextra")]
    res = subprocess.run([hipcc, *flags, "-I" + os.path.join(ROOT, "include"), "-I" + build.CSRC, "--cuda-device-only", "-S", "-o", out,
                          os.path.join(build.CSRC, "adacomp_kernels.hip")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    with open(out) as f:
        text = f.read()
    found = {}
    for symbol, body in re.findall(r"\.amdhsa_kernel (\S*k_unpack\S*)\n(.*?)\.end_amdhsa_kernel", text, re.S):
        name, args = re.search(r"\d+(k_unpack(?:8|_few)?)I(.*?)EEv", symbol).groups()
        args = tuple(int(a) for a in re.findall(r"L[ijb](\d+)E", args + "E"))
        found[(name, *args)] = {d: int(v) for d, v in re.findall(r"\.amdhsa_(\w+) (\d+)\n", body)}
    return found


# k_unpack<MODE, KIND, LG, EARLY>, k_unpack_few<MODE, KIND, MANY, NK>, k_unpack8<MODE, LG>: packets that they can have
def packets_of(kernel):
    if kernel[0] == "k_unpack_few":
        return kernel[4]
    groups = kernel[2] if kernel[0] == "k_unpack8" else kernel[3]
    return {4: 2, 8: 8, 16: 64}[groups]


def test_arguments_end_with_the_last_packet(kernels):
    assert {k[0] for k in kernels} == {"k_unpack", "k_unpack_few", "k_unpack8"}
    for kernel, d in kernels.items():
        assert d["kernarg_size"] == 128 + 8 * packets_of(kernel), kernel


def test_the_launch_of_two_packets_has_few_registers(kernels):
    assert kernels[("k_unpack8", 0, 4)]["next_free_vgpr"] <= 32


# A SIMD has 512 vector registers, given out by 8, and 800 scalar ones, given out by 16 and with 16 more to a wave than it names.
@pytest.mark.parametrize("kernel", [("k_unpack8", 1, 8), ("k_unpack8", 2, 8), ("k_unpack8", 0, 16), ("k_unpack", 1, 1, 8, 0)])
def test_seven_workgroups_of_short_bins_fit_a_compute_unit(kernels, kernel):
    d = kernels[kernel]
    scalar = d["next_free_sgpr"] + 6   # vcc, flat scratch and xnack mask
    assert d["next_free_vgpr"] <= 72 and scalar <= 96, (d["next_free_vgpr"], scalar)
