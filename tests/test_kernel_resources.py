"""The reduce kernels hold a lane's 32 sums and several workers' loads in registers: none of them may spill.  The
compiler's own report of every kernel's resources is read, from a compilation with the library's flags."""
import os
import re
import subprocess

import pytest

from paper_2107_14575_amd import build as dq_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_no_reduce_kernel_spills(tmp_path):
    flags = [f for f in dq_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
                          "-I", os.path.join(ROOT, "include"), "-I", dq_build.CSRC, "-o", str(tmp_path / "reduce.o"),
                          os.path.join(dq_build.CSRC, "dq_unpack_dequant_reduce.hip")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    scratch = dict(re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", res.stderr, re.S))
    assert len(scratch) >= 20, res.stderr[:2000]
    assert {k: v for k, v in scratch.items() if v != "0"} == {}


def _resources(tmp_path, source):
    flags = [f for f in dq_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
                          "-I", os.path.join(ROOT, "include"), "-I", dq_build.CSRC, "-o", str(tmp_path / "kernels.o"),
                          os.path.join(dq_build.CSRC, source)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    found = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+).*?Occupancy \[waves/SIMD\]: (\d+)", res.stderr, re.S)
    return {name: (int(scratch), int(waves)) for name, scratch, waves in found}


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source,least", [("dq_quantize_pack.hip", 30), ("dq_bracketed.hip", 40), ("dq_norm.hip", 6), ("dq_widths.hip", 5)])
def test_no_other_kernel_spills(tmp_path, source, least):
    """The kernel with a widths table that looks twice is told to leave room for seven wavefronts per SIMD (72 registers) and
    takes them all: the first spill would show here."""
    kernels = _resources(tmp_path, source)
    assert len(kernels) >= least, sorted(kernels)
    assert {k: v for k, v in kernels.items() if v[0] != 0} == {}
    told = {k: v for k, v in kernels.items() if "k_quantize_pack_bracketed_v" in k}
    assert all(v[1] >= 7 for v in told.values()), told
    assert bool(told) == (source == "dq_bracketed.hip")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_no_reduce_kernel_with_a_table_spills(tmp_path):
    kernels = _resources(tmp_path, "dq_reduce_widths.hip")
    assert len(kernels) >= 20, sorted(kernels)
    assert {k: v for k, v in kernels.items() if v[0] != 0} == {}
