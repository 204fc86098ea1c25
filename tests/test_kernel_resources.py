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
