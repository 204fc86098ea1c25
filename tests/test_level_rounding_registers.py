"""The statement that rounds levels under another rounding mode (quantize_levels) is many instructions long and writes its
first results while later operands are still to be read: no result may share a register with such an operand, also
where the compiler can prove two of its inputs equal.  A kernel with equal inputs is compiled and the statement's
instructions are followed: every operand read must hold what the statement began with, or the chain's own value."""
import os
import re
import subprocess

import pytest

from paper_2107_14575_amd import build as dq_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "dq_quantize_core.h"
template <int B> __global__ void equal_inputs(const float* in, uint32_t* out, int b)
{
    float a[8], t[8];
    for (int k = 0; k < 8; ++k) a[k] = in[threadIdx.x * 8 + k];
    for (int k = 0; k < 8; ++k) t[k] = a[(k + SHIFT) & 7]; // element k's random number is another element's product
    uint32_t lv[2];
    quantize_levels<B>(a, t, b, lv);
    out[threadIdx.x * 2] = lv[0];
    out[threadIdx.x * 2 + 1] = lv[1];
}
template __global__ void equal_inputs<3>(const float*, uint32_t*, int);
template __global__ void equal_inputs<8>(const float*, uint32_t*, int);
template __global__ void equal_inputs<0>(const float*, uint32_t*, int);
"""


def _statements(asm):
    for text in re.findall(r";;#ASMSTART(.*?);;#ASMEND", asm, re.S):
        if "hwreg(HW_REG_MODE" in text and "v_fma_f32" in text:
            yield [line.split(None, 1) for line in text.strip().splitlines() if line.strip().startswith("v_")]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("shift", [0, 1, 2, 5])
def test_no_result_shares_a_register_with_a_later_operand(tmp_path, shift):
    src, out = tmp_path / "equal.hip", tmp_path / "equal.s"
    src.write_text(SOURCE.replace("SHIFT", str(shift)))
    flags = [f for f in dq_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", "-I", os.path.join(ROOT, "include"), "-I", dq_build.CSRC,
                          "-o", str(out), str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    statements = list(_statements(out.read_text()))
    assert len(statements) == 3
    for lines in statements:
        written = set()
        for op, args in lines:
            dst, *reads = [a.strip().lstrip("-") for a in args.split(",")]
            if op == "v_fma_f32" and dst not in written:  # an element's first: -(its random number) * 2^-24 + its product
                assert reads[2] == dst and len(written & set(reads)) == 0, (op, args, sorted(written))
                assert reads[0] != dst, (op, args)
            elif op == "v_fma_f32":  # value * 2^b + what keeps 1.5 * 2^23
                assert reads[0] == dst and len(written & set(reads[1:])) == 0, (op, args, sorted(written))
            else:
                assert op.startswith("v_add_f32") and dst in reads
            written.add(dst)
        assert len(written) == 8
