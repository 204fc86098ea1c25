"""The chunk code of the quantize kernels takes one entry of the plan's chunk table for the whole chunk of a
workgroup, so that chunk has to be the table's 4096 elements: any other size is refused by the compiler, with
norms given (NORM = 0) as well as computed, and no macro changes the size the library launches."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_14575_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

INSTANTIATE = """
#include "dq_quantize_core.h"
namespace {
__global__ void k(const float* g, const float* n, const dq_chunk_tensor* t, const int32_t* i, const int64_t* e,
                  const dq_cseg_width* wt, uint8_t* p, float* out)
{
#if TRY_PER_TENSOR
    quantize_pack_chunk_v<TRY_TILES, TRY_NORM>(g, 0, n, 1, t, i, i, e, wt, 0, 128, 0u, 0u, 0u, 0u, p, 0, out, blockIdx.x);
#else
    quantize_pack_chunk<4, TRY_TILES, TRY_NORM>(g, 0, n, 1, t, i, i, e, 128, 0u, 0u, 0u, 0u, p, 0, out, blockIdx.x);
#endif
}
} // namespace
"""


def _compile(source, *defines):
    return subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-device-only", "-fsyntax-only", "-std=c++17",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, *defines, str(source)],
                          capture_output=True, text=True)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("per_tensor", [0, 1])
@pytest.mark.parametrize("norm", [0, 1])
@pytest.mark.parametrize("tiles", [1, 2, 4])
def test_only_4096_element_chunks_compile(tmp_path, tiles, norm, per_tensor):
    source = tmp_path / "instantiate.hip"
    source.write_text(INSTANTIATE)
    res = _compile(source, f"-DTRY_TILES={tiles}", f"-DTRY_NORM={norm}", f"-DTRY_PER_TENSOR={per_tensor}")
    if tiles == 2:
        assert res.returncode == 0, res.stderr
    else:
        assert res.returncode != 0 and "static assertion failed" in res.stderr, res.stderr


def test_no_macro_sets_the_chunk_size():
    for name in ("dq_quantize_core.h", "dq_quantize_pack.hip"):
        text = open(os.path.join(CSRC, name)).read()
        assert "#ifndef" not in text and "DQ_QP_TILES" not in text, name
