"""Quantize+pack on layouts around the line where the plan changes the kernels' form: a quarter of the 4096-element
chunks inside one tensor.  Messages bit for bit against the oracle, averages within the tolerance of
test_gpu_parity, one width for all tensors and one per tensor."""
import numpy as np
import pytest

from tests.test_gpu_chunk_edges import _gradients
from tests.test_gpu_parity import _one_step, dq  # noqa: F401  (dq is a fixture)
from tests.test_gpu_per_tensor import _one_step_v

pytestmark = pytest.mark.gpu

LAYOUTS = [
    [4096] + [1000] * 12,                # 1 of 4 chunks
    [4096] + [1000] * 13,                # 1 of 5
    [128] * 65 + [4096 * 2 + 5, 77],     # unaligned large one
    [3000] * 7, [6000] * 7, [129] * 33, [0, 5, 0, 4095, 4097, 300],
]


@pytest.mark.parametrize("seg_len", LAYOUTS, ids=lambda s: f"{len(s)}x{s[0]}_{s[-1]}")
def test_one_width(dq, oracle, seg_len):
    grads = _gradients(seg_len, 3)
    for b in (1, 3, 6, 8):
        _one_step(dq, oracle, seg_len, grads, b, step=b)


@pytest.mark.parametrize("seg_len", LAYOUTS, ids=lambda s: f"{len(s)}x{s[0]}_{s[-1]}")
def test_width_per_tensor(dq, oracle, seg_len):
    grads = _gradients(seg_len, 3)
    widths = [np.array([(l * 3 + k) % 8 + 1 for l in range(len(seg_len))]) for k in (0, 5)]
    _one_step_v(dq, oracle, seg_len, grads, widths, step=2)
