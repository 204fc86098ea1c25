"""Layouts whose tensors begin and end around multiples of 4096 padded elements: there the quantize
and reduce kernels change between the route for a stretch of one tensor and the route with a table
of tensors.  Messages bit for bit against the oracle, averages within the tolerance of test_gpu_parity."""
import numpy as np
import pytest
import torch

from paper_2107_14575_amd import workloads as wl
from tests.test_gpu_parity import _one_step, dq  # noqa: F401  (dq is a fixture)
from tests.test_gpu_per_tensor import _one_step_v

pytestmark = pytest.mark.gpu

LAYOUTS = [
    [4095], [4096], [4097], [3 * 4096, 5], [128, 2 * 4096 - 128, 4096], [1, 4096 * 2],
    [4096 - 128, 8192 + 127, 129], [0, 4096, 0, 4096 * 3 - 1, 0], [8192 - 1, 8192, 2048, 2049, 4096],
]


def _gradients(seg_len, M):
    starts, dp = wl.seg_starts(seg_len)
    grads = torch.full((M, dp), float("nan"), dtype=torch.float32)
    gen = torch.Generator().manual_seed(77)
    for l, (st, n) in enumerate(zip(starts, seg_len)):
        # magnitudes apart by tensor, so that a scale taken from a neighbour cannot go unseen
        grads[:, st:st + n] = torch.randn((M, n), generator=gen) * 10.0 ** (l % 4 - 3)
    return grads


@pytest.mark.parametrize("seg_len", LAYOUTS, ids=lambda s: "_".join(map(str, s)))
def test_one_width(dq, oracle, seg_len):
    grads = _gradients(seg_len, 3)
    for b in (1, 4, 7):
        _one_step(dq, oracle, seg_len, grads, b, step=b)


@pytest.mark.parametrize("seg_len", LAYOUTS, ids=lambda s: "_".join(map(str, s)))
def test_width_per_tensor(dq, oracle, seg_len):
    grads = _gradients(seg_len, 3)
    widths = [np.array([(l * 3 + k) % 8 + 1 for l in range(len(seg_len))]) for k in (0, 5)]
    _one_step_v(dq, oracle, seg_len, grads, widths, step=2)
