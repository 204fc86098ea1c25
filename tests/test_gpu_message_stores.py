"""Messages stored with and without the streaming hint, on both sides of the lines between the two (messages of 4 and 16 MB,
12 and 18 M values): the oracle's bytes.  Lengths that leave the planes on and off the cache lines."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import SEED, dq  # noqa: F401  (dq is a fixture)

pytestmark = pytest.mark.gpu

MI, M = 1 << 20, 2
# MB of both messages at b = 3 and b = 8, and at the six bits that stand for a widths table
LAYOUTS = [[2 * MI + 77],                        # 2, 4.5, 3.5
           [5 * MI, 777],                        # 5, 11.3, 8.8
           [10 * MI + 129],                      # 10, 22.5, 17.5
           [12 * MI - 128], [12 * MI, 300, 4000],  # 12, 27, 21: one worker's line
           [18 * MI], [18 * MI + 1]]             # 18, 40.5, 31.5; beyond


@pytest.mark.parametrize("b", [3, 8])
@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
def test_messages_on_both_sides_of_the_lines(dq, oracle, layout, b):
    seg_len = LAYOUTS[layout]
    plan = dq.Plan(seg_len)
    rng = np.random.default_rng(layout)
    g = rng.standard_normal((M, plan.padded_elems), dtype=np.float32)
    norms = np.abs(g).max() * rng.uniform(0.5, 2.0, size=(M, len(seg_len))).astype(np.float32)
    want = oracle.quantize_pack(seg_len, g, norms, b, SEED, 3)
    gd, nd = torch.from_numpy(g).cuda(), torch.from_numpy(norms).cuda()
    table = dq.Widths(plan, [b] * len(seg_len))
    for pack in (lambda out: dq.quantize_pack(plan, gd, nd, b, SEED, 3, out),
                 lambda out: dq.quantize_pack_v(plan, table, gd, nd, SEED, 3, out)):
        packed = torch.full((M, plan.packed_bytes(b) + 32), 0xA5, dtype=torch.uint8, device="cuda")
        pack(packed)
        got = packed.cpu().numpy()
        # one width everywhere: the widths-table layout is the same bytes
        assert np.array_equal(got[:, :-32], want) and np.all(got[:, -32:] == 0xA5)
    plan.close()
