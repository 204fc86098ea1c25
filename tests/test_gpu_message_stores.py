"""Messages written through to the last-level cache and messages with the streaming hint, on both sides of the lines between the two
(190 to 640 MB of messages, by width, number of workers and layout): the oracle's bytes.  Lengths that leave the planes on and off the
cache lines, plans of large tensors and of small ones."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import SEED, dq  # noqa: F401  (dq is a fixture)

pytestmark = pytest.mark.gpu

MI, M = 1 << 20, 2
# MB of both messages at b = 3 and b = 8
LAYOUTS = [[2 * MI + 77],                        # 2, 4.5
           [5 * MI, 777],                        # 5, 11.3
           [10 * MI + 129],                      # 10, 22.5
           [12 * MI - 128], [12 * MI, 300, 4000],  # 12, 27
           [18 * MI], [18 * MI + 1]]             # 18, 40.5


@pytest.mark.parametrize("b", [3, 8])
@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
def test_moderate_messages(dq, oracle, layout, b):
    """2 to 40 MB, written through; planes on and off the cache lines."""
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


# (width, 0 for a widths table; workers; MB of messages up to which they are written through, a table's at six bits; the same for small tensors)
LINES = [(1, 64, 640, 640), (2, 64, 640, 640), (4, 64, 640, 640), (5, 32, 320, 190), (5, 64, 190, 190), (6, 32, 320, 190), (7, 32, 320, 190), (7, 64, 190, 190),
         (8, 33, 190, 190), (8, 32, 400, 400), (0, 32, 190, 190), (0, 64, 190, 190)]


def _layout(line, small, beyond):
    """A layout whose messages are just up to the line, or one granule beyond it: one large tensor or many of 1000 elements, both
    with a ragged end."""
    b, M, megabytes = line[0], line[1], line[2 + small]
    granules = (megabytes << 20) // (16 * ((b or 6) + 1) * M) + beyond
    seg_len = [1000] * (granules // 8 - 1) if small else []
    return seg_len + [(granules - 8 * len(seg_len)) * 128 - 51]


@pytest.mark.parametrize("beyond", [0, 1])
@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("line", LINES)
def test_messages_on_both_sides_of_the_lines(dq, oracle, line, small, beyond):
    """All workers at once against eight at a time (always written through), and the last worker's against the oracle."""
    b, workers, megabytes = line[0], line[1], line[2 + small]
    seg_len = _layout(line, small, beyond)
    plan = dq.Plan(seg_len)
    assert (workers * plan.packed_bytes(b or 6) > megabytes << 20) == bool(beyond)
    gen = torch.Generator(device="cuda").manual_seed(100 * b + workers + beyond)
    g = torch.randn((workers, plan.padded_elems), generator=gen, device="cuda")
    norms = 0.5 + 7.5 * torch.rand((workers, len(seg_len)), generator=gen, device="cuda")
    if b:
        n_bytes = plan.packed_bytes(b)

        def pack(gd, nd, out, first):
            dq.quantize_pack(plan, gd, nd, b, SEED, 3, out, worker_base=first)
    else:
        widths = [1 + (5 * l + 2) % 8 for l in range(len(seg_len))]
        table = dq.Widths(plan, widths)
        n_bytes = table.packed_bytes

        def pack(gd, nd, out, first):
            dq.quantize_pack_v(plan, table, gd, nd, SEED, 3, out, worker_base=first)
    packed = torch.full((workers, n_bytes + 48), 0xA5, dtype=torch.uint8, device="cuda")
    pack(g, norms, packed, 0)
    some = torch.full((8, n_bytes), 0x5A, dtype=torch.uint8, device="cuda")
    for first in range(0, workers, 8):
        n = min(8, workers - first)
        pack(g[first:first + n], norms[first:first + n], some[:n], first)
        assert torch.equal(packed[first:first + n, :n_bytes], some[:n])
    assert bool((packed[:, n_bytes:] == 0xA5).all())
    w = workers - 1
    gh, nh = g[w:].cpu().numpy(), norms[w:].cpu().numpy()
    want = (oracle.quantize_pack(seg_len, gh, nh, b, SEED, 3, worker_base=w) if b else
            oracle.quantize_pack_v(seg_len, gh, nh, widths, SEED, 3, worker_base=w))
    assert np.array_equal(packed[w:, :n_bytes].cpu().numpy(), want)
    plan.close()
