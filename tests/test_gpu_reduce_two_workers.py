"""The server average with a lane's 32 elements against the form in which two workers share a decoded word (a lane has 16), on layouts and
calls where one entry point takes the one and the other the other: the same bits.  Per-worker widths, tensors alike and mixed, against the workers'
messages decoded one by one, which the shared-width kernel does in the second form; scaled signs on both sides of their line."""
import pytest
import torch

from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

TILE = 8192
# more than 600 tiles; ends inside a lane, a granule and a span, small tensors side by side, an empty one
LAYOUTS = [[TILE * 601 - 5], [TILE * 300 + 77, 1, 0, 129, 4096, TILE * 302 - 1000] + [130] * 60]


@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
@pytest.mark.parametrize("M,widths", [(1, range(1, 9)), (2, range(1, 9)), (3, range(1, 5)), (5, range(1, 5)), (8, [3]), (9, [3]), (11, [3])])
def test_same_bits_with_and_without_update(dq, layout, M, widths):
    seg_len = LAYOUTS[layout]
    plan = dq.Plan(seg_len)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(layout * 100 + M)
    norms = torch.rand((M, len(seg_len)), generator=gen, device="cuda") * 4 + 1e-3
    norms[M // 2, len(seg_len) // 2] = float("nan")
    norms[0, 0] = 0.0 if M > 1 else 2.0 ** -99
    for b in widths:
        packed = torch.randint(0, 256, (M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda", generator=gen)
        want, got = (torch.full((plan.padded_elems,), float("nan"), device="cuda") for _ in range(2))
        x = torch.zeros_like(want)
        dq.unpack_dequant_reduce(plan, packed, norms, b, want)
        dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.25, x, ghat=got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        assert torch.equal(x.view(torch.int32), (-0.25 * want + 0.0).view(torch.int32)), b
        table = dq.Widths(plan, [b] * len(seg_len))
        got.fill_(float("nan"))
        dq.unpack_dequant_reduce_v(plan, table, packed, norms, got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        got.fill_(float("nan"))
        dq.unpack_dequant_reduce_update_v(plan, table, packed, norms, 0.25, x, ghat=got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
    plan.close()


@pytest.mark.parametrize("update", [False, True])
@pytest.mark.parametrize("M", [2, 7, 8, 9, 33, 64])
@pytest.mark.parametrize("odd_share", [0, 1], ids=["most alike", "few alike"])
def test_per_worker_widths(dq, M, odd_share, update):
    """Sums of M products in blocks of eight, times 1 / M: at most M / 8 + 8 roundings of 2^-24 (the products' own among them), and one
    each of the separately decoded values and of the scaling."""
    seg_len = [40000, 300, 0, 128, 1, 5000, 777, 2048, 100]
    mixed = range(1, 9) if odd_share == 0 else range(0, 9)
    plan = dq.Plan(seg_len)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    widths = torch.randint(1, 9, (1, len(seg_len)), generator=torch.Generator().manual_seed(M)).repeat(M, 1)
    for l in mixed:
        if l % 2 == 0:
            widths[:, l] = torch.randint(1, 9, (M,), generator=torch.Generator().manual_seed(M + l))
    rows = [[int(v) for v in row] for row in widths]
    norms = torch.rand((M, len(seg_len)), generator=gen, device="cuda") * 4 + 1e-3
    table = dq.Widths(plan, rows, workers=M)
    packed = torch.randint(0, 256, (M, plan.packed_bytes(8)), dtype=torch.uint8, device="cuda", generator=gen)
    total, size = (torch.zeros(plan.padded_elems, dtype=torch.float64, device="cuda") for _ in range(2))
    for w in range(M):
        one = torch.full((plan.padded_elems,), float("nan"), device="cuda")
        dq.unpack_dequant_reduce_v(plan, dq.Widths(plan, rows[w]), packed[w:w + 1], norms[w:w + 1], one)
        total += one.double()
        size += one.double().abs()
    got = torch.full((plan.padded_elems,), float("nan"), device="cuda")
    if update:
        x = torch.zeros_like(got)
        dq.unpack_dequant_reduce_update_v(plan, table, packed, norms, 0.5, x, ghat=got)
        assert torch.equal(x.view(torch.int32), (-0.5 * got + 0.0).view(torch.int32))
    else:
        dq.unpack_dequant_reduce_v(plan, table, packed, norms, got)
    bound = (M / 8 + 10) * 2.0 ** -24 * size / M + 1e-45
    assert torch.all((got.double() - total / M).abs() <= bound)
    plan.close()


@pytest.mark.parametrize("M", [1, 4, 9, 64])
@pytest.mark.parametrize("tiles", [200, 201])
def test_scaled_signs_on_both_sides_of_the_line(dq, tiles, M):
    """The mean of +-scale, in order of the workers: at most M roundings of 2^-24 of the sum of the scales, and one of the scaling."""
    seg_len = [TILE * (tiles - 1) - 1000, 900, 5000]
    plan = dq.Plan(seg_len)
    assert -(-plan.padded_elems // TILE) == tiles
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    scales = torch.rand((M, 3), generator=gen, device="cuda") + 0.1
    packed = torch.randint(0, 256, (M, plan.padded_elems // 8), dtype=torch.uint8, device="cuda", generator=gen)
    out = torch.full((plan.padded_elems,), float("nan"), device="cuda")
    dq.sign_reduce(plan, packed, out, scales=scales)
    bits = (packed.unsqueeze(2) >> torch.arange(8, device="cuda", dtype=torch.uint8)).bitwise_and(1).reshape(M, -1)
    start = 0
    for l, n in enumerate(seg_len):
        want = ((1.0 - 2.0 * bits[:, start:start + n].double()) * scales[:, l:l + 1].double()).sum(dim=0) / M
        bound = (M + 1) * 2.0 ** -24 * float(scales[:, l].double().sum()) / M
        assert torch.all((out[start:start + n].double() - want).abs() <= bound)
        end = start + -(-n // 128) * 128
        assert torch.all(out[start + n:end] == 0)
        start = end
    plan.close()
