"""The server average in its two forms -- a lane's 32 elements, or 16 with two workers to a decoded word -- on both sides of the lines between them, with
and without update, one width and a shared table: the bits of the kernel with a row of widths per worker, which has the first form only.  Per-worker widths,
tensors alike and mixed, against the workers' messages decoded one by one; scaled signs on both sides of their line."""
import pytest
import torch

from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

TILE = 8192
LINES = [(tiles, M) for tiles in (384, 385, 512, 513, 641, 768, 769, 1024, 1025, 1280, 1281) for M in (1, 3, 4, 5, 6, 9, 10, 13, 14, 16, 17, 32, 33, 64)]


# and beyond: the model passing through (from 3073 tiles on), fewer workgroups on a CU (4096 without and 8192 with update), messages
# of more than 640 MB
@pytest.mark.parametrize("tiles,M", LINES + [(3072, 33), (3073, 1), (3073, 16), (3073, 17), (3073, 33), (4097, 14), (4097, 17), (8192, 16), (8192, 17)])
def test_same_bits_as_with_a_row_of_widths_per_worker(dq, tiles, M):
    # ends inside a lane, a granule and a span, small tensors side by side, an empty one
    seg_len = [TILE * (tiles // 2) + 77, 1, 0, 129, 4096] + [130] * 60
    seg_len.append(TILE * tiles - sum(-(-n // 128) * 128 for n in seg_len) - 1000)
    plan = dq.Plan(seg_len)
    assert -(-plan.padded_elems // TILE) == tiles
    gen = torch.Generator(device="cuda")
    gen.manual_seed(tiles * 100 + M)
    norms = torch.rand((M, len(seg_len)), generator=gen, device="cuda") * 4 + 1e-3
    norms[M // 2, len(seg_len) // 2] = float("nan")
    norms[0, 0] = 0.0 if M > 1 else 2.0 ** -99
    for b in range(1, 9):
        packed = torch.randint(0, 256, (M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda", generator=gen)
        want = torch.full((plan.padded_elems,), float("nan"), device="cuda")
        table, rows = dq.Widths(plan, [b] * len(seg_len)), dq.Widths(plan, [[b] * len(seg_len)] * M, workers=M)
        dq.unpack_dequant_reduce_v(plan, rows, packed, norms, want)
        step = -0.25 * want + 0.0
        for update, call in ((False, lambda out, x: dq.unpack_dequant_reduce(plan, packed, norms, b, out)),
                             (False, lambda out, x: dq.unpack_dequant_reduce_v(plan, table, packed, norms, out)),
                             (True, lambda out, x: dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.25, x, ghat=out)),
                             (True, lambda out, x: dq.unpack_dequant_reduce_update_v(plan, table, packed, norms, 0.25, x, ghat=out))):
            got, x = torch.full_like(want, float("nan")), torch.zeros_like(want)
            call(got, x)
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
            if update:
                assert torch.equal(x.view(torch.int32), step.view(torch.int32)), b
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
