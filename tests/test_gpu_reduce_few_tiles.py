"""The server average on both sides of the lines between its kernels for few tiles (a lane's 8 elements, workers divided over wavefronts, two workers to a
decoded word), one width and a shared table: the same bits as the kernel with a row of widths per worker, which has one form for every size (a lane's 32
elements), and that one is compared with the oracle elsewhere (test_gpu_reduce_routes).  Messages are random bytes, norms include unusable ones."""
import pytest
import torch

from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

TILE = 8192
# elements: below a wavefront, ends inside a lane, a granule and a span, and on and beyond 64, 128 and 192 tiles, on 256
LAYOUTS = [
    [1], [200, 0, 7, 129, 511], [4096], [512 * 3, 1, 2048 * 2 + 77], [300] * 40, [TILE * 64 - 900, 640], [TILE * 64 + 1],
    [TILE * 100, 5, TILE * 28 - 128], [TILE * 128 + 1], [TILE * 192 - 3], [TILE * 193], [TILE * 255, 130, 4000],
]


@pytest.mark.parametrize("M", [1, 4, 8, 9, 16, 24, 25, 32, 40, 41, 57, 64])
@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
def test_same_bits_as_with_a_row_of_widths_per_worker(dq, layout, M):
    seg_len = LAYOUTS[layout]
    plan = dq.Plan(seg_len)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(layout * 100 + M)
    norms = torch.rand((M, len(seg_len)), generator=gen, device="cuda") * 4 + 1e-3
    norms[M // 2, len(seg_len) // 2] = float("nan")
    norms[0, 0] = 0.0 if M > 1 else 2.0 ** -99
    x0 = torch.randn(plan.padded_elems, generator=gen, device="cuda")
    for b in range(1, 9):
        packed = torch.randint(0, 256, (M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda", generator=gen)
        want, got = torch.full_like(x0, float("nan")), torch.full_like(x0, float("nan"))
        table, rows = dq.Widths(plan, [b] * len(seg_len)), dq.Widths(plan, [[b] * len(seg_len)] * M, workers=M)
        dq.unpack_dequant_reduce_v(plan, rows, packed, norms, want)
        dq.unpack_dequant_reduce(plan, packed, norms, b, got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        got.fill_(float("nan"))
        dq.unpack_dequant_reduce_v(plan, table, packed, norms, got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        x, y, z, ghat = x0.clone(), x0.clone(), x0.clone(), torch.full_like(x0, float("nan"))
        dq.unpack_dequant_reduce_update_v(plan, rows, packed, norms, 0.25, x)
        dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.25, y, ghat=ghat)
        dq.unpack_dequant_reduce_update_v(plan, table, packed, norms, 0.25, z)
        assert torch.equal(y.view(torch.int32), x.view(torch.int32)), b
        assert torch.equal(z.view(torch.int32), x.view(torch.int32)), b
        assert torch.equal(ghat.view(torch.int32), want.view(torch.int32)), b
    plan.close()


@pytest.mark.parametrize("M", [40, 57, 64])
@pytest.mark.parametrize("seg_len", [[TILE * 256 + 1], [300, TILE * 299 + 4000], [TILE * 320 - 130], [TILE * 320 - 200, 77, 128],
                                     [TILE * 380 - 5], [TILE * 380 + 1]])
def test_same_bits_on_both_sides_of_the_farthest_lines(dq, seg_len, M):
    """Beyond 256 tiles, on and beyond 320 and 380; 1199 spans, which the order of the workgroups does not divide."""
    plan = dq.Plan(seg_len)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    norms = torch.rand((M, len(seg_len)), generator=gen, device="cuda") * 4 + 1e-3
    x0 = torch.randn(plan.padded_elems, generator=gen, device="cuda")
    for b in range(1, 9):
        packed = torch.randint(0, 256, (M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda", generator=gen)
        want, got = torch.full_like(x0, float("nan")), torch.full_like(x0, float("nan"))
        table, rows = dq.Widths(plan, [b] * len(seg_len)), dq.Widths(plan, [[b] * len(seg_len)] * M, workers=M)
        dq.unpack_dequant_reduce_v(plan, rows, packed, norms, want)
        dq.unpack_dequant_reduce(plan, packed, norms, b, got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        got.fill_(float("nan"))
        dq.unpack_dequant_reduce_v(plan, table, packed, norms, got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        x, y = x0.clone(), x0.clone()
        dq.unpack_dequant_reduce_update_v(plan, rows, packed, norms, 0.25, x)
        dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.25, y)
        assert torch.equal(y.view(torch.int32), x.view(torch.int32)), b
    plan.close()


@pytest.mark.parametrize("M", [2, 7, 8, 9, 24, 32, 40, 64])
@pytest.mark.parametrize("seg_len", [[200, 0, 7, 129, 511], [4096 + 640], [TILE * 64 - 900, 640], [TILE * 100, 5, TILE * 28 - 128]])
def test_sum_beyond_the_largest_value_with_a_finite_average(dq, seg_len, M):
    """Every worker at the top level with one sign and a norm near the largest binary32 value: the sum over the workers
    passes it, the average does not.  The same bits as with a row of widths per worker, and N to the sum's rounding: at most
    7 + ceil(M / 8) roundings of the sum, and three more (N / s, s products, 1 / M), of 2^-24 each."""
    plan = dq.Plan(seg_len)
    N = 3.0e38
    norms = torch.full((M, len(seg_len)), N, device="cuda")
    bound = (7 + -(-M // 8) + 3) * 2.0 ** -24
    for b in range(1, 9):
        packed = torch.full((M, plan.packed_bytes(b)), 255, dtype=torch.uint8, device="cuda")
        packed[:, :plan.padded_elems // 8] = 0  # the signs
        want, got = (torch.full((plan.padded_elems,), float("nan"), device="cuda") for _ in range(2))
        table, rows = dq.Widths(plan, [b] * len(seg_len)), dq.Widths(plan, [[b] * len(seg_len)] * M, workers=M)
        dq.unpack_dequant_reduce_v(plan, rows, packed, norms, want)
        dq.unpack_dequant_reduce(plan, packed, norms, b, got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        got.fill_(float("nan"))
        dq.unpack_dequant_reduce_v(plan, table, packed, norms, got)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), b
        data = got[got != 0].double()
        assert data.numel() == sum(seg_len) and torch.all((data / N - 1).abs() <= bound), b
        x = torch.zeros_like(got)
        dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.25, x)
        assert torch.equal(x.view(torch.int32), (-0.25 * got + 0.0).view(torch.int32)), b
    plan.close()
