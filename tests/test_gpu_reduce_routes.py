"""The server average where its kernels change route: wavefronts of 2048 elements inside one tensor, shared
by several, and cut short by the layout's end; tile counts around the multiples of 32 in which workgroups
are assigned; widths 5 to 8 (levels as 16-bit floats) at both ends of the usable norms; one width for all
workers of a tensor and mixed ones.  Messages are random codes packed by the oracle.  The reference is the mean of the
same binary32 terms in binary64, worked out here; the oracle's average (rounded to binary32) is compared where the norms
are moderate.

Tolerance: that of test_gpu_average_worst_case, 1e-6 of the mean magnitude of the terms."""
import numpy as np
import pytest
import torch

from paper_2107_14575_amd import workloads as wl
from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

LAYOUTS = [
    [2048], [2047], [2049], [128], [1], [2048 * 3 + 128, 1920, 2048],
    [1, 0, 127, 129, 2048 * 2, 5, 2048 - 128, 4096 - 1],
    [8192 * 31 + 5, 700], [8192 * 32], [8192 * 33 + 300, 1, 2048 * 5 + 130],
]


def _codes(seg_len, M, b_of, rng):
    """sign and level [M][D'] with zero padding; level < 2^b, the top level frequent"""
    starts, dp = wl.seg_starts(seg_len)
    sign = np.zeros((M, dp), dtype=np.uint8)
    level = np.zeros((M, dp), dtype=np.uint8)
    for l, (st, n) in enumerate(zip(starts, seg_len)):
        for i in range(M):
            s = (1 << int(b_of(i, l))) - 1
            sign[i, st:st + n] = rng.integers(0, 2, n)
            level[i, st:st + n] = np.where(rng.random(n) < 0.2, s, rng.integers(0, s + 1, n))
    return starts, sign, level


def _reference(seg_len, starts, sign, level, norms, b_of):
    """binary64 mean and mean magnitude of the terms; unit N/s and the products in binary32 as the method has them"""
    M, dp = sign.shape
    mean, mag = np.zeros(dp), np.zeros(dp)
    for l, (st, n) in enumerate(zip(starts, seg_len)):
        for i in range(M):
            unit = np.float32(norms[i, l] / np.float32((1 << int(b_of(i, l))) - 1))
            t = (level[i, st:st + n].astype(np.float32) * unit).astype(np.float64)
            mean[st:st + n] += np.where(sign[i, st:st + n] == 1, -t, t)
            mag[st:st + n] += t
    return mean / M, mag / M


def _check(got, mean, mag):
    assert np.all(np.abs(got.astype(np.float64) - mean) <= 1e-6 * mag)
    assert np.array_equal(got[mag == 0], np.zeros(int((mag == 0).sum()), dtype=np.float32))


@pytest.mark.parametrize("seg_len", LAYOUTS, ids=lambda s: "_".join(map(str, s)))
@pytest.mark.parametrize("b", [1, 2, 3, 4, 5, 6, 7, 8])
def test_one_width(dq, oracle, seg_len, b):
    M = (5, 8, 17, 3)[b % 4]
    rng = np.random.default_rng(b * 100 + len(seg_len))
    plan = dq.Plan(seg_len)
    starts, sign, level = _codes(seg_len, M, lambda i, l: b, rng)
    norms = (10.0 ** rng.uniform(-2, 1, (M, len(seg_len)))).astype(np.float32)
    packed = torch.from_numpy(np.stack([oracle.pack(sign[i], level[i], b) for i in range(M)])).cuda()
    norms_dev = torch.from_numpy(norms).cuda()
    mean, mag = _reference(seg_len, starts, sign, level, norms, lambda i, l: b)
    out = torch.full((plan.padded_elems,), float("nan"), device="cuda")
    dq.unpack_dequant_reduce(plan, packed, norms_dev, b, out)
    _check(out.cpu().numpy(), mean, mag)
    _check(out.cpu().numpy(), oracle.unpack_dequant_reduce(seg_len, packed.cpu().numpy(), norms, b).astype(np.float64), mag)
    # with update: the average beside it has the same bits, x is one FMA of it
    x0 = rng.standard_normal(plan.padded_elems).astype(np.float32)
    x, ghat = torch.from_numpy(x0).cuda(), torch.full_like(out, float("nan"))
    dq.unpack_dequant_reduce_update(plan, packed, norms_dev, b, 0.5, x, ghat=ghat)
    assert torch.equal(ghat, out)
    want = x0.astype(np.float64) - 0.5 * out.cpu().numpy().astype(np.float64)
    assert np.array_equal(x.cpu().numpy(), want.astype(np.float32))
    # the same messages through both kinds of widths tables: the same bits
    for table in (dq.Widths(plan, [b] * len(seg_len)), dq.Widths(plan, [[b] * len(seg_len)] * M, workers=M)):
        again = torch.full_like(out, float("nan"))
        dq.unpack_dequant_reduce_v(plan, table, packed, norms_dev, again)
        assert torch.equal(again, out)
        table.close()
    plan.close()


@pytest.mark.parametrize("b", [1, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("exponent", [-100, -98, -60, 100, 127])
def test_norms_at_the_ends_of_the_range(dq, oracle, b, exponent):
    """Two workers, of which at most one has a level above zero, so that no sum overflows at 1.99 * 2^127."""
    seg_len = [2048 + 300, 4096]
    M = 2
    rng = np.random.default_rng(b)
    plan = dq.Plan(seg_len)
    starts, sign, level = _codes(seg_len, M, lambda i, l: b, rng)
    level[1, level[0] > 0] = 0
    norms = np.full((M, 2), np.float32(np.ldexp(1.99, exponent)), dtype=np.float32)
    packed = torch.from_numpy(np.stack([oracle.pack(sign[i], level[i], b) for i in range(M)])).cuda()
    norms_dev = torch.from_numpy(norms).cuda()
    mean, mag = _reference(seg_len, starts, sign, level, norms, lambda i, l: b)
    tables = [dq.Widths(plan, [b, b]), dq.Widths(plan, [[b, b]] * M, workers=M)]
    for table in [None] + tables:
        out = torch.full((plan.padded_elems,), float("nan"), device="cuda")
        if table is None:
            dq.unpack_dequant_reduce(plan, packed, norms_dev, b, out)
        else:
            dq.unpack_dequant_reduce_v(plan, table, packed, norms_dev, out)
        _check(out.cpu().numpy(), mean, mag)
    for t in tables:
        t.close()
    plan.close()


@pytest.mark.parametrize("M", [2, 5, 12])
def test_workers_of_mixed_widths(dq, oracle, M):
    """tensors of one width for all workers next to mixed ones, whole wavefronts and shared ones, small and large norms"""
    seg_len = [2048 * 3, 2048 * 3, 300, 2048 * 2 + 5, 128, 6000]
    rng = np.random.default_rng(M)
    widths = rng.integers(1, 9, (M, len(seg_len)))
    widths[:, 0], widths[:, 3], widths[:, 5] = 6, 3, 8
    plan = dq.Plan(seg_len)
    starts, sign, level = _codes(seg_len, M, lambda i, l: widths[i, l], rng)
    norms = (2.0 ** rng.uniform(-100, -90, (M, len(seg_len)))).astype(np.float32)
    norms[:, 1] = 1.5
    norms[:, 3] = np.float32(2.0 ** 120)
    table = dq.Widths(plan, widths, workers=M)
    packed = np.zeros((M, table.packed_bytes), dtype=np.uint8)
    for i in range(M):
        one = oracle.pack_v(sign[i], level[i], seg_len, widths[i])
        packed[i, :one.size] = one
    mean, mag = _reference(seg_len, starts, sign, level, norms, lambda i, l: widths[i, l])
    out = torch.full((plan.padded_elems,), float("nan"), device="cuda")
    dq.unpack_dequant_reduce_v(plan, table, torch.from_numpy(packed).cuda(), torch.from_numpy(norms).cuda(), out)
    _check(out.cpu().numpy(), mean, mag)
    _check(out.cpu().numpy(), oracle.unpack_dequant_reduce_w(seg_len, packed, norms, widths).astype(np.float64), mag)
    table.close()
    plan.close()


@pytest.mark.parametrize("b", [1, 2, 3, 4])
@pytest.mark.parametrize("M", [15, 16, 17, 31, 64])
def test_groups_of_workers(dq, oracle, b, M):
    """Several workers' loads go out at once (eight here, by the forms for few tiles): full groups, and what is left of the next one,
    on workgroups all of whose wavefronts hold data and on ones whose last wavefronts hold none."""
    for seg_len in ([8192 + 2048 + 1], [300, 2048, 129, 8192 * 2]):
        rng = np.random.default_rng(1000 * b + M)
        plan = dq.Plan(seg_len)
        starts, sign, level = _codes(seg_len, M, lambda i, l: b, rng)
        norms = (10.0 ** rng.uniform(-2, 1, (M, len(seg_len)))).astype(np.float32)
        packed = torch.from_numpy(np.stack([oracle.pack(sign[i], level[i], b) for i in range(M)])).cuda()
        mean, mag = _reference(seg_len, starts, sign, level, norms, lambda i, l: b)
        out = torch.full((plan.padded_elems,), float("nan"), device="cuda")
        dq.unpack_dequant_reduce(plan, packed, torch.from_numpy(norms).cuda(), b, out)
        _check(out.cpu().numpy(), mean, mag)
        plan.close()


@pytest.mark.parametrize("b", [5, 6, 7])
def test_update_with_more_than_the_last_level_cache_holds(dq, b):
    """Messages and model of more than 256 MB take other loads with the update: the average has the bits of the
    kernel without update, and the model is one FMA of it."""
    M, seg_len = 16, [(1 << 24) + 3 * 2048 + 77, 300, (1 << 20) + 1]
    gen = torch.Generator(device="cuda").manual_seed(b)
    plan = dq.Plan(seg_len)
    assert plan.padded_elems * (M * (b + 1) + 32) // 8 > 256 << 20
    packed = torch.empty((M, plan.packed_bytes(b) // 8), dtype=torch.int64, device="cuda").random_(generator=gen).view(torch.uint8)
    norms = torch.rand((M, len(seg_len)), generator=gen, device="cuda") + 0.5
    out = torch.full((plan.padded_elems,), float("nan"), device="cuda")
    dq.unpack_dequant_reduce(plan, packed, norms, b, out)
    x0 = torch.randn(plan.padded_elems, generator=gen, device="cuda")
    x, ghat = x0.clone(), torch.full_like(out, float("nan"))
    dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.5, x, ghat=ghat)
    assert torch.equal(ghat, out)
    # 0.5 * out is exact, so the FMA is the rounded sum of two binary32 numbers
    assert torch.equal(x, x0 - 0.5 * out)
    plan.close()
