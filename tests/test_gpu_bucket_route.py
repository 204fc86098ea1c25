"""Gradients cut into buckets of 128 to 1024 values: norms and messages of the kernel whose wavefronts work out their own buckets' norms,
against dq_norm and dq_quantize_pack, which take other kernels, bit for bit (the oracle is compared with those elsewhere).  Lengths with a last bucket
that is whole, short, and alone in its chunk; no whole chunk at all; and layouts that look like buckets and are not."""
import pytest
import torch

from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _layouts():
    for size in (128, 256, 512, 1024, 2048, 4096):
        n = 4096 // size
        yield [size] * (3 * n)                 # whole chunks only
        yield [size] * (2 * n) + [1]           # a chunk of its own for one value
        yield [size] * (2 * n + n // 2) + [size - 7]
        yield [size] * max(1, n - 1)           # no whole chunk
    yield [512] * 16 + [511] + [512] * 7       # a shorter one that is not the last
    yield [512] * 8 + [1024] * 4
    yield [256] * 16 + [300]                   # the last one is longer


@pytest.mark.parametrize("linf", [False, True])
@pytest.mark.parametrize("layout", list(_layouts()), ids=lambda lens: f"{lens[0]}x{len(lens)}+{lens[-1]}")
def test_same_norms_and_messages_as_in_two_calls(dq, layout, linf):
    M, seed, step = 3, 0x1234567890ABCDEF, 5
    plan = dq.Plan(layout)
    assert plan.chunk_local
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(layout))
    grads = torch.randn((M, plan.padded_elems), generator=gen, device="cuda") * 1e-3
    start = 0
    for k, n in enumerate(layout):  # pads are never data; some buckets zero, some with one value that is all of the norm
        end = start + -(-n // 128) * 128
        grads[:, start + n:end] = float("nan")
        if k % 5 == 1:
            grads[0, start:start + n] = 0.0
        if k % 7 == 2:
            grads[1, start + n // 2] = 1e3
        start = end
    grads[2, 0] = float("inf")
    want_norms = torch.full((M, len(layout)), float("nan"), device="cuda")
    ws = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
    (dq.norm_linf if linf else dq.norm)(plan, grads, want_norms, ws)
    for b in range(1, 9):
        norms = torch.full_like(want_norms, float("nan"))
        got, want = (torch.full((M, plan.packed_bytes(b)), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(2))
        dq.quantize_pack(plan, grads, want_norms, b, seed, step, want)
        dq.norm_quantize_pack(plan, grads, b, seed, step, norms, got, linf=linf)
        assert torch.equal(norms.view(torch.int32), want_norms.view(torch.int32)), b
        assert torch.equal(got, want), b
    plan.close()


@pytest.mark.parametrize("size", [128, 256, 512, 1024])
@pytest.mark.parametrize("linf", [False, True])
def test_norms_at_the_ends_of_the_range(dq, size, linf):
    """Buckets of subnormal values, of values around the smallest usable norm, near the largest value (a norm beyond it is infinite) and with one
    NaN: the norms of dq_norm (a NaN is one, whatever its bits) and the messages for them."""
    scales = [2.0 ** -149, 2.0 ** -140, 2.0 ** -126, 2.0 ** -101, 2.0 ** -100, 2.0 ** -60, 1.0, 2.0 ** 100, 2.0 ** 122, 2.0 ** 127]
    n = 2 * 4096 // size * len(scales)
    plan = dq.Plan([size] * n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(size)
    of = torch.tensor(scales, dtype=torch.float64, device="cuda").repeat(2 * 4096 // size).unsqueeze(1)
    grads = ((torch.rand((2, n, size), generator=gen, device="cuda", dtype=torch.float64) * 3.9 - 1.95) * of).float()
    grads[1, ::3, size // 2] = float("nan")
    grads[1, ::7, 0] = float("-inf")
    grads = grads.reshape(2, -1)
    want = torch.empty((2, n), device="cuda")
    (dq.norm_linf if linf else dq.norm)(plan, grads, want, torch.empty(plan.workspace_bytes(2), dtype=torch.uint8, device="cuda"))
    if not linf:  # and those are the root of the squares' sum to one rounding
        exact = grads.double().reshape(2, n, size).square().sum(dim=2).sqrt().float()
        lo, hi = torch.nextafter(exact, torch.zeros_like(exact)), torch.nextafter(exact, torch.full_like(exact, float("inf")))
        assert torch.all(torch.isnan(exact) & torch.isnan(want) | (want >= lo) & (want <= hi))
    for b in (1, 4, 8):
        norms = torch.full_like(want, 7.0)
        got, packed = (torch.full((2, plan.packed_bytes(b)), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(2))
        dq.norm_quantize_pack(plan, grads, b, 3, 1, norms, got, linf=linf)
        assert torch.equal(torch.isnan(norms), torch.isnan(want))
        assert torch.equal(torch.nan_to_num(norms, nan=-1.0).view(torch.int32), torch.nan_to_num(want, nan=-1.0).view(torch.int32)), b
        dq.quantize_pack(plan, grads, want, b, 3, 1, packed)
        assert torch.equal(got, packed), b
    plan.close()
