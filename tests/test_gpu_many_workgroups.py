"""Norms and messages on both sides of the line at which fewer workgroups are resident and the norms' partial sums are written through:
the tensor of a plan just below it and the same tensor of a plan with one small one more, which is on it, bit for bit."""
import pytest
import torch

from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

LINE = 8192  # workgroups: norm items (pieces of up to 4096 values of a tensor) or chunks of 4096, all workers


@pytest.mark.parametrize("M", [1, 8, 64])
def test_both_sides_of_the_line(dq, M):
    n = (LINE // M - 1) * 4096 - 5
    below, on = dq.Plan([n]), dq.Plan([n, 1000])
    for plan, count in ((below, LINE // M - 1), (on, LINE // M)):
        assert sum(-(-k // 4096) for k in plan.seg_len) == count and -(-plan.padded_elems // 4096) == count
        assert not plan.chunk_local and plan.workspace_bytes(M) == -(-M * count * 8 // 16) * 16  # 8 bytes an item
    D = below.padded_elems
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    grads = torch.randn((M, on.padded_elems), generator=gen, device="cuda")
    grads[:, n:D] = float("nan")
    grads[:, D + 1000:] = float("nan")
    norms, tops, packed, b = {}, {}, {}, 3
    for plan in (below, on):
        ws = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
        norms[plan], tops[plan] = (torch.full((M, plan.n_seg), float("nan"), device="cuda") for _ in range(2))
        data = grads[:, :plan.padded_elems]
        dq.norm(plan, data, norms[plan], ws)
        dq.norm_linf(plan, data, tops[plan], ws)
        packed[plan] = torch.full((M, plan.packed_bytes(b)), 0xA5, dtype=torch.uint8, device="cuda")
        dq.quantize_pack(plan, data, norms[plan], b, 11, 2, packed[plan])
    assert torch.equal(norms[on][:, 0], norms[below][:, 0]) and torch.equal(tops[on][:, 0], tops[below][:, 0])
    for l, data in enumerate((grads[:, :n], grads[:, D:D + 1000])):
        # one rounding to binary32 of sums of fewer than 2^26 binary64 terms
        want = torch.stack([row.double().square().sum().sqrt() for row in data])
        assert torch.all((norms[on][:, l].double() - want).abs() <= want * 2.0 ** -23)
        assert torch.equal(tops[on][:, l], data.abs().amax(dim=1))
    # the first tensor's stretch of either plane
    level = on.padded_elems // 8
    assert torch.equal(packed[on][:, :D // 8], packed[below][:, :D // 8])
    assert torch.equal(packed[on][:, level:level + D * b // 8], packed[below][:, D // 8:])
    out = torch.empty(on.padded_elems, device="cuda")
    dq.unpack_dequant_reduce(on, packed[on], norms[on], b, out)
    mean = torch.nan_to_num(grads, nan=0.0).double().mean(dim=0)
    assert torch.all((out.double() - mean).abs() <= (norms[on].double() / 7).amax() * 1.0001)  # every level within one of its value
    below.close()
    on.close()


@pytest.mark.parametrize("tensors,length,streams", [(1100, 4200, False), (500, 9000, False), (280, 16200, True)])
def test_norms_of_small_and_large_tensors(dq, tensors, length, streams):
    """Many workgroups of small items, and of nearly full ones: the norms of the first worker alone, which is below the line, bit for bit."""
    M = 8
    plan = dq.Plan([length] * tensors)
    items = tensors * -(-length // 4096)
    assert not plan.chunk_local and M * items >= LINE > items and (plan.padded_elems >= items * 3584) == streams
    gen = torch.Generator(device="cuda")
    gen.manual_seed(tensors)
    grads = torch.randn((M, plan.padded_elems), generator=gen, device="cuda")
    ws = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
    for norm in (dq.norm, dq.norm_linf):
        together, alone = torch.full((M, tensors), float("nan"), device="cuda"), torch.full((1, tensors), float("nan"), device="cuda")
        norm(plan, grads, together, ws)
        for w in range(M):
            norm(plan, grads[w:w + 1], alone, ws)
            assert torch.equal(together[w:w + 1], alone)
    plan.close()
