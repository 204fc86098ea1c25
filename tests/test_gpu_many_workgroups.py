"""Norms and messages on both sides of the line at which fewer workgroups are resident and the norms' partial sums are written through."""
import pytest
import torch

from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

LINE = 8192  # workgroups: norm items or chunks, all workers


@pytest.mark.parametrize("M,chunks", [(8, LINE // 8), (8, LINE // 8 - 1), (1, LINE), (64, LINE // 64)])
def test_both_sides_of_the_line(dq, M, chunks):
    n = chunks * 4096 - 5
    plan = dq.Plan([n - 1000, 1000])
    assert not plan.chunk_local
    gen = torch.Generator(device="cuda")
    gen.manual_seed(chunks)
    grads = torch.randn((M, plan.padded_elems), generator=gen, device="cuda")
    lens, starts = [n - 1000, 1000], [0, -(-(n - 1000) // 128) * 128]
    for s, k in zip(starts, lens):
        grads[:, s + k:s + -(-k // 128) * 128] = float("nan")
    ws = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
    norms, tops = (torch.full((M, 2), float("nan"), device="cuda") for _ in range(2))
    dq.norm(plan, grads, norms, ws)
    dq.norm_linf(plan, grads, tops, ws)
    for l, (s, k) in enumerate(zip(starts, lens)):
        data = grads[:, s:s + k]
        want = torch.stack([row.double().square().sum().sqrt() for row in data])
        # one rounding to binary32 of sums of fewer than 2^26 binary64 terms
        assert torch.all((norms[:, l].double() - want).abs() <= want * 2.0 ** -23)
        assert torch.equal(tops[:, l], data.abs().amax(dim=1))
    b = 3
    packed = torch.full((M, plan.packed_bytes(b)), 0xA5, dtype=torch.uint8, device="cuda")
    dq.quantize_pack(plan, grads, norms, b, 11, 2, packed)
    # the same chunks a few workers at a time, far below the line
    part = torch.full((1, plan.packed_bytes(b)), 0xA5, dtype=torch.uint8, device="cuda")
    for w in range(0, M, max(1, M // 4)):
        if M == 1:
            break
        dq.quantize_pack(plan, grads[w:w + 1], norms[w:w + 1], b, 11, 2, part, worker_base=w)
        assert torch.equal(part[0], packed[w]), w
    out = torch.empty(plan.padded_elems, device="cuda")
    dq.unpack_dequant_reduce(plan, packed, norms, b, out)
    unit = (norms.double() / 7).amax()
    mean = torch.nan_to_num(grads, nan=0.0).double().mean(dim=0)
    assert torch.all((out.double() - mean).abs() <= unit * 1.0001)  # every level within one of its value
    plan.close()
