"""Sign messages of chunks inside and across tensors, at places on and off the cache lines."""
import pytest
import torch

from tests.test_gpu_parity import dq  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _signs(grads, lens, starts, padded):
    bits = torch.zeros((grads.shape[0], padded), dtype=torch.uint8, device=grads.device)
    for s, n in zip(starts, lens):
        bits[:, s:s + n] = torch.signbit(grads[:, s:s + n]).to(torch.uint8)
    weights = (1 << torch.arange(8, device=grads.device)).to(torch.int32)
    return (bits.view(grads.shape[0], -1, 8).to(torch.int32) * weights).sum(dim=2).to(torch.uint8)


@pytest.mark.parametrize("skew", [0, 16, 112])
@pytest.mark.parametrize("lens", [[1], [4096], [4095], [8192, 1], [5000, 0, 9000, 129], [128] * 40, [20000, 4096 * 3], [4096 * 9 - 127],
                                  # small tensors over several groups of four tiles; half of the chunks of one tensor, and one chunk less
                                  [300] * 100, [1000] * 17 + [1], [8192, 3000, 3000], [8192, 3000, 3000, 3000]])
def test_sign_messages(dq, lens, skew):
    M = 2
    plan = dq.Plan(lens)
    starts, at = [], 0
    for n in lens:
        starts.append(at)
        at += -(-n // 128) * 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(at + skew)
    grads = torch.randn((M, plan.padded_elems), generator=gen, device="cuda")
    grads[0, ::3] = -0.0
    grads[1, 1::5] = 0.0
    for s, n in zip(starts, lens):
        grads[:, s + n:s + -(-n // 128) * 128] = -1.0  # pads count as positive whatever they hold
    nbytes = plan.padded_elems // 8
    room = -(-nbytes // 128) * 128 + skew
    flat = torch.full((M * room + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    packed = flat[skew:skew + M * room].view(M, room)
    dq.sign_pack(plan, grads, packed)
    assert torch.equal(packed[:, :nbytes], _signs(grads, lens, starts, plan.padded_elems))
    assert bool((packed[:, nbytes:] == 0xA5).all()) and bool((flat[:skew] == 0xA5).all())
    plan.close()
