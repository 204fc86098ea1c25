"""A runtime error that another part of the program left behind (here: a device number that does not exist, refused
by the host runtime) is not reported by the next call of the library, which does its work and returns ok."""
import ctypes

import pytest
import torch

from tests.test_gpu_parity import SEED, dq  # noqa: F401  (dq is a fixture)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hip(dq):
    torch.zeros(1, device="cuda")
    dq.load_library()
    paths = sorted({line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line})
    assert len(paths) == 1, paths
    return ctypes.CDLL(paths[0])


CALLS = ["norm", "norm_linf", "norm_bracket", "quantize_pack", "quantize_pack_v", "norm_quantize_pack", "bracketed",
         "reduce", "update", "reduce_v", "select_bits_device", "sign_pack", "sign_reduce", "sign_majority"]


@pytest.mark.parametrize("call", CALLS)
def test_an_earlier_error_is_not_this_calls(dq, hip, call):
    M, b, plan = 3, 4, dq.Plan([4096, 2000, 96])
    gen = torch.Generator(device="cuda").manual_seed(3)
    grads = torch.randn((M, plan.padded_elems), generator=gen, device="cuda")
    norms = torch.rand((M, plan.n_seg), generator=gen, device="cuda") * 50 + 50
    lo, hi = norms * 0.9, norms * 1.1
    ws = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
    wsb = torch.empty(dq.bracketed_workspace_bytes(plan, M), dtype=torch.uint8, device="cuda")
    table = dq.Widths(plan, [b] * plan.n_seg)
    packed = torch.zeros((M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda")
    out, x = torch.zeros(plan.padded_elems, device="cuda"), torch.zeros(plan.padded_elems, device="cuda")
    run = {
        "norm": lambda: dq.norm(plan, grads, norms, ws),
        "norm_linf": lambda: dq.norm_linf(plan, grads, norms, ws),
        "norm_bracket": lambda: dq.norm_bracket(norms, 0.1, lo, hi),
        "quantize_pack": lambda: dq.quantize_pack(plan, grads, norms, b, SEED, 1, packed),
        "quantize_pack_v": lambda: dq.quantize_pack_v(plan, table, grads, norms, SEED, 1, packed),
        "norm_quantize_pack": lambda: dq.norm_quantize_pack(plan, grads, b, SEED, 1, norms, packed),
        "bracketed": lambda: dq.norm_quantize_pack_bracketed(plan, grads, lo, hi, b, SEED, 1, norms, packed, wsb),
        "reduce": lambda: dq.unpack_dequant_reduce(plan, packed, norms, b, out),
        "update": lambda: dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.1, x),
        "reduce_v": lambda: dq.unpack_dequant_reduce_v(plan, table, packed, norms, out),
        "select_bits_device": lambda: dq.select_bits_device(plan, table, norms, 1, 10, 1e-3, 0.9, 1, 8, rule="single"),
        "sign_pack": lambda: dq.sign_pack(plan, grads, packed),
        "sign_reduce": lambda: dq.sign_reduce(plan, packed, out),
        "sign_majority": lambda: dq.sign_majority(plan, packed, out),
    }[call]
    torch.cuda.synchronize()
    assert hip.hipSetDevice(1 << 20) != 0 and hip.hipPeekAtLastError() != 0
    run()
    torch.cuda.synchronize()
    assert hip.hipGetLastError() == 0
    table.close()
    plan.close()
