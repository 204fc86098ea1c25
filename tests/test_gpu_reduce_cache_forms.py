"""The reduce with update in its cache forms -- the model left in the last-level cache or passing through, the level loads with the
streaming hint or without -- on both sides of the lines between them, in the forms that such calls take (two workers to a decoded word; one with a
row of widths per worker, and with 33 workers beyond 24 M elements), with a ragged end: the average is that of the reduce without update bit
for bit, the model is x - eta * average, and nothing past the layout's end is touched."""
import pytest
import torch

from paper_2107_14575_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dq():
    import paper_2107_14575_amd as dq
    dq.load_library()
    return dq


ONCE = 24 << 20  # elements


def _check_update(plan, want, gen, update):
    """update(x, ghat) with a step of 0.05 on a model with room behind it."""
    padded = plan.padded_elems
    room = torch.randn(padded + 4096, generator=gen, device="cuda")
    before = room.clone()
    x, got = room[:padded], torch.empty(padded, device="cuda")
    update(x, got)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    assert torch.equal(room[padded:], before[padded:])
    eta = torch.tensor(0.05, dtype=torch.float32).double().item()
    exact = before[:padded].double() - eta * want.double()
    # one rounding to binary32 of the exact value; the binary64 sum above may round the other way at a tie: one unit in the last place
    ulp = torch.nextafter(exact.float().abs(), torch.tensor(float("inf"), device="cuda")) - exact.float().abs()
    assert ((x.double() - exact).abs() <= ulp.double()).all()


@pytest.mark.parametrize("elems,M,b", [(ONCE, 2, 2), (ONCE + 77, 2, 2), (ONCE + 77, 1, 8), (ONCE + 3 * 4096 + 129, 2, 5), (ONCE, 2, 6),
                                       (11_000_077, 5, 6), (11_000_077, 8, 6), (5_200_077, 32, 6), (2_600_077, 32, 7), (5_200_077, 33, 5)])
@pytest.mark.parametrize("table", [False, True])
def test_update_as_average_and_step(dq, elems, M, b, table):
    plan = dq.Plan([elems])
    padded = plan.padded_elems
    gen = torch.Generator(device="cuda").manual_seed(elems % 1000 + b)
    grads = torch.randn((M, padded), generator=gen, device="cuda") * 1e-3
    grads[:, elems:] = 0
    norms = torch.empty((M, 1), device="cuda")
    ws = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
    dq.norm(plan, grads, norms, ws)
    packed = torch.zeros((M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda")
    dq.quantize_pack(plan, grads, norms, b, wl.QUANT_SEED, 1, packed)
    del grads
    want = torch.empty(padded, device="cuda")
    dq.unpack_dequant_reduce(plan, packed, norms, b, want)
    _check_update(plan, want, gen, lambda x, ghat: (
        dq.unpack_dequant_reduce_update_v(plan, dq.Widths(plan, [b]), packed, norms, 0.05, x, ghat=ghat) if table else
        dq.unpack_dequant_reduce_update(plan, packed, norms, b, 0.05, x, ghat=ghat)))
    plan.close()


@pytest.mark.parametrize("elems,M,b", [(ONCE, 1, 6), (ONCE, 2, 6), (ONCE + 77, 2, 6), (ONCE + 77, 1, 8), (ONCE + 3 * 4096 + 129, 3, 5),
                                       (5_200_077, 32, 6), (2_600_077, 32, 7), (5_200_077, 33, 5), (ONCE + 5000, 33, 4)])
@pytest.mark.parametrize("form", ["one tensor per worker", "per worker", "shared"])
def test_update_with_tables(dq, elems, M, b, form):
    """Widths per worker, all alike on one tensor; and mixed, per worker or shared by them, over tensors that share a wavefront with
    others at the layout's start and end.  The average of the same call without update bit for bit."""
    mixed, workers = form != "one tensor per worker", None if form == "shared" else M
    few = [300, 77, 129, 2000]
    seg_len = few + [elems - 2 * sum((n + 127) // 128 * 128 for n in few)] + few if mixed else [elems]
    plan = dq.Plan(seg_len)
    gen = torch.Generator(device="cuda").manual_seed(elems % 1000 + b + M)
    grads = torch.randn((M, plan.padded_elems), generator=gen, device="cuda") * 1e-3
    norms = torch.empty((M, plan.n_seg), device="cuda")
    dq.norm(plan, grads, norms, torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda"))
    rows = [[1 + (b - 1 + mixed * (3 * w + 5 * l)) % 8 for l in range(plan.n_seg)] for w in range(workers or 1)]
    widths = dq.Widths(plan, rows, workers=workers)
    packed = torch.zeros((M, plan.packed_bytes(8)), dtype=torch.uint8, device="cuda")
    dq.quantize_pack_v(plan, widths, grads, norms, wl.QUANT_SEED, 1, packed)
    del grads
    want = torch.empty(plan.padded_elems, device="cuda")
    dq.unpack_dequant_reduce_v(plan, widths, packed, norms, want)
    if not mixed:
        shared = torch.empty_like(want)
        dq.unpack_dequant_reduce(plan, packed, norms, b, shared)
        assert float((shared - want).abs().max()) <= 1e-6 * float(shared.abs().max())
    _check_update(plan, want, gen, lambda x, ghat: dq.unpack_dequant_reduce_update_v(plan, widths, packed, norms, 0.05, x, ghat=ghat))
    plan.close()
