"""Levels where the rounding of a - u decides: values on a whole number, on an element's own random number and one
binary32 step to either side of whole + random, subnormal products, products above s, and NaN or infinite neighbours.
The norm that the caller passes is s, so that an element's a is its value.  Against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SEED, STEP = 0x1234567890ABCDEF, 7


@pytest.fixture(scope="module")
def dq():
    import paper_2107_14575_amd as dq
    dq.load_library()
    return dq


def _random(oracle, dp, M):
    """u of every element: (word >> 8) * 2^-24, exact in binary32."""
    key = np.array([SEED & 0xFFFFFFFF, SEED >> 32], dtype=np.uint32)
    u = np.empty((M, dp), dtype=np.float32)
    for w in range(M):
        for q in range(dp // 4):
            r = oracle.philox4x32_10(np.array([q, 0, w, STEP], dtype=np.uint32), key)
            u[w, 4 * q:4 * q + 4] = (np.asarray(r, dtype=np.uint32) >> 8).astype(np.float32) * np.float32(2.0 ** -24)
    return u


# one chunk of one tensor and a tail; tensors of two granules (the form for layouts of small tensors); both kinds of chunk
LAYOUTS = [[4096 + 640], [256] * 19, [4096, 77, 500, 1, 129]]


@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
def test_levels_at_the_edges_of_the_rounding(dq, oracle, layout):
    seg_len, M = LAYOUTS[layout], 2
    plan = dq.Plan(seg_len)
    dp = plan.padded_elems
    u = _random(oracle, dp, M)
    rng = np.random.default_rng(layout)
    inf = np.float32(np.inf)
    for b in range(1, 9):
        s = np.float32((1 << b) - 1)
        whole = rng.integers(0, int(s) + 1, size=(M, dp)).astype(np.float32)
        on = (whole + u).astype(np.float32)
        kinds = [whole, on, np.nextafter(on, inf), np.nextafter(on, np.float32(0)), u, np.nextafter(u, inf),
                 np.nextafter(u, np.float32(0)), np.nextafter(whole, inf), np.nextafter(whole, np.float32(0)),
                 np.full_like(u, 2.0 ** -24), np.full_like(u, 1e-45), np.full_like(u, 2.0 ** -130), np.zeros_like(u)]
        for above in (False, True):  # above: some products beyond s, and the forms that clamp
            g = np.choose(rng.integers(0, len(kinds), size=(M, dp)), kinds).astype(np.float32)
            g = np.minimum(g, s)
            if above:
                g[:, 5::97] = s * np.float32(3.5)
                g[:, 11::89] = np.nextafter(s, inf)
            g *= rng.choice(np.array([-1, 1], dtype=np.float32), size=(M, dp))
            odd = np.zeros((M, dp), dtype=bool)
            if above:  # their own codes are not specified; their neighbours' are
                odd[:, 3::101] = True
                g[odd] = rng.choice(np.array([np.nan, np.inf, -np.inf], dtype=np.float32), size=int(odd.sum()))
            norms = np.full((M, len(seg_len)), s, dtype=np.float32)
            gd, nd = torch.from_numpy(g).cuda(), torch.from_numpy(norms).cuda()
            want = oracle.quantize_pack(seg_len, g, norms, b, SEED, STEP)
            for table in (None, dq.Widths(plan, [b] * len(seg_len))):
                packed = torch.zeros((M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda")
                if table is None:
                    dq.quantize_pack(plan, gd, nd, b, SEED, STEP, packed)
                else:
                    dq.quantize_pack_v(plan, table, gd, nd, SEED, STEP, packed)
                got = packed.cpu().numpy()
                for w in range(M):
                    for a, z in zip(oracle.unpack(got[w], dp, b), oracle.unpack(want[w], dp, b)):
                        a, z = np.asarray(a), np.asarray(z)
                        assert np.array_equal(a[~odd[w]], z[~odd[w]]), (b, above, table is None, w)
    plan.close()


def _edge_values(oracle, plan, seg_len, M, b, share, rng):
    """Values whose a (for a norm of s = 2^b - 1) is an edge of the rounding for `share` of them and uniform elsewhere.
    Every tensor's first value is s, so that s is its max norm; pads are NaN.  Some products of the others pass s for a
    norm one step below."""
    dp, s, inf = plan.padded_elems, np.float32((1 << b) - 1), np.float32(np.inf)
    u = _random(oracle, dp, M)
    whole = rng.integers(0, int(s) + 1, size=(M, dp)).astype(np.float32)
    on = (whole + u).astype(np.float32)
    kinds = [whole, on, np.nextafter(on, inf), np.nextafter(on, np.float32(0)), u, np.nextafter(u, np.float32(0)),
             np.nextafter(whole, np.float32(0)), np.full_like(u, 1e-45), np.zeros_like(u), np.full_like(u, s)]
    edges = np.choose(rng.integers(0, len(kinds), size=(M, dp)), kinds)
    g = np.where(rng.random((M, dp)) < share, edges, rng.random((M, dp)) * s).astype(np.float32)
    g = np.minimum(g, s) * rng.choice(np.array([-1, 1], dtype=np.float32), size=(M, dp))
    pad = np.ones(dp, dtype=bool)
    start = 0
    for n in seg_len:
        if n:
            g[:, start] = s
        pad[start:start + n] = False
        start += -(-n // 128) * 128
    g[:, pad] = np.nan
    return g, s


# tensors of two granules; a chunk of one tensor, then tensors that share one: all inside their chunks
LOCAL = [[256] * 19, [4096, 77, 0, 500, 1, 129, 3000]]


@pytest.mark.parametrize("layout", range(len(LOCAL)))
def test_kernels_that_compute_the_norms_themselves(dq, oracle, layout):
    seg_len, M = LOCAL[layout], 2
    plan = dq.Plan(seg_len)
    rng = np.random.default_rng(10 + layout)
    want_norm = np.array([0 if n == 0 else 1 for n in seg_len], dtype=np.float32)
    for b in range(1, 9):
        g, s = _edge_values(oracle, plan, seg_len, M, b, 0.9, rng)
        gd = torch.from_numpy(g).cuda()
        want = oracle.quantize_pack(seg_len, g, np.tile(want_norm * s, (M, 1)), b, SEED, STEP)
        for table in (None, dq.Widths(plan, [b] * len(seg_len))):
            norms = torch.full((M, len(seg_len)), float("nan"), device="cuda")
            packed = torch.zeros((M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda")
            if table is None:
                dq.norm_quantize_pack(plan, gd, b, SEED, STEP, norms, packed, linf=True)
            else:
                dq.norm_quantize_pack_v(plan, table, gd, SEED, STEP, norms, packed, linf=True)
            assert np.array_equal(norms.cpu().numpy(), np.tile(want_norm * s, (M, 1)))
            assert np.array_equal(packed.cpu().numpy(), want), (b, table is None)
    plan.close()


# chunks inside a tensor that goes on beyond them, its tail with others, and a chunk of several
CROSSING = [[2 * 4096 + 640], [300, 2 * 4096, 500, 129, 5000]]


@pytest.mark.parametrize("share", [0.9, 0.008])
@pytest.mark.parametrize("layout", range(len(CROSSING)))
def test_both_looks_of_the_bracketed_kernels(dq, oracle, layout, share):
    """Brackets of one step to either side of the norm, so that the elements left open are those on an edge: more than a
    chunk can record (quantized again), or about thirty a chunk (recorded and settled); and a bracket that is the norm."""
    seg_len, M = CROSSING[layout], 2
    plan = dq.Plan(seg_len)
    rng = np.random.default_rng(20 + layout)
    ws = torch.empty(dq.bracketed_workspace_bytes(plan, M), dtype=torch.uint8, device="cuda")
    for b in range(1, 9):
        g, s = _edge_values(oracle, plan, seg_len, M, b, share, rng)
        gd = torch.from_numpy(g).cuda()
        norm = np.full((M, len(seg_len)), s, dtype=np.float32)
        want = oracle.quantize_pack(seg_len, g, norm, b, SEED, STEP)
        for exact in (False, True):
            lo = norm if exact else np.nextafter(norm, np.float32(0))
            hi = norm if exact else np.nextafter(norm, np.float32(np.inf))
            lo, hi = torch.from_numpy(lo.copy()).cuda(), torch.from_numpy(hi.copy()).cuda()
            for table in (None, dq.Widths(plan, [b] * len(seg_len))):
                norms = torch.full((M, len(seg_len)), float("nan"), device="cuda")
                packed = torch.zeros((M, plan.packed_bytes(b)), dtype=torch.uint8, device="cuda")
                stats = torch.zeros(2, dtype=torch.int64, device="cuda")
                if table is None:
                    dq.norm_quantize_pack_bracketed(plan, gd, lo, hi, b, SEED, STEP, norms, packed, ws, stats=stats, linf=True)
                else:
                    dq.norm_quantize_pack_bracketed_v(plan, table, gd, lo, hi, SEED, STEP, norms, packed, ws, stats=stats,
                                                      linf=True)
                assert np.array_equal(norms.cpu().numpy(), norm)
                assert np.array_equal(packed.cpu().numpy(), want), (b, exact, table is None)
                settled, redone = (int(v) for v in stats.cpu())
                if exact:
                    assert settled == 0 and redone == 0
                else:
                    assert (redone > 0) if share > 0.5 else (settled > 0 and redone == 0)
    plan.close()
