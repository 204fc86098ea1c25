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
