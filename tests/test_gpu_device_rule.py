"""The bit rules evaluated on the GPU (dq_select_bits_device) against the host entry points and the
oracle: device and host agree bit for bit; against the oracle the widths and G-bar are equal up to
1024 tensors and valid to the rounding of the sum of squares beyond (the oracle adds in plain index
order); a widths table the per-tensor kernels can use."""
import numpy as np
import pytest
import torch

from paper_2107_14575_amd import workloads as wl
from tests.pyref import rule_factor, single_width_rule_agrees
from tests.test_gpu_parity import SEED, dq, gpu_norm  # noqa: F401  (dq is a fixture)

pytestmark = pytest.mark.gpu


def _device_rule(dq, plan, table, norms_dev, t, T, eps, alpha, b_min, b_max, rule):
    n_seg = plan.n_seg
    b_out = torch.full((n_seg,), -7, dtype=torch.int32, device="cuda")
    g_out = torch.full((n_seg if rule == "per_tensor" else 1,), float("nan"), dtype=torch.float64, device="cuda")
    bytes_out = torch.zeros(1, dtype=torch.int64, device="cuda")
    dq.select_bits_device(plan, table, norms_dev, t, T, eps, alpha, b_min, b_max, rule=rule, b_out=b_out,
                          gbar_out=g_out, packed_bytes_out=bytes_out)
    torch.cuda.synchronize()
    return b_out.cpu().numpy(), g_out.cpu().numpy(), int(bytes_out.item())


@pytest.mark.parametrize("n_seg", [1, 7, 62, 257, 700, 1025, 5000])
def test_same_widths_as_the_host_rules_and_the_oracle(dq, oracle, n_seg):
    rng = np.random.default_rng(80 + n_seg)
    seg_len = [int(x) for x in rng.choice([0, 1, 64, 128, 129, 300, 1000], size=n_seg)]
    if sum(seg_len) == 0:
        seg_len[0] = 5
    plan = dq.Plan(seg_len)
    table = dq.Widths(plan)
    for trial in range(12):
        M = int(rng.choice([1, 2, 8, 16, 64]))
        norms = (10 ** rng.uniform(-5, 0.5, size=(M, n_seg))).astype(np.float32)
        norms[:, np.array(seg_len) == 0] = 0
        if trial % 3 == 0:
            norms[:, rng.integers(0, n_seg)] = 0
        norms_dev = torch.from_numpy(norms).cuda()
        T = int(rng.integers(1, 300))
        t = int(rng.integers(0, T))
        alpha = float(rng.uniform(0.8, 1.0))
        b_min = int(rng.integers(1, 4))
        b_max = int(rng.integers(b_min, 9))
        gbar_l2 = np.sqrt((norms.astype(np.float64) ** 2).sum() / M)
        eps = max(T * alpha ** (T - 1 - t) * (gbar_l2 / float(rng.uniform(1, 200))) ** 2, 1e-30)
        for rule, host, orc in (("single", dq.select_bits, oracle.select_bits),
                                ("single_linf", dq.select_bits_linf, oracle.select_bits_linf)):
            b_dev, g_dev, nbytes = _device_rule(dq, plan, table, norms_dev, t, T, eps, alpha, b_min, b_max, rule)
            b_host, g_host = host(norms, t, T, eps, alpha, b_min, b_max)
            want = orc(norms, t, T, eps, alpha, b_min, b_max)
            if n_seg <= 1024 or rule == "single_linf":
                assert (b_host, g_host) == want
            else:
                # beyond 1024 tensors the library adds a worker's squares in blocks, the oracle in plain
                # index order (Lemma 1): G-bar to the rounding of the sum, b unless s* is on a level count
                assert single_width_rule_agrees((b_host, g_host), want, n_seg, rule_factor(t, T, eps, alpha),
                                                b_min, b_max)
            assert np.all(b_dev == b_host) and g_dev[0] == g_host
            assert nbytes == plan.packed_bytes(b_host)
        b_dev, n_dev, nbytes = _device_rule(dq, plan, table, norms_dev, t, T, eps, alpha, b_min, b_max, "per_tensor")
        b_host, n_host = dq.select_bits_per_tensor(norms, t, T, eps, alpha, b_min, b_max)
        b_or, n_or = oracle.select_bits_per_tensor(norms, t, T, eps, alpha, b_min, b_max)
        assert np.array_equal(b_host, b_or) and np.array_equal(n_host, n_or)
        assert np.array_equal(b_dev, b_host) and np.array_equal(n_dev, n_host)
        assert nbytes == dq.packed_bytes_v(plan, b_host)
        assert table.packed_bytes == dq.packed_bytes_v(plan, [b_max] * n_seg)
    table.close()
    plan.close()


@pytest.mark.parametrize("M", [1, 7, 17, 64])
@pytest.mark.parametrize("n_seg", [63, 65, 256, 1024])
def test_one_launch_rule_at_the_edges_of_its_stages(dq, oracle, n_seg, M):
    """64 tensors are staged at a time, workers are read sixteen at a time, 256 and 1024 tensors are the most that
    the two sizes of the launch take: widths, means (binary64, the same additions in the same order) and message sizes are equal."""
    rng = np.random.default_rng(1000 * n_seg + M)
    seg_len = [int(x) for x in rng.choice([0, 1, 129, 1000], size=n_seg, p=[0.05, 0.35, 0.3, 0.3])]
    norms = (10 ** rng.uniform(-3, 0.5, size=(M, n_seg))).astype(np.float32)
    plan = dq.Plan(seg_len)
    table = dq.Widths(plan)
    norms_dev = torch.from_numpy(norms).cuda()
    T, t, alpha, eps = 100, 60, 0.99, 3e-2
    for rule, host in (("single", oracle.select_bits), ("single_linf", oracle.select_bits_linf),
                       ("per_tensor", oracle.select_bits_per_tensor)):
        b_dev, g_dev, nbytes = _device_rule(dq, plan, table, norms_dev, t, T, eps, alpha, 1, 8, rule)
        want_b, want_g = host(norms, t, T, eps, alpha, 1, 8)
        assert np.all(b_dev == want_b) and np.all(g_dev == want_g)
        assert nbytes == dq.packed_bytes_v(plan, np.broadcast_to(np.asarray(want_b, dtype=np.int32), n_seg))
    table.close()
    plan.close()


@pytest.mark.parametrize("M", [1, 8, 9, 33, 64])
@pytest.mark.parametrize("n_seg", [1, 2, 11, 12, 13])
def test_few_tensors_without_staging(dq, oracle, n_seg, M):
    """Up to twelve tensors a lane reads its worker's norms itself; the workers' sums are added eight at a time.  The largest
    norm belongs to the last tensor of the last worker, and one norm is zero."""
    rng = np.random.default_rng(100 * n_seg + M)
    seg_len = [int(x) for x in rng.choice([1, 129, 1000], size=n_seg)]
    norms = (10 ** rng.uniform(-3, 0.5, size=(M, n_seg))).astype(np.float32)
    norms[0, 0] = 0.0
    norms[-1, -1] = 7.5
    plan = dq.Plan(seg_len)
    table = dq.Widths(plan)
    norms_dev = torch.from_numpy(norms).cuda()
    T, t, alpha, eps = 100, 60, 0.99, 3e-2
    for rule, host in (("single", oracle.select_bits), ("single_linf", oracle.select_bits_linf)):
        b_dev, g_dev, nbytes = _device_rule(dq, plan, table, norms_dev, t, T, eps, alpha, 1, 8, rule)
        want_b, want_g = host(norms, t, T, eps, alpha, 1, 8)
        assert np.all(b_dev == want_b) and np.all(g_dev == want_g)
        assert nbytes == dq.packed_bytes_v(plan, np.broadcast_to(np.asarray(want_b, dtype=np.int32), n_seg))
    table.close()
    plan.close()


@pytest.mark.parametrize("rule", ["single", "per_tensor"])
def test_table_filled_on_the_device_drives_the_kernels(dq, oracle, rule):
    """norm -> rule on the device -> quantize+pack -> reduce, no host step in between; the
    messages are the oracle's for the widths the oracle's rule gives"""
    rng = np.random.default_rng(90)
    seg_len = [int(x) for x in rng.choice([0, 1, 64, 128, 129, 300, 5000], size=300)]
    starts, dp = wl.seg_starts(seg_len)
    M = 4
    gen = torch.Generator().manual_seed(91)
    g = torch.zeros((M, dp), dtype=torch.float32)
    for st, n in zip(starts, seg_len):
        g[:, st:st + n] = torch.randn((M, n), generator=gen) * float(10 ** rng.uniform(-4, -1))
    plan = dq.Plan(seg_len)
    table = dq.Widths(plan)
    g_dev = g.cuda()
    norms_dev = torch.empty((M, plan.n_seg), dtype=torch.float32, device="cuda")
    ws = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
    b_out = torch.zeros(plan.n_seg, dtype=torch.int32, device="cuda")
    T, t, alpha, eps = 50, 30, 0.95, 2e-4
    dq.norm(plan, g_dev, norms_dev, ws)
    dq.select_bits_device(plan, table, norms_dev, t, T, eps, alpha, 1, 8, rule=rule, b_out=b_out)
    packed = torch.full((M, table.packed_bytes), 0xA5, dtype=torch.uint8, device="cuda")
    out = torch.full((dp,), float("nan"), dtype=torch.float32, device="cuda")
    dq.quantize_pack_v(plan, table, g_dev, norms_dev, SEED, t, packed)
    dq.unpack_dequant_reduce_v(plan, table, packed, norms_dev, out)
    torch.cuda.synchronize()
    norms = norms_dev.cpu().numpy()
    if rule == "single":
        widths = np.full(plan.n_seg, oracle.select_bits(norms, t, T, eps, alpha, 1, 8)[0], dtype=np.int32)
    else:
        widths = oracle.select_bits_per_tensor(norms, t, T, eps, alpha, 1, 8)[0]
        assert len(set(widths.tolist())) >= 3
    assert np.array_equal(b_out.cpu().numpy(), widths)
    want = oracle.quantize_pack_v(seg_len, g.numpy(), norms, widths, SEED, t)
    got = packed.cpu().numpy()
    assert np.array_equal(got[:, :want.shape[1]], want)
    assert np.all(got[:, want.shape[1]:] == 0xA5)
    want_out = oracle.unpack_dequant_reduce_v(seg_len, want, norms, widths)
    err = np.abs(out.cpu().numpy().astype(np.float64) - want_out)
    assert err.max() <= 1e-6 * np.abs(want_out).max()
    table.close()
    plan.close()


def test_argument_checks(dq):
    plan = dq.Plan([100, 200])
    other = dq.Plan([100, 200])
    table = dq.Widths(plan)
    norms = torch.ones((2, 2), dtype=torch.float32, device="cuda")
    good = dict(t=0, T=5, eps_hat_q=0.1, alpha=0.9, b_min=1, b_max=8)
    for bad in (dict(t=5), dict(eps_hat_q=0.0), dict(alpha=1.5), dict(b_min=0), dict(b_max=9), dict(b_min=5, b_max=4)):
        args = dict(good)
        args.update(bad)
        with pytest.raises(dq.DQError):
            dq.select_bits_device(plan, table, norms, **args)
    with pytest.raises(dq.DQError):
        dq.select_bits_device(other, table, norms, **good)
    dq.select_bits_device(plan, table, norms, **good)
    torch.cuda.synchronize()
    table.close()
    other.close()
    plan.close()


def _least_squares(seg_len, M, T, seed):
    starts, dp = wl.seg_starts(seg_len)
    gen = torch.Generator().manual_seed(seed)
    target = torch.zeros(dp)
    noise_scale = torch.zeros(dp)
    for k, (st, n) in enumerate(zip(starts, seg_len)):
        scale = (1.0, 0.01, 0.1)[k % 3]
        target[st:st + n] = torch.randn(n, generator=gen) * scale
        noise_scale[st:st + n] = 0.05 * scale
    noise = (torch.randn((T, M, dp), generator=gen) * noise_scale).cuda()
    target = target.cuda()

    def grad_fn(t, x, grads):
        grads.copy_((x - target).unsqueeze(0) + noise[t])

    return dp, target, grad_fn


@pytest.mark.parametrize("lagged", [False, True])
@pytest.mark.parametrize("mode", ["single", "single_linf", "per_tensor"])
def test_loop_without_host_round_trips_equals_the_host_rule_loop(dq, oracle, mode, lagged):
    """Algorithm 1 with the rule on the device against the same loop with the rule on the host
    (itself checked against the oracle loop elsewhere): identical widths, cost and model, bit for
    bit; and every b_t against the oracle's rule on the iteration's norms."""
    from paper_2107_14575_amd import dqsgd
    seg_len = [700, 300, 77, 0, 1500]
    M, T, eta, alpha, tau, eps_hat = 4, 30, 0.2, 0.9, 4, 0.02
    dp, target, grad_fn = _least_squares(seg_len, M, T, 95)
    plan = dq.Plan(seg_len)
    x0 = torch.zeros(dp, dtype=torch.float32, device="cuda")
    kw = dict(b0=2, b_min=1, b_max=8, tau=tau, lagged=lagged, seed=SEED, p="inf" if mode == "single_linf" else 2,
              per_tensor=mode == "per_tensor")
    host = dqsgd.run(plan, x0, grad_fn, M, T, eta, eps_hat, alpha, **kw)
    rule = {"single": oracle.select_bits, "single_linf": oracle.select_bits_linf,
            "per_tensor": oracle.select_bits_per_tensor}[mode]
    checked = []

    def on_step(t, b, grads, norms, packed):
        if not lagged:
            want = rule(norms, t, T, eps_hat, alpha, 1, 8)[0]
            assert np.array_equal(np.asarray(b), np.asarray(want)), t
            checked.append(t)

    dev = dqsgd.run(plan, x0, grad_fn, M, T, eta, eps_hat, alpha, device_rule=True, on_step=on_step, **kw)
    assert len(dev.bits) == T and all(np.array_equal(a, c) for a, c in zip(dev.bits, host.bits))
    assert dev.cost_bits == host.cost_bits
    assert torch.equal(dev.x.view(torch.int32), host.x.view(torch.int32))
    assert np.allclose(dev.gbar, host.gbar, rtol=1e-12, atol=0)
    assert len(np.unique(np.concatenate([np.atleast_1d(b) for b in dev.bits]))) >= 2
    assert lagged or len(checked) == T
    assert float((dev.x - target).norm()) < 0.2 * float(target.norm())
    plan.close()


@pytest.mark.parametrize("mode", ["single", "per_tensor"])
def test_lagged_loop_in_one_pass_per_iteration(dq, oracle, mode):
    """The lagged loop with the rule on the device and norm_margin: from the second iteration on norms and
    messages come from dq_norm_quantize_pack_bracketed_v with the widths table the rule left on the GPU --
    no host round trip, one read of the gradients.  Every iteration's messages equal the oracle's for that
    iteration's norms and widths; the widths and the model follow the two-pass loop."""
    from paper_2107_14575_amd import dqsgd
    seg_len = [9000, 300, 0, 5000, 77]            # two tensors span chunks (bracketed), two lie inside one
    M, T, eta, alpha, tau, eps_hat = 4, 24, 0.2, 0.9, 4, 0.02
    dp, target, grad_fn = _least_squares(seg_len, M, T, 96)
    plan = dq.Plan(seg_len)
    x0 = torch.zeros(dp, dtype=torch.float32, device="cuda")
    kw = dict(b0=2, b_min=1, b_max=8, tau=tau, lagged=True, seed=SEED, per_tensor=mode == "per_tensor", device_rule=True)
    two_pass = dqsgd.run(plan, x0, grad_fn, M, T, eta, eps_hat, alpha, **kw)
    seen = []

    def on_step(t, b, grads, norms, packed):
        g_host = np.ascontiguousarray(grads.cpu().numpy())
        want_n = oracle.norm(seg_len, g_host)
        assert np.all(np.abs(norms.astype(np.float64) - want_n.astype(np.float64)) <= np.spacing(want_n)), t
        b_seg = np.asarray(b, dtype=np.int32) if mode == "per_tensor" else np.full(len(seg_len), b, dtype=np.int32)
        want = oracle.quantize_pack_v(seg_len, g_host, norms, b_seg, SEED, t)
        assert np.array_equal(packed.cpu().numpy(), want), f"messages differ at t={t}"
        seen.append(t)

    one_pass = dqsgd.run(plan, x0, grad_fn, M, T, eta, eps_hat, alpha, on_step=on_step, norm_margin=0.5, **kw)
    assert seen == list(range(T))
    assert all(np.array_equal(a, c) for a, c in zip(one_pass.bits, two_pass.bits))
    assert one_pass.cost_bits == two_pass.cost_bits
    assert float((one_pass.x - two_pass.x).abs().max()) <= 1e-5 * float(two_pass.x.abs().max())
    plan.close()
