"""The work a user of this library has it do, as cases to be timed.

A case is one iteration of the data-parallel hot path (or one side of it) for all M simulated
workers, through the functions of ``paper_2107_14575_amd``: what ``dqsgd.run`` and ``bench.py`` call
per iteration.  Sizes are those of the package's own workloads (``workloads.py``: the flat
gradients, the ResNet-18- and transformer-shaped ones, the d = 4096 convex run), or generic.

    listed()              the cases that are always timed
    draw(rng)             one more case of the same ranges
    prepare(case, seed)   what the program holds before the iteration: plan, buffers, gradients
    run(state)            one iteration; returns everything it produces
    work(case)            bytes and operations the iteration cannot do without
    tolerance(case)       how far another correct implementation may differ
"""
import math

import numpy as np
import torch

import paper_2107_14575_amd as dq
from paper_2107_14575_amd import workloads as wl

T, ALPHA = 1000, 0.999       # iterations and convergence factor the bit rule is given
STEP = T - 1                 # iteration index: the rule's weight is then 1
ETA = 0.05                   # learning rate of the fused model update
MARGIN = 0.125               # half width of the norm brackets, as in bench.py
LARGEST = 1 << 32            # most gradient values (all workers together) of a case


def listed():
    return [
        # the convex run's iteration (d = 4096, 8 workers): norms to the host, rule, messages, update;
        # launches and latency are all there is
        dict(name="host_rule_4096_m8", mode="host_rule", layout="flat", elems=4096, values="normal",
             workers=8, b=8, update=True),
        # the small flat gradient of the package's first configuration
        dict(name="host_rule_2p20_m4", mode="host_rule", layout="flat", elems=1 << 20, values="normal",
             workers=4, b=4, update=False),
        # an image classifier's iteration: 62 tensors, 11.2 M values, 8 workers
        dict(name="host_rule_resnet18_m8", mode="host_rule", layout="resnet18", workers=8, b=6, update=True),
        # bench.py's default workload: one flat gradient of 2^28 heavy-tailed values, 16 workers
        dict(name="host_rule_2p28_m16", mode="host_rule", layout="flat", elems=1 << 28, values="student",
             workers=16, b=4, update=False),
        # a text classifier's iteration with one width per tensor decided on the GPU (no host round trip)
        dict(name="device_rule_transformer_m16", mode="device_rule", layout="transformer", workers=16, b=8,
             rule="per_tensor", update=True),
        # the paper's lagged protocol: b known, norms known to +-12.5 %, one read of the gradient
        dict(name="one_pass_resnet18_m8", mode="bracketed", layout="resnet18", workers=8, b=3, update=True),
        # the same without the host: widths from the GPU's rule of the iteration before
        dict(name="one_pass_device_2p26_m16", mode="bracketed_device", layout="flat", elems=1 << 26,
             values="student", workers=16, b=4, rule="single", update=False),
        # a gradient cut into buckets of 512 with one norm each, the practice of the scheme the paper
        # builds on; the length is not a whole number of buckets
        dict(name="buckets_512_m8", mode="buckets", layout="buckets", elems=(1 << 24) + 1234, bucket=512,
             values="normal", workers=8, b=2, update=False),
        # every worker decides its own widths, one per tensor
        dict(name="per_worker_transformer_m16", mode="per_worker", layout="transformer", workers=16, b=8,
             update=False),
        # the one-bit baseline: sign messages and the scaled mean
        dict(name="sign_resnet18_m8", mode="sign", layout="resnet18", workers=8, b=1, vote=False),
        # the ternary scheme (b = 1 with max norms) on many tensors of uneven length, odd worker count
        dict(name="ternary_ragged_m5", mode="fixed_linf", layout="ragged", elems=3000017, tensors=200,
             layout_seed=11, workers=5, b=1, update=False),
        # the server alone: 64 messages of a ragged 4 M model, average and update
        dict(name="server_ragged_m64", mode="server", layout="ragged", elems=4200001, tensors=50,
             layout_seed=5, workers=64, b=5, update=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    mode = rng.choice(["host_rule", "host_rule", "device_rule", "bracketed", "bracketed_device", "buckets",
                       "per_worker", "sign", "fixed_linf", "server"])
    layout = "buckets" if mode == "buckets" else rng.choice(["flat", "flat", "ragged", "ragged", "resnet18", "transformer"])
    workers = _log_uniform(rng, 1, 64)
    case = dict(mode=mode, layout=layout, workers=workers, b=rng.randint(1, 8))
    if layout in ("flat", "ragged", "buckets"):
        # one worker's length: log-uniform over the whole range, hardly ever a multiple of anything
        case["elems"] = _log_uniform(rng, 1 << 12, min(1 << 28, LARGEST // 4 // workers))
        case["values"] = rng.choice(["normal", "student"])
    if layout == "ragged":
        case["tensors"] = _log_uniform(rng, 2, 400)
        case["layout_seed"] = rng.randrange(1 << 20)
    if layout == "buckets":
        case["bucket"] = rng.choice([128, 256, 512, 1024, 2048, 4096])
    if mode in ("device_rule", "bracketed_device"):
        case["rule"] = rng.choice(["single", "per_tensor"])
    if mode == "sign":
        case["vote"] = rng.random() < 0.5
    else:
        case["update"] = rng.random() < 0.5
    return case


def _lengths(case):
    if case["layout"] == "resnet18":
        return wl.resnet18_cifar10_segments()
    if case["layout"] == "transformer":
        return wl.transformer_classifier_segments()
    n = case["elems"]
    if case["layout"] == "flat":
        return [n]
    if case["layout"] == "buckets":
        size = case["bucket"]
        return [size] * (n // size) + ([n % size] if n % size else [])
    # ragged: log-normal shares, every tensor at least one value, the total exact
    share = np.random.default_rng(case["layout_seed"]).lognormal(0.0, 2.0, case["tensors"])
    lens = np.maximum(1, np.floor(share / share.sum() * n)).astype(np.int64)
    lens[int(np.argmax(lens))] += n - int(lens.sum())
    return [int(v) for v in lens]


def _gradients(case, lens, seed):
    M = case["workers"]
    if case["layout"] == "resnet18":
        return wl.resnet18_like(M=M, config=seed, device="cuda", pad_value=0.0)[1]
    if case["layout"] == "transformer":
        return wl.transformer_like(M=M, config=seed, device="cuda", pad_value=0.0)[1]
    make = wl.flat_gaussian if case.get("values") == "normal" else wl.flat_student_t
    starts, padded = wl.seg_starts(lens)
    _, grads = make(D=padded, M=M, config=seed, device="cuda", pad_value=0.0)
    if case["layout"] == "ragged":
        # every tensor has a magnitude of its own, over three decades as in resnet18_like
        sigma = 10.0 ** np.random.default_rng(seed).uniform(-1.5, 1.5, len(lens))
        scale = np.repeat(sigma.astype(np.float32), [wl.padded(n) // wl.GRANULE for n in lens])
        view = grads.view(M, -1, wl.GRANULE)
        view *= torch.from_numpy(scale).cuda()[None, :, None]
    for start, n in zip(starts, lens):
        if n % wl.GRANULE:
            grads[:, start + n:start + wl.padded(n)] = 0.0
    return grads


def prepare(case, seed):
    lens = _lengths(case)
    M, b = case["workers"], case["b"]
    plan = dq.Plan(lens)
    grads = _gradients(case, lens, seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    st = dict(case=case, plan=plan, grads=grads, seed=(seed << 20) ^ wl.QUANT_SEED)
    st["norms"] = torch.empty((M, plan.n_seg), dtype=torch.float32, device="cuda")
    if case["mode"] == "sign" or not case["update"]:
        st["out"] = torch.empty(plan.padded_elems, dtype=torch.float32, device="cuda")
    if case["mode"] == "sign":
        st["packed"] = torch.zeros((M, -(-plan.padded_elems // 128) * 16), dtype=torch.uint8, device="cuda")
        st["scales"] = torch.rand((M, plan.n_seg), generator=gen, device="cuda") * 1e-3 + 1e-4
        return st
    if case["update"]:
        st["x"] = torch.randn(plan.padded_elems, generator=gen, device="cuda") * 0.05
    st["ws"] = torch.empty(plan.workspace_bytes(M), dtype=torch.uint8, device="cuda")
    (dq.norm_linf if case["mode"] == "fixed_linf" else dq.norm)(plan, grads, st["norms"], st["ws"])
    norms = st["norms"].cpu().numpy().astype(np.float64)
    if case["mode"] in ("host_rule", "per_worker"):
        st["norms_host"] = torch.empty((M, plan.n_seg), dtype=torch.float32).pin_memory()
    if case["mode"] in ("bracketed", "bracketed_device"):
        # the norms of the iteration before: within 8 % of this iteration's
        drift = (torch.rand((M, plan.n_seg), generator=gen, device="cuda") - 0.5) * 0.16
        st["prev"] = st["norms"] * (1.0 + drift)
        st["lo"], st["hi"] = torch.empty_like(st["norms"]), torch.empty_like(st["norms"])
        st["wsb"] = torch.empty(dq.bracketed_workspace_bytes(plan, M), dtype=torch.uint8, device="cuda")
    # the error budget: the one with which the largest s* of Eq. (17) is 0.9 (2^b - 1)
    top = np.sqrt((norms ** 2).sum() / M)
    if case.get("rule") == "per_tensor":
        top = np.sqrt((norms ** 2).sum(axis=0) / M).max()
    if case["mode"] == "per_worker":
        top = norms.max()
    st["eps"] = T * (float(top) / (0.9 * (2 ** b - 1))) ** 2
    widths = None
    if case["mode"] in ("device_rule", "bracketed_device"):
        widths = [b] * plan.n_seg
        if case["rule"] == "per_tensor":
            widths = dq.select_bits_per_tensor(norms, STEP, T, st["eps"], ALPHA, 1, 8)[0]
        st["table"] = dq.Widths(plan, widths)
        st["b_dev"] = torch.zeros(plan.n_seg, dtype=torch.int32, device="cuda")
    if case["mode"] == "per_worker":
        widths = dq.select_bits_per_worker(norms, STEP, T, st["eps"], ALPHA, 1, 8, per_tensor=True)
        st["table"] = dq.Widths(plan, widths, workers=M)
    # room for eight bits everywhere where the widths change from iteration to iteration
    room = plan.packed_bytes(8 if widths is not None else b)
    st["packed"] = torch.zeros((M, room), dtype=torch.uint8, device="cuda")
    if case["mode"] == "server":
        dq.quantize_pack(plan, grads, st["norms"], b, st["seed"], STEP, st["packed"])
        st["grads"] = None
    return st


def run(st):
    case, plan, grads, norms, packed = st["case"], st["plan"], st["grads"], st["norms"], st["packed"]
    mode, seed, b = case["mode"], st["seed"], case["b"]
    res = {"packed": packed}
    if mode == "sign":
        dq.sign_pack(plan, grads, packed)
        if case["vote"]:
            dq.sign_majority(plan, packed, st["out"])
        else:
            dq.sign_reduce(plan, packed, st["out"], scales=st["scales"])
        return {"packed": packed, "out": st["out"]}

    # the workers
    table = st.get("table")
    if mode == "host_rule":
        dq.norm(plan, grads, norms, st["ws"])
        st["norms_host"].copy_(norms, non_blocking=True)
        torch.cuda.current_stream().synchronize()
        b, _ = dq.select_bits(st["norms_host"].numpy(), STEP, T, st["eps"], ALPHA, 1, 8)
        res["b"] = b
        packed = res["packed"] = packed[:, :plan.packed_bytes(b)]
        dq.quantize_pack(plan, grads, norms, b, seed, STEP, packed)
    elif mode == "fixed_linf":
        dq.norm_linf(plan, grads, norms, st["ws"])
        dq.quantize_pack(plan, grads, norms, b, seed, STEP, packed)
    elif mode == "device_rule":
        dq.norm(plan, grads, norms, st["ws"])
        dq.select_bits_device(plan, table, norms, STEP, T, st["eps"], ALPHA, 1, 8, rule=case["rule"], b_out=st["b_dev"])
        dq.quantize_pack_v(plan, table, grads, norms, seed, STEP, packed)
        res["b"] = st["b_dev"]
    elif mode == "bracketed":
        dq.norm_bracket(st["prev"], MARGIN, st["lo"], st["hi"])
        dq.norm_quantize_pack_bracketed(plan, grads, st["lo"], st["hi"], b, seed, STEP, norms, packed, st["wsb"])
    elif mode == "bracketed_device":
        dq.norm_bracket(st["prev"], MARGIN, st["lo"], st["hi"])
        dq.norm_quantize_pack_bracketed_v(plan, table, grads, st["lo"], st["hi"], seed, STEP, norms, packed, st["wsb"])
    elif mode == "buckets":
        dq.norm_quantize_pack(plan, grads, b, seed, STEP, norms, packed)
    elif mode == "per_worker":
        dq.norm(plan, grads, norms, st["ws"])
        st["norms_host"].copy_(norms, non_blocking=True)
        torch.cuda.current_stream().synchronize()
        widths = dq.select_bits_per_worker(st["norms_host"].numpy(), STEP, T, st["eps"], ALPHA, 1, 8, per_tensor=True)
        table.set(widths)
        dq.quantize_pack_v(plan, table, grads, norms, seed, STEP, packed)
        res["b"] = widths
    res["norms"] = norms

    # the server
    if table is not None:
        if case["update"]:
            dq.unpack_dequant_reduce_update_v(plan, table, packed, norms, ETA, st["x"])
        else:
            dq.unpack_dequant_reduce_v(plan, table, packed, norms, st["out"])
        if mode == "bracketed_device":  # the widths of the next iteration
            dq.select_bits_device(plan, table, norms, STEP, T, st["eps"], ALPHA, 1, 8, rule=case["rule"], b_out=st["b_dev"])
            res["b"] = st["b_dev"]
    elif case["update"]:
        dq.unpack_dequant_reduce_update(plan, packed, norms, b, ETA, st["x"])
    else:
        dq.unpack_dequant_reduce(plan, packed, norms, b, st["out"])
    if case["update"]:
        res["x"] = st["x"]
    else:
        res["out"] = st["out"]
    if mode == "server":
        del res["packed"], res["norms"]  # inputs there
    return res


def work(case):
    lens = _lengths(case)
    M, mode = case["workers"], case["mode"]
    n, padded = sum(lens), sum(wl.padded(v) for v in lens)
    bits = 1 if mode == "sign" else case["b"] + 1
    if mode == "per_worker" or case.get("rule") == "per_tensor":
        bits = 1 + max(1, case["b"] - 1) if len(lens) > 1 else bits  # most tensors take fewer than the largest
    message = M * padded * bits / 8
    # the workers read the gradients and write the messages, the server reads the messages and writes
    # the average (or reads and writes the model); norms and tables are a few bytes per tensor
    bytes_ = message + (8 if case.get("update") else 4) * padded + 4 * M * len(lens)
    flops = 2 * M * n
    if mode != "server":
        bytes_ += 4 * M * n + message
        flops += (0 if mode == "sign" else 7) * M * n  # square, add; scale, clamp, floor, subtract, compare
    return {"bytes": float(bytes_), "flops": float(flops)}


def tolerance(case):
    # Codes and widths are whole values that follow from norms whose squares are summed in binary64: the
    # same ones.  The average is a binary32 sum over the workers; against the same terms summed in
    # binary64 it was seen to differ by up to 5.7e-8 (2-norm) and 9.6e-7 (largest, at 64 workers), and
    # the norms by 4e-8 (their rounding to binary32): four times that.
    return {"rel": 2.4e-7, "max": 4e-6, "differ": 0.0}
