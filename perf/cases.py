"""Performance cases of the plan executor.

A case is one execution of a compiled orchestration plan of a workload graph,
through the calls that a serving loop makes: the graph is built
(``graphs.build``), its plan compiled and loaded once (``PlanRunner``), its
arguments bound once (``bind``), and every pass is one library call
(``launch_bound``) that launches the plan's kernels.

The listed cases are the workloads of this repository at the sizes of its
benchmark and of its shape sweeps, and at the smaller, larger, ragged and
other-dtype sizes that the same graphs meet in use.  ``draw`` spreads over the
ranges they stand for.
"""

import math

import torch

from paper_2406_09465_amd import graphs
from paper_2406_09465_amd.runner import TORCH_DTYPE, PlanRunner
from synthetic import workloads

# A case: workload, plan ("fused", "layered", or "moments": the two-kernel plan
# of the graph after the split-moments transformation), dtype and the sizes the
# workload's builder takes.


def listed():
    return [
        # the smallest calls, where launches and latency count: one head of
        # self-attention over a short sequence in fp32 (the benchmark's size)
        dict(name="attention_128_f32", workload="attention", plan="fused", dtype="f32", n=128, d=64, nk=128),
        # a longer sequence, past the length one kernel holds: three kernels
        # (scores, softmax, values), in fp16
        dict(name="attention_1024_f16", workload="attention", plan="layered", dtype="f16", n=1024, d=64, nk=1024),
        # a transformer MLP block on few rows (a short prompt, a small batch):
        # the weights are the traffic, the chip is hard to fill
        dict(name="mlp_128_f16", workload="mlp", plan="layered", dtype="f16", m=128, d=768, h=3072),
        # the benchmark's MLP block
        dict(name="mlp_4096_f16", workload="mlp", plan="layered", dtype="f16", m=4096, d=768, h=3072),
        # a batch of eight sequences of 197 tokens (an image in 16 x 16 patches
        # and a class token) through a narrower block in bf16: ragged rows
        dict(name="mlp_1576_bf16", workload="mlp", plan="layered", dtype="bf16", m=1576, d=384, h=1536),
        # the largest: a wide block over a long batch in bf16
        dict(name="mlp_16384_bf16", workload="mlp", plan="layered", dtype="bf16", m=16384, d=1024, h=4096),
        # the same block in single precision, as a model is validated in
        dict(name="mlp_2048_f32", workload="mlp", plan="layered", dtype="f32", m=2048, d=768, h=3072),
        # spatial-reduction attention over a 128 x 128 map (the benchmark's size)
        dict(name="sra_128_f16", workload="sra", plan="fused", dtype="f16", hh=128, ww=128, c=64, r=8),
        # convolution, BatchNorm and Mish early in a detector (the benchmark's
        # size: a large map, few channels) ...
        dict(name="conv_416_f16", workload="conv", plan="fused", dtype="f16", hh=416, ww=416, cin=32, cout=64, k=3),
        # ... and late in it (a small map, many channels), in bf16
        dict(name="conv_52_bf16", workload="conv", plan="fused", dtype="bf16", hh=52, ww=52, cin=128, cout=256, k=3),
        # ReLU linear attention over 4096 tokens (the benchmark's size)
        dict(name="linattn_4096_bf16", workload="linattn", plan="fused", dtype="bf16", heads=16, n=4096, d=16),
        # InstanceNorm, ReLU and padding on a style-transfer image, the largest
        # of the shape sweep
        dict(name="instnorm_448_f16", workload="instnorm", plan="moments", dtype="f16", hh=448, ww=448, c=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _pick(rng, weighted):
    return rng.choices([v for v, _ in weighted], [w for _, w in weighted])[0]


def draw(rng):
    w = rng.choice(("attention", "mlp", "mlp", "sra", "conv", "linattn", "instnorm"))
    if w == "attention":
        dtype = _pick(rng, (("f32", 3), ("f16", 4), ("bf16", 3)))
        n, d = _log(rng, 96, 2048), rng.choice((16, 24, 32, 40, 64, 64, 80, 96, 128))
        nk = n if rng.random() < 0.7 else _log(rng, 96, 2048)
        # one kernel as long as its keys and values fit in LDS
        most = 128 if dtype == "f32" and d <= 64 else 64 if dtype == "f32" else 256 if d <= 64 else 128
        return dict(workload=w, plan="fused" if nk <= most else "layered", dtype=dtype, n=n, d=d, nk=nk)
    if w == "mlp":
        dtype = _pick(rng, (("f32", 2), ("f16", 5), ("bf16", 4)))
        m = _log(rng, 16, 4096 if dtype == "f32" else 16384)
        step = _pick(rng, ((64, 5), (8, 3), (4, 1)))
        d = max(step, _log(rng, 96, 1024) // step * step)
        h = d * 4 if rng.random() < 0.6 else max(step, int(d * rng.uniform(1.5, 4)) // step * step)
        return dict(workload=w, plan="layered", dtype=dtype, m=m, d=d, h=h)
    if w == "sra":
        dtype = _pick(rng, (("f16", 6), ("bf16", 4)))
        r, c = rng.choice((4, 8, 8)), rng.choice((16, 32, 64, 64, 128))
        hh, ww = (r * max(1, _log(rng, 16, 256) // r) for _ in range(2))
        keys = (hh // r) * (ww // r)
        return dict(workload=w, plan="fused" if keys <= (256 if c <= 64 else 128) else "layered", dtype=dtype, hh=hh, ww=ww, c=c, r=r)
    if w == "conv":
        dtype = _pick(rng, (("f32", 1), ("f16", 5), ("bf16", 4)))
        while True:
            hh = _log(rng, 13, 416)
            ww = hh if rng.random() < 0.6 else _log(rng, 13, 416)
            cin = rng.choice((8, 16, 24, 32, 48, 64, 96, 128, 256))
            cout = rng.choice((16, 24, 32, 48, 64, 64, 128, 256))
            k = _pick(rng, ((1, 2), (3, 6), (5, 1)))
            if 3e8 < 2.0 * hh * ww * cin * cout * k * k < (4e9 if dtype == "f32" else 4e10):
                break
        return dict(workload=w, plan="fused", dtype=dtype, hh=hh, ww=ww, cin=cin, cout=cout, k=k)
    if w == "linattn":
        dtype = _pick(rng, (("f32", 1), ("f16", 4), ("bf16", 5)))
        return dict(workload=w, plan="fused", dtype=dtype, heads=rng.choice((1, 2, 3, 4, 8, 12, 16, 32)), n=_log(rng, 64, 16384),
                    d=rng.choice((8, 16, 16, 32)))
    dtype = _pick(rng, (("f32", 2), ("f16", 5), ("bf16", 3)))
    hh = _log(rng, 13, 640)
    ww = hh if rng.random() < 0.6 else _log(rng, 13, 640)
    return dict(workload=w, plan="moments", dtype=dtype, hh=hh, ww=ww, c=rng.choice((8, 16, 24, 32, 32, 64, 128)))


def _sizes(case):
    return {k: v for k, v in case.items() if k not in ("name", "workload", "plan", "dtype")}


def _inputs(case, seed):
    """The workload's inputs on the GPU, drawn from its own distributions."""
    out = {}
    for i, (name, _, shape, dtype, dist, a, b) in enumerate(workloads.specs(case["workload"], dtype=case["dtype"], **_sizes(case))):
        gen = torch.Generator(device="cuda").manual_seed(1000 * seed + i)
        if dist == "normal":
            x = torch.randn(shape, generator=gen, device="cuda") * b + a
        else:
            x = torch.rand(shape, generator=gen, device="cuda") * (b - a) + a
        out[name] = x.to(TORCH_DTYPE[dtype])
    return out


def prepare(case, seed):
    w = graphs.build(case["workload"], dtype=case["dtype"], **_sizes(case))
    kernels = None
    if case["plan"] == "moments":
        w, _ = graphs.rewritten(w)
        kernels = graphs.moments_plan(w)
    r = PlanRunner(w, case["plan"], kernels=kernels)
    x = _inputs(case, seed)
    r.ins = [x[n] for n in w.input_names]
    return r.bind()


def run(state):
    state.launch_bound()
    return state.outs


def work(case):
    """Bytes: every graph input read once, every graph output written once.
    Flops: the products (none: what the reductions and the normalization do)."""
    s, w = _sizes(case), case["workload"]
    e = 4 if case["dtype"] == "f32" else 2
    if w == "attention":
        n, d, nk = s["n"], s["d"], s["nk"]
        return dict(bytes=e * (2 * n * d + 2 * nk * d), flops=4 * n * nk * d)
    if w == "mlp":
        m, d, h = s["m"], s["d"], s["h"]
        return dict(bytes=e * (2 * m * d + 2 * d * h + 2 * d), flops=4 * m * d * h)
    if w == "sra":
        px, c, r = s["hh"] * s["ww"], s["c"], s["r"]
        keys = px // (r * r)
        return dict(bytes=e * (2 * px * c + r * r * c * c + 2 * c), flops=2 * px * c * c + 4 * px * keys * c)
    if w == "conv":
        px = s["hh"] * s["ww"]
        kk = s["k"] ** 2 * s["cin"] * s["cout"]
        return dict(bytes=e * (px * (s["cin"] + s["cout"]) + kk + 2 * s["cout"]), flops=2 * px * kk)
    if w == "linattn":
        t = s["heads"] * s["n"] * s["d"]
        return dict(bytes=e * 4 * t, flops=4 * t * s["d"] + 4 * t)
    px, c = s["hh"] * s["ww"], s["c"]
    return dict(bytes=e * c * (px + (s["hh"] + 2) * (s["ww"] + 2) + 2), flops=9 * px * c)


# Largest relative error (2-norm) and largest difference (over the result's root
# mean square, or over the value itself where that is larger) that another
# correct order of sums and rounding shows: about four times the error of the
# plans against 64 bits over these ranges, which is the rounding of the tensors
# that a plan materializes.  Attention rounds its scores and probabilities.
_TOLERANCE = {"f32": (2e-6, 1.5e-5), "f16": (1.1e-3, 4.5e-3), "bf16": (9e-3, 3.6e-2)}
_ATTENTION_TOLERANCE = {"f32": (2e-6, 1.5e-5), "f16": (2.4e-3, 1.8e-2), "bf16": (1.6e-2, 1.5e-1)}


def tolerance(case):
    rel, most = (_ATTENTION_TOLERANCE if case["workload"] in ("attention", "sra") else _TOLERANCE)[case["dtype"]]
    return {"rel": rel, "max": most}


def _layernorm(x, gamma, beta):
    d = x - x.mean(-1, keepdim=True)
    return d / torch.sqrt((d * d).mean(-1, keepdim=True) + 1e-5) * gamma + beta


def _softmax_attention(q, k, v):
    s = (q @ k.t().contiguous()) / math.sqrt(q.shape[-1])
    e = torch.exp(s - s.max(-1, keepdim=True).values)
    return (e / e.sum(-1, keepdim=True)) @ v


def exact(case, seed):
    x = {k: v.double() for k, v in _inputs(case, seed).items()}
    s, w = _sizes(case), case["workload"]
    if w == "attention":
        return [_softmax_attention(x["Q"], x["K"], x["V"])]
    if w == "mlp":
        h = _layernorm(x["X"], x["gamma"], x["beta"]) @ x["W1"]
        g = 0.5 * h * (1 + torch.tanh(math.sqrt(2 / math.pi) * (h + 0.044715 * h ** 3)))
        return [g @ x["W2"] + x["X"]]
    if w == "sra":
        hh, ww, c, r = s["hh"], s["ww"], s["c"], s["r"]
        a = x["X"].reshape(hh // r, r, ww // r, r, c).permute(0, 2, 1, 3, 4).reshape(-1, r * r * c)
        kv = _layernorm(a @ x["Wsr"], x["gamma"], x["beta"])
        return [_softmax_attention(x["X"].reshape(hh * ww, c), kv, kv)]
    if w == "conv":
        hh, ww, k = s["hh"], s["ww"], s["k"]
        p = torch.nn.functional.pad(x["X"], (0, 0, k // 2, k // 2, k // 2, k // 2))
        y = torch.zeros(hh * ww, s["cout"], dtype=torch.float64, device=p.device)
        for i in range(k):
            for j in range(k):
                y += p[i:i + hh, j:j + ww].reshape(hh * ww, -1) @ x["W"][i, j]
        b = y * x["scale"] + x["shift"]
        return [(b * torch.tanh(torch.logaddexp(b, torch.zeros_like(b)))).reshape(hh, ww, -1)]
    if w == "linattn":
        q, k = x["Q"].relu(), x["K"].relu()
        out = [qh @ (kh.t().contiguous() @ vh) / ((qh @ kh.sum(0)[:, None]) + 1e-6) for qh, kh, vh in zip(q, k, x["V"])]
        return [torch.stack(out)]
    d = x["X"] - x["X"].mean((0, 1))
    y = d / torch.sqrt((d * d).mean((0, 1)) + 1e-5) * x["gamma"] + x["beta"]
    return [torch.nn.functional.pad(y.relu(), (0, 0, 1, 1, 1, 1))]
