"""Performance cases of the skeleton library, through its public entry points.

Every case is one execution request (or one training step) as a program that
keeps its plan and its bound device buffers makes it: `prepare` compiles the
plan and binds the buffers, `run` is one pass.  Sizes are those of the paper's
benchmarks and of this repository's benchmark (`bench.py`, `synth.py`) plus
ragged ones of the same ranges; `draw` spreads over the ranges.

Kinds
  image   a chain of image stages over one RGBA uint8 image, with or without
          the histogram/sum reduce side (Pipeline, MapReduce)
  batch   many uneven image requests in one persistent launch
  while   a while Loop over an image MapReduce, stop condition on the device
  nbody   a counted Loop over force + kick-drift
  vector  a chain of saxpy / reversal stages over fp32, with or without a sum
  fft     batched 65536-point complex FFT chains
  gray    Segmentation chains over a gray volume
  mlp     the cost model: one training step (gradient + Adam), or a forward
          pass over candidate configurations
"""
import math
import random

import numpy as np
import torch

import paper_1510_06585_amd as sk

DEV = "cuda"
FFT_N = 65536
NSBM = "noise,solarise,blur5,mirror"


def listed():
    return [
        # the smallest image of the paper's Table 5: one launch, latency
        {"name": "filter_256x512", "kind": "image", "H": 256, "W": 512, "chain": "noise,solarise,mirror",
         "reduce": "none"},
        # a photograph-sized ragged image (Table 5's 1800 x 1125, odd by one) through the fused MapReduce
        {"name": "mapreduce_1125x1799", "kind": "image", "H": 1125, "W": 1799, "chain": NSBM, "reduce": "hist_sum"},
        # the benchmark's headline: fused Pipeline + MapReduce on the paper's largest image
        {"name": "mapreduce_8192", "kind": "image", "H": 8192, "W": 8192, "chain": NSBM, "reduce": "hist_sum"},
        # an unnamed composition (two stencils, value stages around them, sum reduce), as the
        # configuration selector meets them: kernels that no benchmark names
        {"name": "composition_2847x4289", "kind": "image", "H": 2847, "W": 4289,
         "chain": "solarise,blur5,noise,mirror,blur5,solarise", "reduce": "sum"},
        # the serving form: 256 uneven requests of 256 to 4096 pixels a side in one launch
        {"name": "batch_256", "kind": "batch", "nreq": 256, "lo": 256, "hi": 4096, "sizes": 4},
        # an iterated MapReduce, stopped by the device's condition on its sum
        {"name": "while_2048", "kind": "while", "H": 2048, "W": 2048, "chain": "blur5", "limit": 10},
        # the paper's smallest and largest body counts
        {"name": "nbody_8192x20", "kind": "nbody", "N": 8192, "iters": 20},
        {"name": "nbody_65536x20", "kind": "nbody", "N": 65536, "iters": 20},
        # the paper's largest saxpy, as a two-stage MapReduce
        {"name": "saxpy_sum_5e7", "kind": "vector", "n": 50000000, "chain": "saxpy,saxpy", "reduce": "sum"},
        # the paper's FFT pipelined with its inverse, 256 MB
        {"name": "fft_ifft_512", "kind": "fft", "B": 512, "chain": "fft,ifft"},
        # the paper's largest volume, three stages
        {"name": "segment_240x512x512", "kind": "gray", "D": 240, "H": 512, "W": 512, "stages": 3},
        # the cost model's mini-batch training step
        {"name": "mlp_train_256", "kind": "mlp", "n": 256, "what": "train"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["image", "image", "batch", "while", "nbody", "vector", "fft", "gray", "mlp"])
    if kind == "image":
        ops = ["noise", "solarise", "mirror", "blur5"]
        chain = rng.choice([NSBM, "noise,solarise,mirror",
                            ",".join(rng.choice(ops) for _ in range(rng.randint(1, 6)))])
        return {"kind": kind, "H": _log_int(rng, 64, 8192), "W": _log_int(rng, 64, 8192), "chain": chain,
                "reduce": rng.choice(["none", "hist_sum", "sum"])}
    if kind == "batch":
        return {"kind": kind, "nreq": _log_int(rng, 4, 256), "lo": 256, "hi": _log_int(rng, 512, 4096),
                "sizes": rng.randrange(1 << 20)}
    if kind == "while":
        return {"kind": kind, "H": _log_int(rng, 128, 4096), "W": _log_int(rng, 128, 4096),
                "chain": rng.choice(["blur5", "blur5,mirror"]), "limit": rng.randint(2, 16)}
    if kind == "nbody":
        return {"kind": kind, "N": _log_int(rng, 500, 65536), "iters": rng.randint(1, 20)}
    if kind == "vector":
        return {"kind": kind, "n": _log_int(rng, 1000, 50000000),
                "chain": rng.choice(["saxpy", "saxpy,saxpy", "saxpy,mirror,saxpy", "mirror,saxpy"]),
                "reduce": rng.choice(["none", "sum"])}
    if kind == "fft":
        return {"kind": kind, "B": _log_int(rng, 1, 512), "chain": rng.choice(["fft", "ifft", "fft,ifft"])}
    if kind == "gray":
        return {"kind": kind, "D": _log_int(rng, 16, 240), "H": _log_int(rng, 64, 512), "W": _log_int(rng, 64, 512),
                "stages": rng.randint(1, 4)}
    what = rng.choice(["train", "forward"])
    return {"kind": kind, "n": _log_int(rng, 16, 512 if what == "train" else 16384), "what": what}


# ------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _image(g, H, W):
    return torch.randint(0, 256, (H, W, 4), dtype=torch.uint8, device=DEV, generator=g)


def _uniform(g, *shape, lo=-1.0, hi=1.0):
    return torch.rand(*shape, device=DEV, generator=g) * (hi - lo) + lo


def _image_stages(case):
    return [(op, {"seed": 0x1510 + 77 * k}) if op == "noise" else (op, {}) for k, op in
            enumerate(case["chain"].split(","))]


def _sides(case):
    r = random.Random(case["sizes"])
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** r.random())) for _ in range(case["nreq"])]


def _coeffs(case):
    return [(-1.0) ** k * (0.75 + 0.5 * k) for k in range(len(case["chain"].split(",")))]


def _bodies(case, seed):
    """Cube of bodies, masses U[0.5, 1.5] (`synth.nbody`); G = 1 / N, so that the total G m is
    about 1 and the positions stay smooth over any number of passes."""
    g = _gen(seed)
    N = case["N"]
    pos = torch.cat([_uniform(g, N, 3), _uniform(g, N, 1, lo=0.5, hi=1.5)], dim=1).contiguous()
    return pos, torch.zeros(N, 4, device=DEV)


def _nbody_prm(case):
    return {"eps": 1e-2, "G": float(np.float32(1.0 / case["N"])), "dt": 1e-3}


def _vector_args(case, seed):
    g = _gen(seed)
    nside = case["chain"].split(",").count("saxpy")
    return [_uniform(g, case["n"]) for _ in range(1 + nside)]


def _fft_in(case, seed):
    return _uniform(_gen(seed), case["B"], FFT_N, 2)


def _thresholds(case):
    return [(85, 170), (64, 192), (100, 129), (0, 200)][:case["stages"]]


def _mlp_in(case, seed):
    """Standardised features, log-runtime targets and He-uniform parameters (`synth.mlp_init`)."""
    g = _gen(seed)
    X = torch.randn(case["n"], 24, device=DEV, generator=g)
    t = 4.0 + X[:, 0] - 0.5 * X[:, 3] * X[:, 7] + 0.3 * X[:, 11].abs()
    parts = []
    for out, fan in ((64, 24), (64, 64), (1, 64)):
        lim = math.sqrt(6.0 / fan)
        parts += [_uniform(g, out * fan, lo=-lim, hi=lim), torch.zeros(out, device=DEV)]
    return X, t.contiguous(), torch.cat(parts).contiguous()


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    kind = case["kind"]
    if kind == "image":
        x = _image(_gen(seed), case["H"], case["W"])
        args = [x, torch.empty_like(x)]
        red = None if case["reduce"] == "none" else case["reduce"]
        if red == "hist_sum":
            args.append(torch.zeros(4, 256, dtype=torch.int32, device=DEV))
        if red:
            args.append(torch.zeros(4, dtype=torch.int64, device=DEV))
        return {"kind": kind, "plan": sk.Plan(sk.image_chain(_image_stages(case), red), args), "bound": sk.bind(args),
                "out": args[1:]}
    if kind == "batch":
        # the program serves from one input and one output arena; every request is a 256-byte aligned piece
        sides = _sides(case)
        offs, total = [], 0
        for s in sides:
            offs.append(total)
            total += (4 * s * s + 255) // 256 * 256
        pool_in = torch.randint(0, 256, (total,), dtype=torch.uint8, device=DEV, generator=_gen(seed))
        pool_out = torch.zeros(total, dtype=torch.uint8, device=DEV)
        hist = torch.zeros(len(sides), 4, 256, dtype=torch.int32, device=DEV)
        sums = torch.zeros(len(sides), 4, dtype=torch.int64, device=DEV)
        reqs = [[pool_in[o:o + 4 * s * s].view(s, s, 4), pool_out[o:o + 4 * s * s].view(s, s, 4), hist[r], sums[r]]
                for r, (o, s) in enumerate(zip(offs, sides))]
        root = sk.image_chain([(op, {"seed": 0x1510}) if op == "noise" else (op, {}) for op in NSBM.split(",")],
                              "hist_sum")
        return {"kind": kind, "plan": sk.Plan(root, reqs[0]), "bound": sk.bind_batch(reqs),
                "out": [pool_out, hist, sums]}
    if kind == "while":
        x = _image(_gen(seed), case["H"], case["W"])
        args = [x, torch.empty_like(x), torch.zeros(4, 256, dtype=torch.int32, device=DEV),
                torch.zeros(4, dtype=torch.int64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)]
        body = sk.image_chain(_image_stages(case), "hist_sum")
        # each blur's floor lowers a channel's mean by about half a level from 127.5: five or six iterations
        root = sk.LoopWhile(body, case["limit"], 1, ">", 125 * case["H"] * case["W"])
        return {"kind": kind, "plan": sk.Plan(root, args), "bound": sk.bind(args), "out": args[1:]}
    if kind == "nbody":
        pos, vel = _bodies(case, seed)
        args = [pos, vel, torch.empty_like(pos)]
        return {"kind": kind, "plan": sk.Plan(sk.nbody_loop(case["iters"], **_nbody_prm(case)), args),
                "bound": sk.bind(args), "out": args[:2]}
    if kind == "vector":
        args = _vector_args(case, seed)
        args.append(torch.empty_like(args[0]))
        red = None if case["reduce"] == "none" else case["reduce"]
        if red:
            args.append(torch.zeros(1, device=DEV))
        stages = [(op, {"a": a}) for op, a in zip(case["chain"].split(","), _coeffs(case))]
        return {"kind": kind, "plan": sk.Plan(sk.image_chain(stages, red), args), "bound": sk.bind(args),
                "out": args[-2:] if red else args[-1:]}
    if kind == "fft":
        x = _fft_in(case, seed)
        args = [x, torch.empty_like(x)]
        return {"kind": kind, "plan": sk.Plan(sk.image_chain([(op, {}) for op in case["chain"].split(",")]), args),
                "bound": sk.bind(args), "out": args[1:]}
    if kind == "gray":
        x = torch.randint(0, 256, (case["D"], case["H"], case["W"]), dtype=torch.uint8, device=DEV,
                          generator=_gen(seed))
        args = [x, torch.empty_like(x)]
        root = sk.image_chain([("segment", {"lo": lo, "hi": hi}) for lo, hi in _thresholds(case)])
        return {"kind": kind, "plan": sk.Plan(root, args), "bound": sk.bind(args), "out": args[1:]}
    X, t, params = _mlp_in(case, seed)
    st = {"kind": kind, "what": case["what"], "X": X, "t": t, "params": params, "step": 0}
    if case["what"] == "train":
        st.update(m=torch.zeros_like(params), v=torch.zeros_like(params), grad=torch.empty_like(params),
                  loss=torch.zeros(1, device=DEV))
    else:
        st["y"] = torch.empty(case["n"], device=DEV)
    return st


def run(state):
    if state["kind"] == "batch":
        state["plan"].batch_run(state["bound"])
        return state["out"]
    if state["kind"] == "mlp":
        if state["what"] == "forward":
            sk.mlp_forward(state["params"], state["X"], state["y"])
            return [state["y"]]
        state["step"] += 1
        sk.mlp_grad(state["params"], state["X"], state["t"], state["grad"], state["loss"])
        sk.mlp_adam(state["params"], state["grad"], state["m"], state["v"], state["step"])
        return [state["loss"], state["grad"], state["params"], state["m"], state["v"]]
    state["plan"].run(state["bound"])
    return state["out"]


# --------------------------------------------------------------------- work
def work(case):
    """Inputs read once, outputs written once; flops only where arithmetic is the path's own (a pair
    interaction counts 20, an FFT 5 N log2 N, an MLP sample 2 per weight and pass)."""
    kind = case["kind"]
    red = {"none": 0, "sum": 32, "hist_sum": 4128}
    if kind == "image":
        return {"bytes": 8 * case["H"] * case["W"] + red[case["reduce"]], "flops": 0}
    if kind == "batch":
        return {"bytes": sum(8 * s * s + 4128 for s in _sides(case)), "flops": 0}
    if kind == "while":   # the first iteration's read and the last one's write
        return {"bytes": 8 * case["H"] * case["W"] + 4132, "flops": 0}
    if kind == "nbody":
        return {"bytes": 64 * case["N"], "flops": 20.0 * case["N"] ** 2 * case["iters"]}
    if kind == "vector":
        nops = case["chain"].split(",").count("saxpy")
        return {"bytes": 4 * (2 + nops) * case["n"], "flops": 2 * nops * case["n"]}
    if kind == "fft":
        k = len(case["chain"].split(","))
        return {"bytes": 16 * FFT_N * case["B"], "flops": 5.0 * FFT_N * 16 * k * case["B"]}
    if kind == "gray":
        return {"bytes": 2 * case["D"] * case["H"] * case["W"], "flops": 0}
    w = 24 * 64 + 64 * 64 + 64
    if case["what"] == "forward":
        return {"bytes": 4 * (25 * case["n"] + 5825), "flops": 2 * w * case["n"]}
    return {"bytes": 4 * (25 * case["n"] + 7 * 5825), "flops": 6 * w * case["n"]}


# -------------------------------------------------------------------- exact
def _nbody_exact(case, seed):
    pos, vel = (t.double() for t in _bodies(case, seed))
    prm = {k: float(np.float32(v)) for k, v in _nbody_prm(case).items()}
    r, m, v = pos[:, :3].clone(), pos[:, 3].clone(), vel[:, :3].clone()
    rows = max(1, (1 << 26) // case["N"])
    for _ in range(case["iters"]):
        acc = torch.empty_like(v)
        for i in range(0, case["N"], rows):
            d = [r[None, :, k] - r[i:i + rows, None, k] for k in range(3)]
            s = (d[0] * d[0]).addcmul_(d[1], d[1]).addcmul_(d[2], d[2]).add_(prm["eps"] ** 2)
            s = s.pow_(-1.5).mul_(m[None, :])
            for k in range(3):
                acc[i:i + rows, k] = (s * d[k]).sum(1)
        v += prm["dt"] * prm["G"] * acc
        r += prm["dt"] * v
    pad = torch.zeros(case["N"], 1, dtype=torch.float64, device=DEV)
    return [torch.cat([r, m[:, None]], 1), torch.cat([v, pad], 1)]


def _vector_exact(case, seed):
    args = [a.double() for a in _vector_args(case, seed)]
    x, side = args[0], iter(args[1:])
    for op, a in zip(case["chain"].split(","), _coeffs(case)):
        x = x.flip(0) if op == "mirror" else float(np.float32(a)) * x + next(side)
    return [x] if case["reduce"] == "none" else [x, x.sum().reshape(1)]


def _fft_exact(case, seed):
    z = torch.view_as_complex(_fft_in(case, seed).cpu().double())
    for op in case["chain"].split(","):
        z = torch.fft.fft(z) if op == "fft" else torch.fft.ifft(z)
    return [torch.view_as_real(z)]


def _mlp_exact(case, seed):
    X, t, p = (v.double() for v in _mlp_in(case, seed))
    n = case["n"]
    W1, b1, W2, b2, W3, b3 = p.split([1536, 64, 4096, 64, 64, 1])
    W1, W2 = W1.view(64, 24), W2.view(64, 64)
    h1 = (X @ W1.T + b1).clamp_min(0)
    h2 = (h1 @ W2.T + b2).clamp_min(0)
    y = h2 @ W3 + b3
    if case["what"] == "forward":
        return [y]
    dy = 2.0 / n * (y - t)
    d2 = dy[:, None] * W3 * (h2 > 0)
    d1 = (d2 @ W2) * (h1 > 0)
    grad = torch.cat([(d1.T @ X).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0), dy @ h2,
                      dy.sum().reshape(1)])
    lr, be1, be2, eps = (float(np.float32(v)) for v in (1e-3, 0.9, 0.999, 1e-8))
    m, v = (1 - be1) * grad, (1 - be2) * grad ** 2
    new = p - lr * (m / (1 - be1)) / ((v / (1 - be2)).sqrt() + eps)
    return [((y - t) ** 2).mean().reshape(1), grad, new, m, v]


def exact(case, seed):
    """Floating outputs in 64 bits; whole-number outputs (images, volumes, counts) have one right answer
    and are compared for equality."""
    f = {"nbody": _nbody_exact, "vector": _vector_exact, "fft": _fft_exact, "mlp": _mlp_exact}.get(case["kind"])
    return f(case, seed) if f else None
