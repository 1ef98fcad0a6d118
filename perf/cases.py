"""Performance cases: the calls a program makes through the package's public entry points.

One case is a dict of plain values.  `kind` names the entry point:

  gemm      tgemm.gemm, float32 operands, plain F32 or split-bf16x3
  scaled    tgemm.gemm_scaled on operands that are already quantised per 128 x 128 tile
  linear    tgemm.quantize_tiles on the activations, then tgemm.gemm_scaled with kept weights
  quantize  tgemm.quantize_tiles alone
  grouped   tgemm.gemm_batched over many uneven problems, replayed from a HIP graph
  conv      tgemm.conv2d, the implicit-gemm convolution
  gemm2     tgemm.gemm2, two chained layers with the intermediate kept on chip
  contract  tgemm.contract, a batched contraction over labelled modes
  mlp       tgemm.mlp_train_step (forward, backward, Adam) or tgemm.mlp_forward

Matrices are U[-1, 1], as the paper's synthetic sgemm inputs; the low-precision forms take N(0, 1)
with 1% of the rows multiplied by 1e3; the network takes N(0, 1) features and scaled weights.
"""
import math

import numpy as np
import torch

from paper_1804_10694_amd import tgemm as tg

DEV = "cuda"


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest product: one small call, bound by latency and launches
        {"name": "gemm f32 256", "kind": "gemm", "dtype": "f32", "M": 256, "N": 256, "K": 256,
         "alpha": 1.5, "beta": 0.5},
        # the paper's own sgemm size (1060 x 1060): ordinary, no tile size divides it
        {"name": "gemm f32 1060", "kind": "gemm", "dtype": "f32", "M": 1060, "N": 1060, "K": 1060,
         "alpha": 1.0, "beta": 1.0},
        # odd in every dimension: rows off 16-byte alignment, partial tiles on both edges
        {"name": "gemm f32 4097x3001x2053", "kind": "gemm", "dtype": "f32", "M": 4097, "N": 3001, "K": 2053,
         "alpha": 1.0, "beta": 1.0},
        # the largest plain product of the benchmark
        {"name": "gemm f32 8192", "kind": "gemm", "dtype": "f32", "M": 8192, "N": 8192, "K": 8192,
         "alpha": 1.0, "beta": 1.0},
        # the same product through the bf16 matrix cores
        {"name": "gemm x3 8192", "kind": "gemm", "dtype": "x3", "M": 8192, "N": 8192, "K": 8192,
         "alpha": 1.0, "beta": 1.0},
        # the largest low-precision product: both operands quantised beforehand
        {"name": "scaled fp8 16384", "kind": "scaled", "dtype": "fp8", "M": 16384, "N": 16384, "K": 16384},
        # a layer at inference: new activations are quantised, then meet kept weights
        {"name": "linear bf16 2048x4096x4096", "kind": "linear", "dtype": "bf16", "M": 2048, "N": 4096, "K": 4096},
        # 512 uneven problems with sides from 16 to 2048 in one call, as a serving loop replays it
        {"name": "grouped x3 512", "kind": "grouped", "dtype": "x3", "count": 512, "lo": 16, "hi": 2048,
         "dims_seed": 4},
        # a 3x3 convolution layer of the middle of an image network
        {"name": "conv3x3 x3 32x56x56x256", "kind": "conv", "dtype": "x3", "batch": 32, "H": 56, "W": 56,
         "cin": 256, "cout": 256, "R": 3},
        # two 256-wide layers over the same pixels, fused
        {"name": "gemm2 f32 100352x256x256x256", "kind": "gemm2", "dtype": "f32", "M": 100352, "K": 256,
         "N1": 256, "N2": 256, "relu": True},
        # 64 products of 256^3 whose operands need reordering first
        {"name": "contract f32 64x256x256x256", "kind": "contract", "dtype": "f32", "P": 64, "M": 256, "N": 256,
         "K": 256, "permuted": True},
        # one training step of the cost model's network (forward, backward, Adam) at its batch of 512
        {"name": "mlp train 512", "kind": "mlp", "train": True, "rows": 512, "features": 22, "width": 256,
         "hidden": 3},
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# flops of a drawn product: at most these, so that it costs no more than the largest listed one
_CAP = {"f32": 1.0e12, "x3": 1.0e12, "bf16": 4.0e12, "fp8": 8.0e12}


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "scaled", "linear", "quantize", "grouped", "conv", "gemm2",
                       "contract", "mlp"])
    while True:
        c = {"kind": kind}
        if kind == "gemm":
            c.update(dtype=rng.choice(["f32", "x3"]), M=_log(rng, 64, 8192), N=_log(rng, 64, 8192),
                     K=_log(rng, 64, 8192), alpha=1.0, beta=rng.choice([0.0, 0.5, 1.0]))
        elif kind == "scaled":
            c.update(dtype=rng.choice(["fp8", "bf16"]), M=_log(rng, 256, 16384), N=_log(rng, 256, 16384),
                     K=_log(rng, 256, 16384))
            if rng.random() < 0.6:  # most layers' widths are multiples of 16
                c.update(N=-(-c["N"] // 16) * 16, K=-(-c["K"] // 16) * 16)
        elif kind == "linear":
            c.update(dtype=rng.choice(["fp8", "bf16"]), M=_log(rng, 128, 8192),
                     N=16 * _log(rng, 32, 512), K=16 * _log(rng, 32, 512))
        elif kind == "quantize":
            c.update(dtype=rng.choice(["fp8", "bf16"]), M=_log(rng, 256, 16384), K=_log(rng, 256, 16384))
        elif kind == "grouped":
            c.update(dtype=rng.choice(["f32", "x3"]), count=_log(rng, 16, 512), lo=16,
                     hi=rng.choice([512, 1024, 2048]), dims_seed=rng.randrange(1 << 20))
        elif kind == "conv":
            s = rng.choice([7, 14, 28, 56, 112])
            c.update(dtype=rng.choice(["f32", "x3"]), batch=_log(rng, 4, 32), H=s, W=s,
                     cin=8 * _log(rng, 4, 64), cout=8 * _log(rng, 4, 64), R=rng.choice([1, 3, 3, 3, 5, 7]))
        elif kind == "gemm2":
            c.update(dtype=rng.choice(["f32", "x3"]), M=_log(rng, 1024, 100352), K=_log(rng, 64, 1024),
                     N1=_log(rng, 32, 256), N2=_log(rng, 32, 1024), relu=rng.random() < 0.75)
        elif kind == "contract":
            c.update(dtype=rng.choice(["f32", "x3"]), P=_log(rng, 1, 256), M=_log(rng, 32, 512),
                     N=_log(rng, 32, 512), K=_log(rng, 32, 512), permuted=rng.random() < 0.7)
        else:
            c.update(train=rng.random() < 0.7, rows=_log(rng, 64, 4096), features=_log(rng, 8, 64),
                     width=_log(rng, 64, 512), hidden=rng.choice([2, 3, 4]))
        w = work(c)
        if w["flops"] <= _CAP.get(c.get("dtype", "f32"), 1.0e12) and w["bytes"] <= 2.5e9:
            return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV).mul_(2.0).sub_(1.0)


def _outlier_normal(g, rows, cols):
    x = torch.randn(rows, cols, generator=g, device=DEV)
    hot = torch.randperm(rows, generator=g, device=DEV)[:max(1, round(0.01 * rows))]
    x[hot] *= 1e3
    return x


def _raw(case, seed):
    """The inputs before the library sees them, from the seed alone."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"A": _uniform(g, M, K), "B": _uniform(g, K, N), "C": _uniform(g, M, N)}
    if kind in ("scaled", "linear"):
        return {"A": _outlier_normal(g, case["M"], case["K"]), "B": _outlier_normal(g, case["K"], case["N"])}
    if kind == "quantize":
        return {"X": _outlier_normal(g, case["M"], case["K"])}
    if kind == "grouped":
        # every matrix starts on a 256-byte boundary of one buffer per operand, as an allocator gives them
        def split(sizes):
            starts = np.concatenate([[0], np.cumsum([-(-r * c // 64) * 64 for r, c in sizes])])
            flat = _uniform(g, int(starts[-1]))
            return flat, [flat[s:s + r * c].view(r, c) for s, (r, c) in zip(starts[:-1].tolist(), sizes)]
        dims = _grouped_dims(case)
        _, As = split([(m, k) for m, n, k in dims])
        _, Bs = split([(k, n) for m, n, k in dims])
        flat, Cs = split([(m, n) for m, n, k in dims])
        return {"As": As, "Bs": Bs, "Cs": Cs, "flat": flat}
    if kind == "conv":
        b, H, W, ci, co, R = (case[k] for k in ("batch", "H", "W", "cin", "cout", "R"))
        return {"X": _uniform(g, b, H, W, ci), "Wt": _uniform(g, R, R, ci, co)}
    if kind == "gemm2":
        M, K, N1, N2 = case["M"], case["K"], case["N1"], case["N2"]
        return {"A": _uniform(g, M, K), "B": _uniform(g, K, N1), "D": _uniform(g, N1, N2)}
    if kind == "contract":
        P, M, N, K = case["P"], case["M"], case["N"], case["K"]
        a, b = ((K, P, M), (P, N, K)) if case["permuted"] else ((P, M, K), (P, K, N))
        return {"A": _uniform(g, *a), "B": _uniform(g, *b)}
    dims = _mlp_dims(case)
    parts = []
    for i, o in zip(dims[:-1], dims[1:]):
        parts += [torch.randn(i * o, generator=g, device=DEV) * math.sqrt(2.0 / i),
                  torch.randn(o, generator=g, device=DEV) * 0.1]
    return {"params": torch.cat(parts), "X": torch.randn(case["rows"], dims[0], generator=g, device=DEV),
            "y": torch.randn(case["rows"], generator=g, device=DEV)}


def _grouped_dims(case):
    rng = np.random.default_rng(case["dims_seed"])
    d = np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), size=(case["count"], 3))))
    return [tuple(int(v) for v in r) for r in np.clip(d, case["lo"], case["hi"])]


def _mlp_dims(case):
    return [case["features"]] + [case["width"]] * case["hidden"] + [1]


def _contract_modes(case):
    """Mode labels of A, B and C: 9 is the batch, 0 the rows, 2 the columns, 1 the contracted mode."""
    if case["permuted"]:
        return [1, 9, 0], [9, 2, 1], [9, 0, 2]
    return [9, 0, 1], [9, 1, 2], [9, 0, 2]


def prepare(case, seed):
    s = _raw(case, seed)
    s["case"] = case
    kind, dt = case["kind"], case.get("dtype")
    if kind == "scaled":  # quantised once, then kept
        A, B = s.pop("A"), s.pop("B")
        s["QA"], s["SA"] = tg.quantize_tiles(A, dt)
        s["QB"], s["SB"] = tg.quantize_tiles(B, dt)
        s["C"] = torch.empty(case["M"], case["N"], device=DEV)
    elif kind == "linear":  # the weights are quantised once, then kept
        s["QB"], s["SB"] = tg.quantize_tiles(s.pop("B"), dt)
        s["C"] = torch.empty(case["M"], case["N"], device=DEV)
    elif kind == "grouped":  # plan and graph are made once for the set
        n = len(s["As"])
        args = (s["As"], s["Bs"], s["Cs"], [1.0] * n, [0.5] * n, dt)
        start = s["flat"].clone()
        tg.gemm_batched(*args)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            tg.gemm_batched(*args)
        s["graph"] = graph
        s["flat"].copy_(start)
    elif kind == "conv":
        s["Y"] = torch.empty(case["batch"], case["H"], case["W"], case["cout"], device=DEV)
    elif kind == "gemm2":
        s["E"] = torch.empty(case["M"], case["N2"], device=DEV)
    elif kind == "contract":
        s["C"] = torch.empty(case["P"], case["M"], case["N"], device=DEV)
    elif kind == "mlp":
        p = s["params"]
        s.update(dims=_mlp_dims(case), grads=torch.zeros_like(p), m=torch.zeros_like(p), v=torch.zeros_like(p),
                 loss=torch.zeros(1, device=DEV), step=0, work=tg.mlp_workspace(_mlp_dims(case), case["rows"], DEV),
                 out=torch.empty(case["rows"], device=DEV))
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    c = s["case"]
    kind, dt = c["kind"], c.get("dtype")
    if kind == "gemm":
        return tg.gemm(s["A"], s["B"], s["C"], c["alpha"], c["beta"], dt)
    if kind == "scaled":
        return tg.gemm_scaled(s["QA"], s["SA"], s["QB"], s["SB"], s["C"], 1.0, 0.0, dt)
    if kind == "linear":
        Q, S = tg.quantize_tiles(s["A"], dt)
        return [Q, S, tg.gemm_scaled(Q, S, s["QB"], s["SB"], s["C"], 1.0, 0.0, dt)]
    if kind == "quantize":
        return list(tg.quantize_tiles(s["X"], dt))
    if kind == "grouped":
        s["graph"].replay()
        return s["flat"]
    if kind == "conv":
        tg.conv2d(s["X"], s["Wt"], s["Y"], 1.0, 0.0, dt)
        return s["Y"]
    if kind == "gemm2":
        return tg.gemm2(s["A"], s["B"], s["D"], s["E"], 1.0, 0.0, c["relu"], dt)
    if kind == "contract":
        ma, mb, mc = _contract_modes(c)
        return tg.contract(s["A"], ma, s["B"], mb, s["C"], mc, 1.0, 0.0, dt)
    if not c["train"]:
        return tg.mlp_forward(s["dims"], s["params"], s["X"], s["out"], s["work"])
    s["step"] += 1
    tg.mlp_train_step(s["dims"], s["params"], s["grads"], s["m"], s["v"], s["step"], 1e-3, s["X"], s["y"],
                      s["loss"], s["work"])
    return [s["params"], s["grads"], s["m"], s["v"], s["loss"]]


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 4 * (M * K + K * N + M * N * (2 if case["beta"] else 1)), "flops": 2 * M * N * K}
    if kind in ("scaled", "linear"):
        M, N, K = case["M"], case["N"], case["K"]
        es = 1 if case["dtype"] == "fp8" else 2
        first = (4 + es) * M * K if kind == "linear" else es * M * K
        return {"bytes": first + es * K * N + 4 * M * N, "flops": 2 * M * N * K}
    if kind == "quantize":
        return {"bytes": (4 + (1 if case["dtype"] == "fp8" else 2)) * case["M"] * case["K"],
                "flops": 2 * case["M"] * case["K"]}
    if kind == "grouped":
        dims = _grouped_dims(case)
        return {"bytes": sum(4 * (m * k + k * n + 2 * m * n) for m, n, k in dims),
                "flops": sum(2 * m * n * k for m, n, k in dims)}
    if kind == "conv":
        b, H, W, ci, co, R = (case[k] for k in ("batch", "H", "W", "cin", "cout", "R"))
        return {"bytes": 4 * (b * H * W * (ci + co) + R * R * ci * co), "flops": 2 * b * H * W * R * R * ci * co}
    if kind == "gemm2":
        M, K, N1, N2 = case["M"], case["K"], case["N1"], case["N2"]
        return {"bytes": 4 * (M * K + K * N1 + N1 * N2 + M * N2), "flops": 2 * M * N1 * (K + N2)}
    if kind == "contract":
        P, M, N, K = case["P"], case["M"], case["N"], case["K"]
        return {"bytes": 4 * P * (M * K + K * N + M * N), "flops": 2 * P * M * N * K}
    dims, rows = _mlp_dims(case), case["rows"]
    mats = [i * o for i, o in zip(dims[:-1], dims[1:])]
    params = sum(mats) + sum(dims[1:])
    if not case["train"]:
        return {"bytes": 4 * (params + rows * (dims[0] + 1)), "flops": 2 * rows * sum(mats)}
    return {"bytes": 4 * (7 * params + rows * (dims[0] + 1)), "flops": 2 * rows * (3 * sum(mats) - mats[0])}


# ------------------------------------------------------------------ the same in 64 bits
def _tiles(x, f):
    """f over the 128 x 128 tiles' largest magnitudes of x: (per-tile values, the same spread over x)."""
    r, c = x.shape
    R, Cc = -(-r // 128), -(-c // 128)
    pad = torch.zeros(R * 128, Cc * 128, dtype=x.dtype, device=x.device)
    pad[:r, :c] = x.abs()
    s = f(pad.view(R, 128, Cc, 128).amax(dim=(1, 3)))
    return s, s.repeat_interleave(128, 0)[:r].repeat_interleave(128, 1)[:, :c]


def _quantised(x, dtype):
    """(scales, the values the codes stand for) in 64 bits: power-of-two scales, round to nearest even."""
    def scale(amax):
        m, e = torch.frexp(amax)
        if dtype == "fp8":   # the power of two with amax / s in (224, 448]
            e = torch.where(m <= 0.875, e - 9, e - 8)
        else:                # 2^ceil(log2 amax)
            e = torch.where(m == 0.5, e - 1, e)
        return torch.where(amax > 0, torch.ldexp(torch.ones_like(amax), e), torch.ones_like(amax))
    s, full = _tiles(x, scale)
    q = (x / full).to(torch.float8_e4m3fn if dtype == "fp8" else torch.bfloat16)
    return s.double(), q.double() * full.double()


def exact(case, seed):
    s = _raw(case, seed)
    kind = case["kind"]
    if kind == "gemm":
        return case["alpha"] * (s["A"].double() @ s["B"].double()) + case["beta"] * s["C"].double()
    if kind in ("scaled", "linear"):
        sa, a = _quantised(s.pop("A"), case["dtype"])
        _, b = _quantised(s.pop("B"), case["dtype"])
        return a @ b if kind == "scaled" else [None, sa, a @ b]
    if kind == "quantize":
        return [None, _quantised(s["X"], case["dtype"])[0]]
    if kind == "grouped":
        flat = s["flat"].double()
        at = 0
        for A, B, C in zip(s["As"], s["Bs"], s["Cs"]):
            n = C.numel()
            flat[at:at + n] = (A.double() @ B.double() + 0.5 * C.double()).reshape(-1)
            at += -(-n // 64) * 64
        return flat
    if kind == "conv":
        b, H, W, ci, co, R = (case[k] for k in ("batch", "H", "W", "cin", "cout", "R"))
        h = R // 2
        Y = torch.zeros(b * H * W, co, dtype=torch.float64, device=DEV)
        Xp = torch.nn.functional.pad(s["X"], (0, 0, h, h, h, h))
        for dy in range(R):
            for dx in range(R):
                Y += Xp[:, dy:dy + H, dx:dx + W].double().reshape(-1, ci) @ s["Wt"][dy, dx].double()
        return Y.view(b, H, W, co)
    if kind == "gemm2":
        T = s["A"].double() @ s["B"].double()
        return (torch.relu(T) if case["relu"] else T) @ s["D"].double()
    if kind == "contract":
        A, B = s["A"].double(), s["B"].double()
        if case["permuted"]:
            A, B = A.permute(1, 2, 0), B.permute(0, 2, 1)
        return torch.bmm(A.contiguous(), B.contiguous())
    dims, p = _mlp_dims(case), s["params"].double()
    layers, at = [], 0
    for i, o in zip(dims[:-1], dims[1:]):
        layers.append((p[at:at + i * o].view(i, o), p[at + i * o:at + i * o + o]))
        at += i * o + o
    acts = [s["X"].double()]
    for k, (Wm, bias) in enumerate(layers):
        z = acts[-1] @ Wm + bias
        acts.append(torch.relu(z) if k + 1 < len(layers) else z)
    out = acts[-1].view(-1)
    if not case["train"]:
        return out
    diff = out - s["y"].double()
    d = (2.0 * diff / case["rows"]).view(-1, 1)
    parts = []
    for k in range(len(layers) - 1, -1, -1):
        if k + 1 < len(layers):
            d = d * (acts[k + 1] > 0)
        parts = [(acts[k].T.contiguous() @ d).reshape(-1), d.sum(0)] + parts
        d = d @ layers[k][0].T.contiguous()
    g = torch.cat(parts)
    m, v = 0.1 * g, 0.001 * g * g
    return [p - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8), g, m, v, (diff * diff).mean().view(1)]
