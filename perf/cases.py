"""Performance cases of the GaLore optimizer step: what a training program has this library do.

A case is one of five kinds of call, each through the public Python face (``binding``):

  step       ``galore_step`` / ``galore_step_static`` over one or more LLaMA-shaped layers between two refreshes
             (project, Adam, project back), one call per layer in backward order, as per-layer hooks call it
  refresh    ``galore_refresh_subspace``: the projectors of a layer's matrices from their gradients
  period     ``galore_step`` over a whole update interval: T steps of one layer, one of which carries the refresh
  two_sided  ``GaLoreTwoSided.step`` on one weight (projectors on both sides)
  adafactor  ``GaLoreAdafactor.step`` on one weight

Sizes: the 60M, 130M, 350M, 1B and 7B stacks of ``workloads.CONFIGS``, and for drawn cases any width between them,
aligned or not.  Weights and states are made as a resumed run has them: the projector holds the leading singular
vectors of the gradient's signal, the moments are those of earlier steps.
"""
import math

import torch

from paper_2403_03507_amd import binding as gb
from paper_2403_03507_amd.workloads import layer_shapes

_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
_NEVER = 1 << 30  # an update gap that no pass reaches: the steps between two refreshes
_LR = 1e-3


def _case(name, kind, **kw):
    c = dict(kind=kind, dtype="bf16", layers=1, moments="f32", schedule="chains", iters=4, decay=0.0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # One small fp32 weight updated on its own, as a per-parameter hook does: launches and latency.
        _case("step_weight_512_f32", "step", shape="square", d=512, f=1376, rank=128, dtype="f32"),
        # The 60M configuration: fp32 layer, T = 5: five steps of which one refreshes all seven projectors.
        _case("period_60m_f32", "period", shape="layer", d=512, f=1376, rank=128, dtype="f32", gap=5, iters=6),
        # 130M stack, two layers in one call, three calls' worth of streams and Adam in the projection (bench.py's schedule).
        _case("step_130m_bf16", "step", shape="layer", d=768, f=2048, rank=256, layers=2, per_call=2, schedule="overlap3"),
        # 350M stack, three layers, one call each, in the library's default schedule, with weight decay.
        _case("step_350m_bf16", "step", shape="layer", d=1024, f=2736, rank=256, layers=3, decay=0.01),
        # 1B stack: rows of 5461 elements start at odd offsets.
        _case("step_1b_bf16", "step", shape="layer", d=2048, f=5461, rank=512, layers=2, schedule="overlap3plain"),
        # 7B stack at r = 1024, the headline configuration: three layers in backward order, two calls in flight.
        _case("step_7b_bf16", "step", shape="layer", d=4096, f=11008, rank=1024, layers=3, schedule="overlap2"),
        # The same layer at a small rank: bound by the traffic of G and W, not by the products.
        _case("step_7b_rank128_bf16", "step", shape="layer", d=4096, f=11008, rank=128),
        # 8-bit moments, one 7B layer (8-bit GaLore).
        _case("step_7b_q8", "step", shape="layer", d=4096, f=11008, rank=1024, moments="q8"),
        # Subspace refresh of a 350M layer: short launches, latency.
        _case("refresh_350m_bf16", "refresh", shape="layer", d=1024, f=2736, rank=256),
        # Subspace refresh of a 7B layer at r = 1024: the longest call of the library.
        _case("refresh_7b_bf16", "refresh", shape="layer", d=4096, f=11008, rank=1024),
        # The two-sided rule on one 4096 x 4096 weight.
        _case("two_sided_4096_bf16", "two_sided", shape="square", d=4096, f=11008, rank=1024),
        # GaLore with Adafactor on one 4096 x 11008 weight.
        _case("adafactor_7b_up_bf16", "adafactor", shape="wide", d=4096, f=11008, rank=1024),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _ragged(rng, x):
    """x at one of the alignments that models have: mostly multiples of 64, some of 8, some of nothing."""
    step = rng.choice([64, 64, 8, 1])
    return max(int(round(x / step)) * step, step)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "q8", "refresh", "refresh", "two_sided", "adafactor", "adafactor"])
    shape = rng.choice(["layer", "layer", "square", "wide", "tall"])
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    if kind == "q8":  # blocks of 256 elements along the rows of the moments
        d = 256 * rng.randint(4, 16)
        return _case(None, "step", shape=shape, d=d, f=256 * int(round(d * rng.uniform(2.0, 2.7) / 256)),
                     rank=256 * rng.randint(1, max(1, d // 1024)), moments="q8", schedule=rng.choice(["chains", "overlap2"]))
    d = _ragged(rng, _log_uniform(rng, 256, 2048 if dtype == "f32" else 4096))
    f = _ragged(rng, d * rng.uniform(2.0, 2.7))
    rank = int(_log_uniform(rng, 8, d / 4 if kind == "refresh" else d / 3))
    rank = max(8, rank // 8 * 8) if rng.random() < 0.8 else rank
    if kind == "refresh":
        return _case(None, "refresh", shape=shape, d=d, f=f, rank=rank, dtype=dtype, iters=rng.choice([4, 4, 6]))
    if kind in ("two_sided", "adafactor"):
        return _case(None, kind, shape=shape if shape != "layer" else "square", d=d, f=f, rank=rank, dtype=dtype)
    layers = rng.randint(1, 3)
    schedule = rng.choice(["chains", "overlap2", "overlap3", "overlap3plain", "static"])
    if schedule == "static" and 8 * rank * f + (2 * d * (f + 8) if f % 8 else 0) > 75 << 20:  # beyond the static array
        schedule = "chains"
    return _case(None, "step", shape=shape, d=d, f=f, rank=rank, dtype=dtype, layers=layers,
                 per_call=rng.choice([1, 1, layers]), schedule=schedule, decay=rng.choice([0.0, 0.0, 0.01]))


def _shapes(case):
    d, f = case["d"], case["f"]
    return {"layer": layer_shapes(d, f), "square": [(d, d)], "wide": [(d, f)], "tall": [(f, d)]}[case["shape"]]


# ---- inputs ---------------------------------------------------------------------------------------

def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)


def _orthonormal(gen, rows, cols, spike=0.0):
    """rows x cols, orthonormal columns.  With `spike`, column j leans towards a coordinate of its own (an outlier
    channel), so that its largest entry, which decides its sign, stands clear of the others."""
    a = _randn(gen, rows, cols) / math.sqrt(rows)
    if spike:
        at = torch.randperm(rows, generator=gen, device="cuda")[:cols]
        a[at, torch.arange(cols, device="cuda")] += spike
    for _ in range(2):
        c = torch.linalg.cholesky(a.t() @ a)
        a = torch.linalg.solve_triangular(c, a.t(), upper=False).t().contiguous()
    return a


class _Factors:
    """Singular factors of the gradients of one shape; fresh noise for every gradient."""

    def __init__(self, gen, m, n, rank, gapped):
        k = min(m, n)
        if gapped:
            # `rank` directions, geometric over a factor of 8, well above the noise: the leading subspace and its
            # vectors are determined by the gradient, so two correct refreshes agree on them.
            count = rank
            self.sigma = 10.0 * 8.0 ** (-torch.arange(count, device="cuda", dtype=torch.float32) / max(count - 1, 1))
            self.noise = float(self.sigma[-1]) / 4 / (math.sqrt(m) + math.sqrt(n)) / 1.1
        else:  # power law over a noise floor, as the 350M and 7B configurations have it
            count = min(max(rank, 32), k // 2)
            self.sigma = 1e-2 * math.sqrt(m * n) / torch.arange(1, count + 1, device="cuda", dtype=torch.float32)
            self.noise = 1e-3
        self.u = _orthonormal(gen, m, count, 0.5 if gapped and m <= n else 0.0)
        self.v = _orthonormal(gen, n, count, 0.5 if gapped and m > n else 0.0)
        self.us = self.u * self.sigma
        self.m, self.n, self.rank = m, n, rank

    def grad(self, gen, dtype):
        return torch.addmm(_randn(gen, self.m, self.n), self.us, self.v.t(), beta=self.noise).to(dtype)

    def projector(self, gen):
        side = self.u if self.m <= self.n else self.v
        return side[:, :self.rank] if self.rank <= side.shape[1] else _orthonormal(gen, side.shape[0], self.rank)

    def other(self, gen):
        side = self.v if self.m <= self.n else self.u
        return side[:, :self.rank] if self.rank <= side.shape[1] else _orthonormal(gen, side.shape[0], self.rank)


def _earlier(gen, proj, grad, left):
    """Moments as earlier steps left them: around the projected gradient of one of them."""
    g = grad.float()
    r = proj.t() @ g if left else g @ proj
    m = 0.7 * r + 0.3 * r.square().mean().sqrt() * _randn(gen, *r.shape)
    return m, 1.2 * r.square() + 0.1 * r.square().mean()


def _encode(x, mantissa_base, signed):
    """8-bit codes of a block-wise scaled matrix (the number format of ``galore.h``: blocks of 256, 3 mantissa bits)."""
    blocks = x.view(x.shape[0], -1, 256)
    scale = blocks.abs().amax(2).clamp_min(1e-30)
    y = (blocks.abs() / scale.unsqueeze(2)).clamp(max=1.0)
    e = (torch.floor(torch.log2(y.clamp_min(1e-30))) + mantissa_base).clamp_min(0)
    norm = e > 0
    frac = torch.where(norm, (y * torch.exp2(mantissa_base - e) - 1) * 8, y * 2.0 ** (mantissa_base - 1) * 8)
    code = (e * 8 + frac.round()).clamp(max=mantissa_base * 8).to(torch.int32)
    if signed:
        code = code + 128 * (blocks < 0).to(torch.int32)
    return code.to(torch.uint8).view(x.shape), scale


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)
    dtype, rank, kind = _DTYPE[case["dtype"]], case["rank"], case["kind"]
    shapes = _shapes(case) * case["layers"]
    refreshes = kind in ("refresh", "period")
    factors = {s: _Factors(gen, s[0], s[1], rank, refreshes) for s in dict.fromkeys(shapes)}
    W = [(0.02 * _randn(gen, m, n)).to(dtype) for m, n in shapes]
    steps = case["gap"] if kind == "period" else 1
    G = [[factors[s].grad(gen, dtype) for s in shapes] for _ in range(steps)]

    if kind in ("two_sided", "adafactor"):
        (m, n), fac = shapes[0], factors[shapes[0]]
        opt = (gb.GaLoreTwoSided if kind == "two_sided" else gb.GaLoreAdafactor)(W[0], rank, update_gap=_NEVER, weight_decay=case["decay"])
        opt.t = 1001
        short, long_ = fac.projector(gen), fac.other(gen)
        if kind == "two_sided":
            p, q = (short, long_) if m <= n else (long_, short)
            opt.P.copy_(p)
            opt.Q.copy_(q)
            mom, var = _earlier(gen, q, p.t() @ fac.grad(gen, dtype).float(), False)
            opt.V.copy_(var)
        else:
            opt.proj.copy_(short)
            mom, var = _earlier(gen, short, fac.grad(gen, dtype), m <= n)
            opt.row.copy_(var.sum(1))
            opt.col.copy_(var.sum(0))
            mom = mom / var.sqrt()
        opt.M.copy_(mom)
        return {"kind": kind, "opt": opt, "W": W, "G": G}

    schedule = case["schedule"]
    overlap = {"overlap2": 2, "overlap3": 3, "overlap3plain": 3}.get(schedule, 0)
    opt = gb.GaLore(W, rank, update_gap=case.get("gap", _NEVER), moments=case["moments"], refresh_iters=case["iters"],
                    weight_decay=case["decay"], workspace_factor=max(overlap, 1), seed=7)
    if overlap:
        opt.set_call_overlap(overlap)
        opt.set_fused_adam(schedule != "overlap3plain")
    if kind == "step":  # a run resumed from a checkpoint
        for i, s in enumerate(shapes):
            p = factors[s].projector(gen)
            opt.proj[i].copy_(p)
            mom, var = _earlier(gen, p, factors[s].grad(gen, dtype), s[0] <= s[1])
            if case["moments"] == "q8":
                code, scale = _encode(mom, 15, True)
                opt.M[i].copy_(code)
                opt.M_scale[i].copy_(scale)
                code, scale = _encode(var, 31, False)
                opt.V[i].copy_(code)
                opt.V_scale[i].copy_(scale)
            else:
                opt.M[i].copy_(mom)
                opt.V[i].copy_(var)
            opt.set_step(i, 1001)
    per_layer = len(_shapes(case))
    per_call = per_layer * case.get("per_call", 1)
    calls = [(a, min(a + per_call, len(W))) for a in range(0, len(W), per_call)][::-1]  # backward order
    return {"kind": kind, "opt": opt, "W": W, "G": G, "calls": calls, "static": schedule == "static", "overlap": overlap,
            "arrays": [gb.tensor_array(gb.desc(w) for w in W[a:b]) for a, b in calls]}


def run(state):
    opt, W, kind = state["opt"], state["W"], state["kind"]
    if kind == "two_sided":
        opt.step(W[0], state["G"][0][0], _LR)
        return [W[0], opt.M, opt.V]
    if kind == "adafactor":
        opt.step(W[0], state["G"][0][0], _LR)
        return [W[0], opt.M, opt.row, opt.col]
    if kind == "refresh":
        opt.refresh(state["G"][0])
        return [opt.proj, opt.proj_t]
    step = gb.galore_step_static if state["static"] else gb.galore_step
    for G in state["G"]:
        for (a, b), weights in zip(state["calls"], state["arrays"]):
            step(opt.ctx, weights, [gb.desc(g) for g in G[a:b]], a, b - a, _LR)
        if state["overlap"]:
            opt.join()  # the next forward pass reads the weights
    return [W, opt.M, opt.V] + ([opt.proj] if kind == "period" else []) + ([opt.M_scale, opt.V_scale] if opt.moments == "q8" else [])


# ---- what a pass cannot do without -------------------------------------------------------------------

def work(case):
    s = 2 if case["dtype"] == "bf16" else 4
    r, kind, total_b, total_f = case["rank"], case["kind"], 0.0, 0.0
    for m, n in _shapes(case) * case["layers"]:
        k, l = min(m, n), max(m, n)
        # G read, W read and written, the projector read, the moments read and written
        step_b = 3.0 * m * n * s + k * r * s + r * l * (16 if case["moments"] == "f32" else 4 + 16 / 256)
        step_f = 4.0 * m * n * r
        # Gram matrix (half by symmetry), the rounds and the Ritz product, orthogonalisation, rotation, eigen-solve
        fresh_b = float(m * n * s + 2 * k * r * s)
        fresh_f = 1.0 * k * k * l + (case["iters"] + 1) * 2.0 * k * k * r + (case["iters"] + 2) * 2.0 * k * r * r + 9.0 * r ** 3
        if kind == "step":
            total_b, total_f = total_b + step_b, total_f + step_f
        elif kind == "refresh":
            total_b, total_f = total_b + fresh_b, total_f + fresh_f
        elif kind == "period":
            total_b, total_f = total_b + case["gap"] * step_b + fresh_b, total_f + case["gap"] * step_f + fresh_f
        elif kind == "two_sided":
            total_b += 3.0 * m * n * s + (m + n) * r * s + 16.0 * r * r
            total_f += 4.0 * m * n * r + 4.0 * l * r * r
        else:  # adafactor: one moment and the two statistics
            total_b += 3.0 * m * n * s + k * r * s + 8.0 * r * l + 8.0 * (r + l)
            total_f += step_f
    return {"bytes": total_b, "flops": total_f}


def tolerance(case):
    """Four times what the path differs by from its formulas in 64 bits, rounded to the stored types (2-norms).
    Seen: bf16 steps 1.9e-4 (a weight in two hundred one ulp off), fp32 steps 6e-8 at contractions of 512;
    projectors 1.6e-3 (bf16, r = 1024) and 4.5e-4 (fp32, r = 512), where neighbouring singular values lie under a
    per cent apart; over an update interval the projector's own 9e-5 enters everything."""
    if case["kind"] == "refresh":
        return {"rel": 6.5e-3} if case["dtype"] == "bf16" else {"rel": 2e-3}
    if case["kind"] == "period":
        return {"rel": 1e-3}
    if case["dtype"] == "bf16":
        return {"rel": 8e-4, "differ": 1e-3 if case["moments"] == "q8" else 0.0}
    return {"rel": 2e-6}
