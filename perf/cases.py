"""What a user of this library has it do, as timed cases.

A case is a plain dict.  Three kinds, one for each way a program calls the
library:

* ``layer``: one branch-cached MoE layer (``MoecaLayer``) over a refresh
  cycle of a sampling loop: the cache is reset as for a new batch of images,
  then ``steps`` steps follow (a full step and the cache steps after it),
  each with its own input and attention feature.  In the uncached mode the
  cycle is a single step.
* ``noalloc``: one call of ``moeca_forward_noalloc`` (the uncached layer for
  callers that cannot allocate).
* ``stack``: a run of DiT-MoE blocks (``MoecaStack``) over a refresh cycle,
  with the timestep and class embedding of every step.

``graph`` replays the cycle from one HIP graph captured beforehand, as a
serving loop with fixed buffers does; otherwise every step is launched
eagerly.

Inputs follow the drift model of ``synth.py`` (a per-token rate a_i,
log-uniform), drawn on the GPU.  The rates lie in [1e-3, 2e-2], the lower
part of that model's range: consecutive steps of a 250-step sampler.
"""
from __future__ import annotations

import math

import torch

from paper_2606_15615_amd import _lib
from paper_2606_15615_amd.layer import MoecaLayer
from paper_2606_15615_amd.stack import MoecaStack

MODES = {"full": _lib.MOECA_MODE_FULL, "threshold": _lib.MOECA_MODE_THRESHOLD,
         "ratio": _lib.MOECA_MODE_RATIO}
# share of the branches that a threshold-mode cache step recomputes on these
# inputs with the default settings (for the work estimate only)
THRESHOLD_SHARE = 0.6
DRIFT = (1e-3, 2e-2)
# controller settings: the defaults of the binding
TAU0, ALPHA, BETA = 0.80, 0.6, 0.65
DEV = "cuda:0"


def _layer(name, d, E, k, d_ff, B, N, **kw):
    c = {"name": name, "kind": "layer", "d": d, "E": E, "k": k, "d_ff": d_ff, "B": B, "N": N,
         "dtype": "bf16", "act": "gelu_tanh", "n_shared": 0, "mode": "ratio", "ratio": 0.3,
         "norm_topk": True, "zipf": False, "steps": 4, "graph": False}
    c.update(kw)
    return c


def _stack(name, L, d, heads, E, k, d_ff, B, N, **kw):
    c = {"name": name, "kind": "stack", "L": L, "d": d, "heads": heads, "E": E, "k": k,
         "d_ff": d_ff, "B": B, "N": N, "dtype": "bf16", "act": "gelu_tanh", "n_shared": 0,
         "mode": "ratio", "ratio": 0.3, "norm_topk": True, "zipf": False, "steps": 4,
         "graph": False}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the small fp32 layer, uncached, from code that may not allocate
        _layer("forward_small_fp32", 384, 8, 2, 1536, 1, 256, kind="noalloc", dtype="fp32",
               mode="full", steps=1),
        # the same layer through a refresh cycle of a sampling loop
        _layer("cycle_small_fp32", 384, 8, 2, 1536, 1, 256, dtype="fp32"),
        # one image at a 32 x 32 latent (256 tokens), from a captured graph: latency
        _layer("cycle_256x1_graph", 1152, 16, 2, 4608, 1, 256, graph=True),
        # a batch of eight such images
        _layer("cycle_256x8", 1152, 16, 2, 4608, 8, 256),
        # eight images at a 64 x 64 latent: the benchmarked layer
        _layer("cycle_1024x8", 1152, 16, 2, 4608, 8, 1024),
        # the uncached comparator at that size
        _layer("full_1024x8", 1152, 16, 2, 4608, 8, 1024, mode="full", steps=1),
        # the paper's own threshold rule, a ragged token count and batch, erf GELU and gates
        # without renormalisation
        _layer("cycle_threshold_1000x3", 1152, 16, 2, 4608, 3, 1000, mode="threshold",
               act="gelu_erf", norm_topk=False),
        # the wide layer with a skewed expert load (a Zipf prior on the router)
        _layer("cycle_skewed_4096x2", 3072, 32, 2, 8192, 2, 4096, zipf=True),
        # fine-grained experts: 64 gated experts, top-8, two shared ones
        _layer("cycle_fine_4096x4", 2048, 64, 8, 1408, 4, 4096, act="swiglu", n_shared=2,
               ratio=0.25),
        # fp32 at the XL width, a ragged token count
        _layer("cycle_fp32_333x2", 1152, 16, 2, 4608, 2, 333, dtype="fp32"),
        # DiT-MoE blocks with attention: one image, ragged tokens, from a graph
        _stack("stack_250x1_graph", 4, 1152, 16, 16, 2, 4608, 1, 250, graph=True),
        # and the benchmarked batch
        _stack("stack_1024x8", 2, 1152, 16, 16, 2, 4608, 8, 1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    fam = rng.choice(["xl", "xl", "xl", "wide", "fine", "fp32", "noalloc", "stack", "stack"])
    mode = rng.choice(["ratio", "ratio", "ratio", "threshold", "full"])
    ratio = round(rng.uniform(0.1, 0.6), 3)
    graph = rng.random() < 0.3
    steps = 1 if mode == "full" else rng.choice([2, 3, 4, 4])
    act = rng.choice(["gelu_tanh", "gelu_tanh", "gelu_erf"])
    kw = dict(mode=mode, ratio=ratio, graph=graph, steps=steps, act=act,
              norm_topk=rng.random() < 0.7)
    if fam == "xl":
        d = 64 * rng.randint(9, 20)
        c = _layer("", d, rng.choice([8, 12, 16, 24]), rng.choice([1, 2, 2, 3]),
                   rng.choice([4 * d, 4 * d, 64 * rng.randint(16, 72)]), rng.randint(1, 8),
                   _log_int(rng, 60, 1100), **kw)
    elif fam == "wide":
        c = _layer("", 64 * rng.randint(32, 48), rng.choice([16, 32]), 2,
                   64 * rng.randint(64, 128), rng.randint(1, 2), _log_int(rng, 500, 4096), **kw)
        c["zipf"] = rng.random() < 0.6
    elif fam == "fine":
        kw["act"] = "swiglu"
        c = _layer("", 64 * rng.randint(16, 32), rng.choice([32, 64]), rng.choice([4, 6, 8]),
                   64 * rng.randint(8, 22), rng.randint(1, 4), _log_int(rng, 120, 2048), **kw)
        c["n_shared"] = rng.choice([0, 1, 2])
    elif fam == "fp32":
        d = 64 * rng.randint(5, 18)
        c = _layer("", d, rng.choice([4, 8, 16]), rng.choice([1, 2]), 4 * d, rng.randint(1, 3),
                   _log_int(rng, 60, 600), dtype="fp32", **kw)
    elif fam == "noalloc":
        kw.update(mode="full", steps=1, graph=False)
        d = 64 * rng.randint(5, 18)
        f32 = rng.random() < 0.4
        rows = (40 << 20) // (5 * d * (4 if f32 else 2) * 2)  # top-2 within the library's array
        n = min(rows, _log_int(rng, 40, 1100))
        c = _layer("", d, rng.choice([4, 8, 16]), 2, 4 * d, rng.randint(1, max(1, rows // n)), n,
                   dtype="fp32" if f32 else "bf16", **kw)
        c["B"] = min(c["B"], 8)
        c["kind"] = "noalloc"
    else:
        heads, dh = rng.choice([(8, 72), (16, 64), (16, 72), (12, 64), (8, 96)])
        kw.pop("norm_topk")
        c = _stack("", rng.randint(1, 4), heads * dh, heads, rng.choice([8, 16]), 2,
                   64 * rng.randint(18, 72), rng.randint(1, 8), _log_int(rng, 60, 1024), **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dt(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, *shape, scale=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV) * scale

    def mat(self, case, *shape, scale=None):
        """A weight tensor of the case's type, ~N(0, 1/fan_in), drawn a leading slice at a time."""
        s = 1.0 / math.sqrt(shape[-1]) if scale is None else scale
        if len(shape) < 3:
            return self.normal(*shape, scale=s).to(_dt(case))
        out = torch.empty(shape, device=DEV, dtype=_dt(case))
        for e in range(shape[0]):
            out[e] = self.normal(*shape[1:], scale=s)
        return out

    def trajectory(self, case, dtype):
        B, N, d = case["B"], case["N"], case["d"]
        lo, hi = (math.log(v) for v in DRIFT)
        u = torch.rand(B, N, 1, generator=self.g, device=DEV)
        a = torch.exp(lo + (hi - lo) * u)
        x = self.normal(B, N, d)
        out = [x.to(dtype, copy=True)]
        for _ in range(1, case["steps"]):
            x = torch.sqrt(1.0 - a) * x + torch.sqrt(a) * self.normal(B, N, d)
            out.append(x.to(dtype, copy=True))
        return out


def _layer_inputs(case, seed):
    g, s, up = _Draws(seed), case["n_shared"], case["d_ff"] * (2 if case["act"] == "swiglu" else 1)
    w = {"r": g.mat(case, case["E"], case["d"]),
         "up": g.mat(case, case["E"], up, case["d"]),
         "down": g.mat(case, case["E"], case["d"], case["d_ff"]),
         "b": None, "up_s": None, "down_s": None}
    if case["zipf"]:
        w["b"] = -1.2 * torch.log(torch.arange(1, case["E"] + 1, device=DEV, dtype=torch.float32))
    if s:
        w["up_s"] = g.mat(case, s, up, case["d"])
        w["down_s"] = g.mat(case, s, case["d"], case["d_ff"])
    return w, g.trajectory(case, _dt(case)), g.trajectory(case, _dt(case))


def _stack_inputs(case, seed):
    g, d = _Draws(seed), case["d"]
    blocks = []
    for _ in range(case["L"]):
        blocks.append({
            # AdaLN maps start from zero in training and stay small
            "W_ada": g.mat(case, 6 * d, d, scale=0.25 / math.sqrt(d)),
            "b_ada": g.normal(6 * d, scale=0.02),
            "W_qkv": g.mat(case, 3 * d, d), "b_qkv": g.normal(3 * d, scale=0.02),
            "W_o": g.mat(case, d, d), "b_o": g.normal(d, scale=0.02),
            "W_r": g.mat(case, case["E"], d), "b_r": None,
            "W_up": g.mat(case, case["E"], case["d_ff"], d),
            "W_down": g.mat(case, case["E"], d, case["d_ff"])})
    emb = {"W1": g.mat(case, d, 256), "b1": g.normal(d, scale=0.02), "W2": g.mat(case, d, d),
           "b2": g.normal(d, scale=0.02), "table": g.mat(case, 1000, d, scale=1.0)}
    labels = torch.randint(0, 1000, (case["B"],), generator=g.g, device=DEV, dtype=torch.int32)
    ts = [torch.full((case["B"],), 999.0 * (1.0 - t / 250.0), device=DEV)
          for t in range(case["steps"])]
    return blocks, emb, labels, ts, g.trajectory(case, torch.float32)


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------
class _LayerLoop:
    """A layer handle with its weights, and the buffers of a refresh cycle."""

    def __init__(self, case, seed):
        self.w, self.xs, self.attn = _layer_inputs(case, seed)
        self.cached = case["mode"] != "full"
        self.layer = MoecaLayer(case["d"], case["E"], case["k"], case["d_ff"], batch=case["B"],
                                tokens=case["N"], mode=MODES[case["mode"]], ratio=case["ratio"],
                                tau0=TAU0, alpha=ALPHA, beta=BETA, act=case["act"],
                                dtype=case["dtype"], norm_topk=case["norm_topk"],
                                n_shared=case["n_shared"], device=DEV)
        w = self.w
        self.layer.set_weights(w["r"], w["b"], w["up"], w["down"])
        if case["n_shared"]:
            self.layer.set_shared(w["up_s"], w["down_s"])
        self.ys = [torch.empty_like(x) for x in self.xs]
        self.attn_cache = torch.empty_like(self.xs[0])
        self.out = {"y": self.ys}
        if self.cached:
            B, N, k = case["B"], case["N"], case["k"]
            view = lambda n, t, *s: self.layer.buffer(n).view(t).view(*s)  # noqa: E731
            self.out.update(
                attention=self.attn_cache, rows=view("h_c", _dt(case), B, N, k, case["d"]),
                norms=view("n_c", torch.float32, B, N, k),
                experts=view("e_c", torch.int32, B, N, k),
                statistic=view("stat", torch.float32, B, case["E"], N))

    def cycle(self):
        if not self.cached:
            self.layer.step(self.xs[0], 0, self.ys[0])
            return self.out
        self.layer.reset()
        for t, x in enumerate(self.xs):
            self.layer.bind_attention(self.attn[t], self.attn_cache)
            self.layer.step(x, t, self.ys[t])  # t = 0 is a full step, t = 1, 2, 3 cache steps
        return self.out


class _Forward:
    """A layer handle for the call that allocates nothing."""

    def __init__(self, case, seed):
        self.loop = _LayerLoop(case, seed)
        self.B = case["B"]

    def cycle(self):
        L = self.loop
        _lib.moeca_forward_noalloc(L.layer.h, L.xs[0].data_ptr(), self.B, L.ys[0].data_ptr(),
                                   torch.cuda.current_stream().cuda_stream)
        return L.out


class _StackLoop:
    """A stack handle with its weights, and the buffers of a refresh cycle."""

    def __init__(self, case, seed):
        self.blocks, self.emb, self.labels, self.ts, self.xs = _stack_inputs(case, seed)
        self.cached = case["mode"] != "full"
        self.stack = MoecaStack(case["L"], case["d"], case["heads"], case["E"], case["k"],
                                case["d_ff"], batch=case["B"], tokens=case["N"],
                                mode=MODES[case["mode"]], ratio=case["ratio"], tau0=TAU0,
                                alpha=ALPHA, beta=BETA, act=case["act"], device=DEV)
        for l, b in enumerate(self.blocks):
            self.stack.set_block(l, **b)
        self.c = [torch.empty(case["B"], case["d"], device=DEV) for _ in self.xs]
        self.work = [torch.empty_like(x) for x in self.xs]
        B, N, d = case["B"], case["N"], case["d"]
        self.out = {"x": self.work, "c": self.c,
                    "attention": [self.stack.buffer("a", l).view(torch.bfloat16)[:B * N * d]
                                  .view(B, N, d) for l in range(case["L"])]}

    def cycle(self):
        e = self.emb
        if self.cached:
            self.stack.reset()
        for t, x in enumerate(self.xs):
            self.work[t].copy_(x)  # the blocks update the residual stream in place
            self.stack.embed(self.ts[t], self.labels, e["W1"], e["b1"], e["W2"], e["b2"],
                             e["table"], self.c[t])
            self.stack.step(self.work[t], self.c[t], t)
        return self.out


class _Replay:
    """A cycle captured in a HIP graph."""

    def __init__(self, loop):
        self.loop = loop
        loop.cycle()
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            loop.cycle()

    def cycle(self):
        self.graph.replay()
        return self.loop.out


def prepare(case, seed):
    kind = {"layer": _LayerLoop, "noalloc": _Forward, "stack": _StackLoop}[case["kind"]]
    loop = kind(case, seed)
    return _Replay(loop) if case["graph"] else loop


def run(state):
    return state.cycle()


# ---------------------------------------------------------------------------
# work and tolerance
# ---------------------------------------------------------------------------
def _steps_share(case):
    """Recomputed share of the branches at each step."""
    share = THRESHOLD_SHARE if case["mode"] == "threshold" else case["ratio"]
    return [1.0] + [share] * (case["steps"] - 1)


def work(case):
    d, E, k, f, S = case["d"], case["E"], case["k"], case["d_ff"], case["n_shared"]
    T = case["B"] * case["N"]
    act = 4 if case["dtype"] == "fp32" else 2
    cached = case["kind"] != "noalloc" and case["mode"] != "full"
    mats = 3 if case["act"] == "swiglu" else 2
    nbytes = flops = 0.0
    for share in _steps_share(case):
        rec = share * T * k
        # routed experts that receive a branch, and the shared ones, read once
        experts = min(E, rec) + S
        nbytes += experts * mats * d * f * act + E * d * act
        flops += 2.0 * mats * d * f * (rec + S * T) + 2.0 * T * E * d
        # input and output of every token; cached rows read and written, the refreshed
        # attention features, the statistic and the slots' ids, weights and norms
        nbytes += 2.0 * T * d * act
        if cached:
            sync = T * min(1.0, 1.0 - (1.0 - share) ** k)
            nbytes += (T * k - rec) * d * act + rec * d * act + 2.0 * sync * d * act
            nbytes += 8.0 * T * E + 2.0 * 12.0 * T * k
        if case["kind"] == "stack":
            sync = T * min(1.0, 1.0 - (1.0 - share) ** k)
            L = case["L"]
            nbytes += (6 + 4) * d * d * 2.0 - T * d * act  # AdaLN, q/k/v and output matrices
            flops += (2.0 * 6 * case["B"] * d * d + 2.0 * 2 * T * d * d + 2.0 * 2 * sync * d * d
                      + 4.0 * sync * case["N"] * d)
            nbytes += 2.0 * T * d * 4 / L  # the residual stream in and out of the run
    scale = case["L"] if case["kind"] == "stack" else 1
    return {"bytes": nbytes * scale, "flops": flops * scale}


def tolerance(case):
    """bf16: about four times the distance of a step from its 64-bit value.  A branch whose margin
    ties with the last one taken, to within the rounding of the cached norms, may fall on either
    side: its row then lags by a few steps of drift (about a quarter of its size), hence ``max``
    and the term in one row of T.  fp32 norms do not move a margin."""
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-3}
    if case["mode"] == "full" and case["kind"] != "stack":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 1e-2 + 0.25 / math.sqrt(case["B"] * case["N"]), "max": 0.95}


# ---------------------------------------------------------------------------
# the same steps in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _act64(z, act):
    if act == "swiglu":
        return torch.nn.functional.silu(z[:, 0::2]) * z[:, 1::2]
    return torch.nn.functional.gelu(z, approximate="tanh" if act == "gelu_tanh" else "none")


class _Exact:
    """The branch-cached layer: router, statistic, threshold, match and score, selection, expert
    FFN, combine and cache update."""

    def __init__(self, case, w):
        self.c, self.w = case, w
        self.valid = False
        B, N, E = case["B"], case["N"], case["E"]
        self.C = torch.zeros(B, E, N, device=DEV, dtype=torch.float64)

    def ffn(self, x, up, down):
        return _act64(x @ up.double().T, self.c["act"]) @ down.double().T

    def decide(self, x):
        """Router and decision on x [T, d]: experts, gates, recompute mask, slots."""
        c = self.c
        B, N, k, E = c["B"], c["N"], c["k"], c["E"]
        logits = x @ self.w["r"].double().T
        if self.w["b"] is not None:
            logits = logits + self.w["b"].double()
        e = torch.sort(logits, dim=1, descending=True, stable=True).indices[:, :k].contiguous()
        z = torch.exp(logits - logits.max(dim=1, keepdim=True).values)
        zk = z.gather(1, e)
        wt = zk / (zk if c["norm_topk"] else z).sum(dim=1, keepdim=True)
        full = not self.valid or c["mode"] == "full"
        slot = torch.arange(k, device=DEV).expand(B * N, k).contiguous()
        mask = torch.ones(B * N, k, dtype=torch.bool, device=DEV)
        if c["mode"] != "full":
            ind = torch.zeros(B, N, E, device=DEV, dtype=torch.float64)
            ind.scatter_(2, e.view(B, N, k), 1.0)
            self.C = BETA * self.C + (1.0 - BETA) * ind.transpose(1, 2)
        if full:
            return e, wt, mask, slot, full
        P = self.C / self.C.sum(dim=2, keepdim=True).clamp_min(1e-300)
        H = -torch.special.xlogy(P, P).sum(dim=2) / math.log(N) if N > 1 else P.sum(dim=2) * 0
        tau = TAU0 * (1.0 + ALPHA * (2.0 * H.clamp(0.0, 1.0) - 1.0))
        hit = e[:, :, None] == self.e[:, None, :]
        matched = hit.any(dim=2)
        q = hit.to(torch.int32).argmax(dim=2)
        o = self.n.gather(1, q) / self.n.sum(dim=1, keepdim=True)
        s = wt + (wt - self.g.gather(1, q)).abs() + o
        m = (s.view(B, N, k) - tau.gather(1, e.view(B, N * k)).view(B, N, k)).view(B, N * k)
        mt = matched.view(B, N * k)
        if c["mode"] == "threshold":
            mask = (~mt | (m > 0)).view(-1, k)
        else:
            ratio = torch.tensor(c["ratio"], dtype=torch.float32).item()
            budget = int(math.floor(ratio * N * k + 0.5))
            key = torch.where(mt, m, torch.full_like(m, math.inf))
            order = torch.sort(key, dim=1, descending=True, stable=True).indices
            rank = torch.empty_like(order)
            rank.scatter_(1, order, torch.arange(N * k, device=DEV).expand(B, -1))
            mask = (~mt | (rank < budget)).view(-1, k)
        taken = (torch.nn.functional.one_hot(q, k).bool() & matched[:, :, None]).any(dim=1)
        free = torch.sort(taken.to(torch.int8), dim=1, stable=True).indices
        rank_u = ((~matched).cumsum(dim=1) - 1).clamp_min(0)
        slot = torch.where(matched, q, free.gather(1, rank_u))
        return e, wt, mask, slot, full

    def finish(self, x, e, wt, mask, slot, full):
        """Expert FFN of the masked branches on x [T, d], cache update and combine."""
        c, w = self.c, self.w
        k, d, T = c["k"], c["d"], x.shape[0]
        if full:
            self.rows = torch.zeros(T, k, d, device=DEV, dtype=torch.float64)
            self.e = torch.zeros(T, k, dtype=torch.int64, device=DEV)
            self.g = torch.zeros(T, k, device=DEV, dtype=torch.float64)
            self.n = torch.zeros(T, k, device=DEV, dtype=torch.float64)
        for ex in range(c["E"]):
            t, p = torch.nonzero(mask & (e == ex), as_tuple=True)
            for a in range(0, t.numel(), 16384):
                ta, sa = t[a:a + 16384], slot[t[a:a + 16384], p[a:a + 16384]]
                h = self.ffn(x[ta], w["up"][ex], w["down"][ex])
                self.rows[ta, sa] = h
                self.e[ta, sa] = ex
                self.g[ta, sa] = wt[ta, p[a:a + 16384]]
                self.n[ta, sa] = h.norm(dim=1)
        y = torch.zeros(T, d, device=DEV, dtype=torch.float64)
        for s in range(c["n_shared"]):
            for a in range(0, T, 16384):
                y[a:a + 16384] += self.ffn(x[a:a + 16384], w["up_s"][s], w["down_s"][s])
        for p in range(k):
            y += wt[:, p:p + 1] * self.rows[torch.arange(T, device=DEV), slot[:, p]]
        self.valid = c["mode"] != "full"
        return y


def _exact_layer(case, seed):
    w, xs, attn = _layer_inputs(case, seed)
    B, N, d = case["B"], case["N"], case["d"]
    L, ys, feat = _Exact(case, w), [], None
    for t, x in enumerate(xs):
        xd = x.double().view(B * N, d)
        dec = L.decide(xd)
        ys.append(L.finish(xd, *dec).view(B, N, d))
        sync = dec[2].any(dim=1).view(B, N, 1)
        feat = attn[t].double() if feat is None else torch.where(sync, attn[t].double(), feat)
    out = {"y": ys}
    if case["mode"] != "full":
        k = case["k"]
        out.update(attention=feat, rows=L.rows.view(B, N, k, d), norms=L.n.view(B, N, k),
                   experts=None, statistic=L.C)
    return out


def _ln(x):
    mu = x.mean(dim=-1, keepdim=True)
    return (x - mu) / torch.sqrt(((x - mu) ** 2).mean(dim=-1, keepdim=True) + 1e-6)


def _attention64(q, k, v, heads):
    B, N, d = q.shape
    out = torch.empty_like(q)
    dh = d // heads
    for b in range(B):
        qh, kh, vh = (t[b].view(N, heads, dh).transpose(0, 1).contiguous() for t in (q, k, v))
        p = torch.softmax(torch.bmm(qh, kh.transpose(1, 2).contiguous()) / math.sqrt(dh), dim=2)
        out[b] = torch.bmm(p, vh).transpose(0, 1).reshape(N, d)
    return out


def _exact_stack(case, seed):
    blocks, emb, labels, ts, xs = _stack_inputs(case, seed)
    B, N, d, heads = case["B"], case["N"], case["d"], case["heads"]
    layers = [_Exact(case, {"r": b["W_r"], "b": None, "up": b["W_up"], "down": b["W_down"]})
              for b in blocks]
    feats, outs, cs = [None] * len(blocks), [], []
    i = torch.arange(128, device=DEV, dtype=torch.float64)
    freq = torch.exp(-math.log(10000.0) * i / 128)
    for t, x in enumerate(xs):
        arg = ts[t].double()[:, None] * freq[None, :]
        h1 = torch.cat([torch.cos(arg), torch.sin(arg)], 1) @ emb["W1"].double().T + emb["b1"]
        c = torch.nn.functional.silu(h1) @ emb["W2"].double().T + emb["b2"].double()
        c = c + emb["table"][labels.long()].double()
        cs.append(c)
        v = x.double()
        for l, (w, L) in enumerate(zip(blocks, layers)):
            mod = torch.nn.functional.silu(c) @ w["W_ada"].double().T + w["b_ada"].double()
            sa, ca, ga, sm, cm, gm = (m[:, None, :] for m in mod.view(B, 6, d).unbind(1))
            h = _ln(v) * (1.0 + ca) + sa
            qkv = h @ w["W_qkv"].double().T + w["b_qkv"].double()
            o = _attention64(*(m.contiguous() for m in qkv.split(d, dim=2)), heads)
            fresh = o @ w["W_o"].double().T + w["b_o"].double()
            # the routing input is stored in bf16: the router sees that value
            def mlp_in(a, v=v, ga=ga, sm=sm, cm=cm):
                x1 = v + ga * a
                return x1, _ln(x1) * (1.0 + cm) + sm
            full = not L.valid or case["mode"] == "full"
            feat = fresh if full else feats[l]
            x1, u = mlp_in(feat)
            ur = u.to(torch.bfloat16).double().view(B * N, d)
            dec = L.decide(ur)
            if not full:
                sync = dec[2].any(dim=1).view(B, N, 1)
                feat = torch.where(sync, fresh, feat)
                x1, u = mlp_in(feat)
            feats[l] = feat
            y = L.finish(u.reshape(B * N, d), *dec).view(B, N, d)
            v = x1 + gm * y
        outs.append(v)
    return {"x": outs, "c": cs, "attention": feats}


def exact(case, seed):
    w = work(case)
    if w["flops"] > 2e13:
        return None
    return _exact_stack(case, seed) if case["kind"] == "stack" else _exact_layer(case, seed)
