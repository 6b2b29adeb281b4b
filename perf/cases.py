"""What a program that serves a model with a budgeted Crystal-KV cache has the library do, as cases to time.

A case is a dict of plain values; `prepare` builds what such a program has in hand before the call (caches in the
middle of a sequence, the coming steps' queries, keys and values, a captured graph, a prompt), `run` makes one pass
through the binding, `exact` says what its floating-point outputs are in 64 bits.  Kinds of case:

  step     one decode step of all layers in one call: append, attend, score, evict
  layers   the same step as one call per layer, as a model makes it; `defer`: bookkeeping on the context's own
           streams; `graph`: the calls of the step captured once and replayed
  window   the sink-plus-recent-window baseline over a full cache: an attention-only step, then the window eviction
  seed     scores of loaded prompts from the last queries of each, layer by layer
  probe    answer-probe classes of one layer
  admit    a new batch of sequences: a context on memory the program holds, per layer load the prompt, score it,
           evict to the budget; then the first steps, with a re-allocation of the budgets after the first

Geometries, lengths, budgets and parameters are those of the workloads in `paper_2601_16986_amd.workloads` (or plain
generic ones in drawn cases); the content of the caches follows the same recipe, with one mean query and one drift per
state instead of one per head, so that a step's inputs can be taken at any row offset of a buffer: a state holds the
inputs of RING consecutive steps and moves them up one row each time round, so no unit sees the same key twice for
RING * PAD steps (keys replayed exactly would tie with their cached copies, which a model's never do).
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2601_16986_amd import ckv
from paper_2601_16986_amd import workloads as wl

DEVICE = "cuda:0"
D = 128                  # head dimension, the only one the library takes
RING, PAD = 32, 64
N_SINK = 4


def _case(name, kind, layers, batch, hq, hkv, budget, **more):
    c = dict(name=name, kind=kind, layers=layers, batch=batch, hq=hq, hkv=hkv, budget=budget, adaptive=False, lam=0.5, top_p=0.9,
             weighted=False, bf16=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one sequence, one layer of two KV heads; latency and launches are all there is
        _case("step_tiny", "step", 1, 1, 8, 2, 128),
        # 7B geometry (G = 7), a small batch
        _case("step_7b", "step", 28, 8, 28, 4, 2048, bf16=True),
        # 14B geometry with budgets that differ by head (257 .. 8193 entries), the headline workload
        _case("step_14b", "step", 48, 16, 40, 8, 2048, adaptive=True),
        # Llama-8B geometry, a large batch of short caches
        _case("step_llama8b", "step", 32, 64, 32, 8, 1024),
        # the 14B layers as a model calls them, scores and eviction on the caller's stream
        _case("layers_14b", "layers", 12, 16, 40, 8, 2048, adaptive=True, defer=False, graph=False),
        # the same with the bookkeeping on the context's own streams
        _case("layers_14b_defer", "layers", 12, 16, 40, 8, 2048, adaptive=True, defer=True, graph=False),
        # one sequence on a whole 14B model, captured in a graph: interactive decoding
        _case("graph_14b_one", "layers", 48, 1, 40, 8, 2048, adaptive=True, defer=True, graph=True),
        # full caches of 9350 tokens (8K level) on the Llama-8B geometry with the window policy
        _case("window_8b", "window", 4, 16, 32, 8, 9350),
        # scores of 8K-level prompts from their last 32 queries
        _case("seed_14b", "seed", 8, 16, 40, 8, 2048, prompt=9350, queries=32),
        # answer probe on one layer of the 14B geometry
        _case("probe_14b", "probe", 2, 16, 40, 8, 2048, adaptive=True),
        # one short chat prompt on a small model's cache
        _case("admit_one", "admit", 4, 1, 28, 4, 256, prompt=777, queries=16),
        # a batch of 8K-level prompts on a third of the 14B layers
        _case("admit_14b", "admit", 16, 8, 40, 8, 2048, adaptive=True, prompt=9350, queries=32),
    ]


HEADS = [(8, 2), (28, 4), (40, 8), (32, 8), (16, 16), (24, 8), (64, 8), (4, 1)]


def draw(rng):
    def log_int(lo, hi):
        return int(round(float(lo) * (float(hi) / lo) ** rng.random()))

    kind = rng.choice(["step", "step", "step", "layers", "layers", "layers", "window", "seed", "probe", "admit"])
    hq, hkv = rng.choice(HEADS)
    adaptive = rng.random() < 0.4
    budget = log_int(96, 6000)
    layers, batch = log_int(1, 48), log_int(1, 64)
    most = {"step": 12_000_000, "layers": 3_000_000, "window": 4_000_000, "seed": 9_000_000, "probe": 1_200_000, "admit": 9_000_000}[kind]
    more = {}
    per_unit = budget
    if kind == "layers":
        more["defer"] = rng.random() < 0.5
        more["graph"] = rng.random() < 0.3
        layers = min(layers, 24)
    if kind in ("seed", "admit"):
        more["prompt"] = per_unit = log_int(max(200, budget // 2), 12000)
        more["queries"] = log_int(1, 48)
        layers = min(layers, 8)
    if kind == "window":
        budget = per_unit = log_int(300, 12000)
        adaptive = False
        layers = min(layers, 8)
    if kind == "probe":
        layers = 1
    while layers > 1 and layers * batch * hkv * per_unit > most:
        layers = (layers + 1) // 2
    while batch > 1 and layers * batch * hkv * per_unit > most:
        batch = (batch + 1) // 2
    if layers * hkv == 1:
        adaptive = False               # a single unit per sequence has nothing to share its budget with
    c = _case("", kind, layers, batch, hq, hkv, budget, adaptive=adaptive, lam=rng.choice([0.5, 0.6, 0.7]), top_p=rng.choice([0.8, 0.9, 0.95]),
              weighted=rng.random() < 0.15, bf16=rng.random() < 0.5, **more)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _config(case, seed):
    b = case["budget"]
    lo, hi = (max(16, b // 8), 4 * b) if case["adaptive"] else (b, b)
    return wl.Config("perf", case["layers"], case["batch"], case["hq"], case["hkv"], D, case.get("prompt", 0), 0, b, lo, hi, case["adaptive"], 0,
                     lam=case["lam"], top_p=case["top_p"], seed=int(seed))


def _t_now(case):
    return case["budget"] if case["kind"] == "window" else case["prompt"] if case["kind"] in ("seed", "admit") else max(8704, 8 * case["budget"])


def _shared(cfg):
    """The state's mean query and drift, [d] each."""
    g = wl.torch_generator(cfg, 1, DEVICE)
    m = torch.randn(D, generator=g, device=DEVICE)
    return m * (wl.M_NORM / m.norm()), float(np.sqrt(wl.DRIFT_VAR)) * torch.randn(D, generator=g, device=DEVICE)


def _steps(cfg, m, r, rows, count, group):
    """Inputs of `count` consecutive steps for `rows` units (and PAD rows more): q [count][rows + PAD][G][d], k, v."""
    g = wl.torch_generator(cfg, 7, DEVICE)
    q = torch.empty((count, rows + PAD, group, D), dtype=torch.bfloat16, device=DEVICE)
    k = torch.empty((count, rows + PAD, D), dtype=torch.bfloat16, device=DEVICE)
    v = torch.empty_like(k)
    for s in range(count):
        r = wl.RHO * r + float(np.sqrt((1 - wl.RHO ** 2) * wl.DRIFT_VAR)) * torch.randn(D, generator=g, device=DEVICE)
        heavy = torch.rand((rows + PAD, 1), generator=g, device=DEVICE) < wl.HEAVY_FRACTION
        q[s] = torch.randn((rows + PAD, group, D), generator=g, device=DEVICE) + (m + r)
        k[s] = torch.randn((rows + PAD, D), generator=g, device=DEVICE) + (wl.HEAVY_GAIN * heavy * m + r)
        v[s] = torch.randn((rows + PAD, D), generator=g, device=DEVICE)
    return q, k, v


def _cache_layer(case, cfg, layer, budgets, m, r):
    """One layer's caches mid-way through a sequence: bf16 k, v [Bz][Hkv][P][d], int32 lengths, crf, tau, pos."""
    e = (cfg.batch, cfg.n_kv_heads, D)
    return wl.torch_steady_layer(cfg, layer, budgets[layer], _t_now(case), m.expand(e), r.expand(e), DEVICE)


def _prompt_layer(case, cfg, layer, m):
    """One layer's prompt: bf16 k, v [Bz][Hkv][P][d], the queries of its last positions [W][Bz][Hq][d], and the drift there.
    The drift of the prompt's positions is one AR(1) path for all heads."""
    P, W = case["budget" if case["kind"] == "window" else "prompt"], case.get("queries", 1)
    g = wl.torch_generator(cfg, 100 + layer, DEVICE)
    h = np.random.Generator(np.random.Philox(key=[cfg.seed, layer]))
    xi = h.standard_normal((P, D)).astype(np.float32) * np.float32(np.sqrt((1 - wl.RHO ** 2) * wl.DRIFT_VAR))
    xi[0] = h.standard_normal(D) * np.sqrt(wl.DRIFT_VAR)
    # r_i = rho r_{i-1} + xi_i, in pieces short enough for the powers of rho to stay in range
    path, last = np.empty((P, D), np.float64), np.zeros(D)
    for a in range(0, P, 512):
        n = min(512, P - a)
        pw = wl.RHO ** np.arange(1, n + 1)[:, None]
        path[a:a + n] = pw * (last + np.cumsum(xi[a:a + n] / pw, axis=0))
        last = path[a + n - 1]
    drift = torch.from_numpy(path.astype(np.float32)).to(DEVICE)
    shape = (cfg.batch, cfg.n_kv_heads, P, D)
    k = torch.randn(shape, generator=g, device=DEVICE)
    heavy = torch.rand(shape[:3] + (1,), generator=g, device=DEVICE) < wl.HEAVY_FRACTION
    k += drift
    k += wl.HEAVY_GAIN * heavy * m
    v = torch.randn(shape, generator=g, device=DEVICE)
    q = torch.randn((W, cfg.batch, cfg.n_q_heads, D), generator=g, device=DEVICE) + m + drift[P - W:].reshape(W, 1, 1, D)
    return k.to(torch.bfloat16), v.to(torch.bfloat16), q.to(torch.bfloat16), drift[-1]


class State:
    """What the program holds between passes."""

    def __init__(self, case, seed):
        self.case, self.cfg = case, _config(case, seed)
        self.budgets = wl.draw_budgets(self.cfg)
        self.rows = self.cfg.n_units
        self.m, self.r = _shared(self.cfg)
        self.step = 0
        self.g = None

    def inputs(self):
        """The next step's q [L][Bz][Hq][d], k, v [L][Bz][Hkv][d]."""
        s, up = self.step % RING, (self.step // RING) % (PAD + 1)
        self.step += 1
        c, n = self.cfg, self.rows
        return (self.q[s, up:up + n].view(c.n_layers, c.batch, c.n_q_heads, D), self.k[s, up:up + n].view(c.n_layers, c.batch, c.n_kv_heads, D),
                self.v[s, up:up + n].view(c.n_layers, c.batch, c.n_kv_heads, D))

    def context_args(self):
        c, case = self.cfg, self.case
        longest = max(int(self.budgets.max()), c.budget_max, case.get("prompt", 0)) + 2
        args = (c.n_layers, c.batch, c.n_q_heads, c.n_kv_heads, D, (longest + 31) // 32 * 32, self.budgets)
        # prompts that stay (seed) are held by every layer at once; elsewhere the pools follow the budgets
        more = dict(lam=c.lam, top_p=c.top_p, t0=_t_now(case), budget_min=c.budget_min, budget_max=c.budget_max,
                    reward_mode=ckv.REWARD_ATTN_WEIGHTED if case["weighted"] else ckv.REWARD_TOPP_HIT,
                    out_dtype=ckv.BF16 if case["bf16"] else ckv.F32, headroom=0 if case["kind"] == "seed" else 1,
                    prompt_len=case["prompt"] if case["kind"] == "admit" else 0)
        return args, more

    def scores(self):
        """The per-slot arrays: whole, or each unit's live entries where all units hold the same number."""
        g = self.g
        if self.case["adaptive"]:
            return {"crf": g.crf, "tau": g.tau, "pos": g.pos}
        live = self.case["prompt"] if self.case["kind"] == "seed" else self.case["budget"]
        held = g.pool_slots // self.rows // 256 * 256 if g.headroom == 0 else (live + 1 + 255) // 256 * 256
        return {n: x[:self.rows * held].view(self.rows, held)[:, :live] for n, x in (("crf", g.crf), ("tau", g.tau), ("pos", g.pos))}


def prepare(case, seed):
    st = State(case, seed)
    cfg, kind = st.cfg, case["kind"]
    args, more = st.context_args()
    if kind == "admit":
        st.arena = torch.empty(ckv.arena_bytes(*args, **more), dtype=torch.uint8, device=DEVICE)
        st.prompts = [_prompt_layer(case, cfg, l, st.m) for l in range(cfg.n_layers)]
        st.q, st.k, st.v = _steps(cfg, st.m, st.prompts[0][3], st.rows, 3, cfg.group)
        return st
    st.g = ckv.CrystalKV(*args, **more)
    if kind in ("seed", "window"):
        prompts = [_prompt_layer(case, cfg, l, st.m) for l in range(cfg.n_layers)]
        for l, p in enumerate(prompts):
            st.g.load_prompt(l, p[0], p[1])
        st.q_obs = [p[2] for p in prompts]
        st.r = prompts[0][3]
    else:
        for l in range(cfg.n_layers):
            st.g.load_cache(l, *_cache_layer(case, cfg, l, st.budgets, st.m, st.r))
    if kind == "probe":
        gen = wl.torch_generator(cfg, 9, DEVICE)
        st.probe = (torch.randn((cfg.batch, cfg.n_q_heads, D), generator=gen, device=DEVICE) + st.m).to(torch.bfloat16)
    if kind in ("step", "layers", "window"):
        st.q, st.k, st.v = _steps(cfg, st.m, st.r, st.rows, RING, cfg.group)
    if kind == "layers":
        st.out = torch.empty((cfg.n_layers, cfg.batch, cfg.n_q_heads, D), dtype=torch.bfloat16 if case["bf16"] else torch.float32, device=DEVICE)
        if case["graph"]:
            st.now = [torch.empty_like(x) for x in st.inputs()]
            st.step = 0
            torch.cuda.synchronize()
            st.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(st.graph):
                _layer_calls(st, *st.now)
    return st


def _layer_calls(st, q, k, v):
    defer = st.case["defer"]
    for l in range(st.cfg.n_layers):
        st.g.decode_step(q[l], k[l], v[l], layer=l, out=st.out[l], defer=defer)
    if defer:
        st.g.join()


def run(st):
    case, g = st.case, st.g
    kind = case["kind"]
    if kind == "step":
        return {"out": g.decode_step(*st.inputs()), **st.scores()}
    if kind == "layers":
        if case["graph"]:
            for x, y in zip(st.now, st.inputs()):
                x.copy_(y)
            st.graph.replay()
        else:
            _layer_calls(st, *st.inputs())
        return {"out": st.out, **st.scores()}
    if kind == "window":
        out = g.decode_step(*st.inputs(), attention_only=True)
        g.evict_window(N_SINK)
        return {"out": out, "pos": st.scores()["pos"]}
    if kind == "seed":
        for l in range(st.cfg.n_layers):
            g.seed_prompt(l, st.q_obs[l])
        s = st.scores()
        return {"crf": s["crf"], "tau": s["tau"]}
    if kind == "probe":
        return {"classes": g.probe(0, st.probe)}
    # admit: the sequences served before are done
    if g is not None:
        g.close()
    args, more = st.context_args()
    st.g = g = ckv.CrystalKV(*args, arena=st.arena, **more)
    for l, (k, v, q_obs, _) in enumerate(st.prompts):
        g.load_prompt(l, k, v)
        g.seed_prompt(l, q_obs)
        g.evict(l)
    st.step = 0
    outs = [g.decode_step(*st.inputs())]
    g.rebudget()
    outs.append(g.decode_step(*st.inputs()))
    outs.append(g.decode_step(*st.inputs()))
    return {"out": outs}


def work(case):
    units, group = case["layers"] * case["batch"] * case["hkv"], case["hq"] // case["hkv"]
    kind, n = case["kind"], case["budget"] + 1
    width = 2 if case["bf16"] else 4
    q_out = units * group * D * (2 + width)                     # queries in, attention out
    if kind in ("step", "layers"):
        # K and V rows, score, time and position of every entry; the new entry in, one row over the evicted one
        return {"bytes": units * (n * (4 * D + 12) + 2 * 4 * D) + q_out, "flops": 4 * D * group * units * n}
    if kind == "window":
        return {"bytes": units * (n * (4 * D + 4) + 2 * 4 * D) + q_out, "flops": 4 * D * group * units * n}
    if kind == "seed":
        P, W = case["prompt"], case["queries"]
        return {"bytes": units * (P * (2 * D + 8) + W * group * 2 * D), "flops": 2 * D * group * W * units * P}
    if kind == "probe":
        units //= case["layers"]
        return {"bytes": units * (case["budget"] * (2 * D + 4 + 1) + group * 2 * D), "flops": 2 * D * group * units * case["budget"]}
    P, W = case["prompt"], case["queries"]
    kept = min(P, case["budget"])
    return {"bytes": units * (P * 4 * D + kept * (4 * D + 12) + W * group * 2 * D + 3 * (kept + 1) * (4 * D + 12)) + 3 * q_out,
            "flops": 2 * D * group * W * units * P + 3 * 4 * D * group * units * (kept + 1)}


def tolerance(case):
    """Measured against runs whose logits were scaled by one unit in the last place more or less (another rounding of every weight): about
    four times what that moved."""
    kind, units = case["kind"], case["layers"] * case["batch"] * case["hkv"]
    # fp32 outputs moved by 7.5e-7 (largest single one 3.4e-5), bf16 ones by 4e-5 (one unit in the last place, 2^-7)
    out = {"rel": 1e-3, "max": 0.016} if case["bf16"] else {"rel": 4e-6, "max": 2e-4}
    if kind == "window":
        return out                                              # positions follow the policy alone and stay the same
    if kind == "probe":
        # two entries next to the edge of a class changed places in none of 128 units; the weights' spacing there allows for one in 500
        return {"rel": 0.0, "differ": min(0.01, max(4, units / 60) / (units * case["budget"]))}
    if kind == "admit":
        # a hit that falls the other way can keep one entry in another's place: 5.5e-5 over 1024 units (largest 0.01)
        return {"rel": min(0.02, max(1e-3, 0.03 / units ** 0.5)), "max": 0.2}
    if case["weighted"]:
        return {"rel": max(out["rel"], 4e-6), "max": out["max"]}    # scores are sums of weights: 2.6e-7
    # a weight within rounding of the top-p threshold is hit or not: up to 6 of 6144 units per step (9 of 32768 replayed queries), one
    # entry's score by 1 at most (scores are 1.3 on average) and its time; later queries of a replay then differ on that entry too
    entries = units * (case["prompt"] if kind == "seed" else case["budget"])
    flips = 4 * max(1.0, units * (case["queries"] if kind == "seed" else 1) / 1000.0)
    return {"rel": min(0.03, max(out["rel"], (flips / entries) ** 0.5)), "max": 0.95, "differ": min(0.01, flips / entries)}


# ------------------------------------------------------------------ the same in 64 bits
def _attend(q, k, v, lengths):
    """q [Bz][Hkv][G][d], k, v [Bz][Hkv][P][d], lengths [Bz][Hkv] -> softmax(q k^T / sqrt(d)) v over each unit's entries, in 64 bits."""
    k, v = k.double(), v.double()
    dead = torch.arange(k.shape[2], device=k.device) >= lengths.unsqueeze(-1)
    out = []
    for h in range(q.shape[2]):
        s = (k * q[:, :, h:h + 1].double()).sum(-1) / float(np.sqrt(D))
        a = torch.softmax(s.masked_fill(dead, float("-inf")), dim=-1)
        out.append((a.unsqueeze(-1) * v).sum(2))
    return torch.stack(out, dim=2)


def _exact_seed(case, st):
    """Scores of the prompts' entries under the attention-weighted reward, where no threshold decides anything."""
    P, W, lam, c = case["prompt"], case["queries"], float(np.float32(case["lam"])), st.cfg
    crfs = []
    for l in range(c.n_layers):
        k, _, q, _ = _prompt_layer(case, c, l, st.m)
        kt = k.double().transpose(2, 3).contiguous()
        pos = torch.arange(P, device=DEVICE)
        crf = torch.where(pos < P - W, 1.0, 0.0).double().expand(c.batch, c.n_kv_heads, P).clone()
        tau = pos.clone()
        for j in range(W):
            t = P - W + j
            s = torch.matmul(q[j].view(c.batch, c.n_kv_heads, c.group, D).double(), kt) / float(np.sqrt(D))
            a = torch.softmax(s[..., :t + 1], dim=-1).mean(2)
            crf[..., :t + 1] = crf[..., :t + 1] * lam ** (t - tau[:t + 1]).double() + a
            tau[:t + 1] = t
        crfs.append(crf.reshape(-1, P))
    return torch.cat(crfs)


def exact(case, seed):
    kind = case["kind"]
    st = State(case, seed)
    cfg = st.cfg
    if kind == "seed":
        # under the top-p reward scores follow hits, and a weight within rounding of the threshold may fall either way
        return {"crf": _exact_seed(case, st), "tau": None} if case["weighted"] else None
    if kind not in ("step", "layers", "window"):
        return None                     # classes are whole numbers; what an admitted batch attends to follows from its hits
    if kind == "window":
        prompts = [_prompt_layer(case, cfg, l, st.m) for l in range(cfg.n_layers)]
        st.r = prompts[0][3]
    st.q, st.k, st.v = _steps(cfg, st.m, st.r, st.rows, 1, cfg.group)
    q, kn, vn = st.inputs()
    out = []
    for l in range(cfg.n_layers):
        if kind == "window":
            k, v = prompts[l][:2]
            n = torch.full((cfg.batch, cfg.n_kv_heads), k.shape[2], device=DEVICE)
        else:
            k, v, n = _cache_layer(case, cfg, l, st.budgets, st.m, st.r)[:3]
        k, v = torch.cat([k, kn[l].unsqueeze(2)], dim=2), torch.cat([v, vn[l].unsqueeze(2)], dim=2)
        at = n.long()[..., None, None].expand(-1, -1, 1, D)      # the new entry right behind the unit's own
        k, v = k.scatter(2, at, kn[l].unsqueeze(2)), v.scatter(2, at, vn[l].unsqueeze(2))
        out.append(_attend(q[l].view(cfg.batch, cfg.n_kv_heads, cfg.group, D), k, v, n + 1).reshape(cfg.batch, cfg.n_q_heads, D))
    none = {"pos": None} if kind == "window" else {"crf": None, "tau": None, "pos": None}
    return {"out": torch.stack(out), **none}
