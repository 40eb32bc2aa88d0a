"""The work that users of the library have it do, as timed cases: subgraph
builds, mean and attention layers, the alignment, the temporal module and a
whole small training step, each through the public entry points of
``paper_2608_02168_amd.api`` (the step through ``runner``).

``listed()`` names fixed cases, ``draw(rng)`` more of the same ranges;
``prepare`` makes the inputs, weights, subgraph and buffers that a program has
in hand (all from the seed), ``run`` is one pass, ``work`` the bytes and
operations a pass cannot do without, ``exact`` the outputs in float64 by plain
torch, ``tolerance`` how far a correct implementation of the same precision
may be from another.

Graphs follow the synthetic workloads of ``paper_2608_02168_amd.synth`` (a
shifted Zipf law over the sources, uniform destinations and relations, the top
1 % of ranks as the second node type, a prefix or a random block as the base
set), drawn on the GPU.
"""
from __future__ import annotations

import math
from dataclasses import replace

import torch

from paper_2608_02168_amd import api, runner, synth

DEV = "cuda"
F32, BF16, F64 = torch.float32, torch.bfloat16, torch.float64


# ---- cases ------------------------------------------------------------------

def listed():
    medium = dict(nodes=1_000_000, edges=20_000_000, rels=4, zipf_s=1.2, zipf_k0=0.0, base=900_000, parts=0,
                  budget=100_000, key=api.HG_KEY_OUTDEG, theta=api.HG_THETA_NONE)
    large = dict(nodes=10_000_000, edges=200_000_000, rels=5, zipf_s=1.3, zipf_k0=634.0, base=9_200_000, parts=0,
                 budget=800_000, key=api.HG_KEY_OUTDEG, theta=api.HG_THETA_NONE)
    # the large graph's recipe at a tenth of its size
    tenth = dict(large, nodes=1_000_000, edges=20_000_000, zipf_k0=63.4, base=920_000, budget=80_000)
    # one block of a random 8-way partition, the h-index filter at 2, an overlap of 0.3 of a block: the
    # paper's default selection, one worker's build of a graph shared by eight
    block = dict(large, nodes=2_500_000, edges=50_000_000, zipf_k0=158.5, base=0, parts=8, budget=93_750,
                 key=api.HG_KEY_HINDEX, theta=2)
    f32 = dict(dtype="f32", weighted=False)
    return [
        # a whole training step (build, two mean layers, head and BCE, alignment, backward, Adam) on the
        # smallest workload: launches, host work and latency
        dict(name="step_small", kind="step", model="full", scale=1.0),
        # subgraph construction: once before training, or per step where the graph changes
        dict(name="build_1m", kind="build", **medium),
        dict(name="build_block", kind="build", **block),
        dict(name="build_large", kind="build", **large),
        # one mean layer, forward (inference too) and backward, float32 rows at the default width
        dict(name="mean_fwd_1m", kind="mean_fwd", d=128, **f32, **medium),
        dict(name="mean_bwd_1m", kind="mean_bwd", d=128, **f32, **medium),
        dict(name="mean_bwd_large", kind="mean_bwd", d=128, **f32, **large),
        # the bfloat16 workload's width and storage
        dict(name="mean_fwd_bf16", kind="mean_fwd", d=256, dtype="bf16", weighted=False, **tenth),
        dict(name="mean_bwd_bf16", kind="mean_bwd", d=256, dtype="bf16", weighted=False, **tenth),
        # one attention layer in training, the paper's width and heads
        dict(name="hgt_1m", kind="hgt", d=64, heads=4, lean=False, **tenth),
        # the alignment of a worker's overlap rows
        dict(name="align_100k", kind="align", d=128, dtype="f32", rows=1_000_000, overlap=100_003, weighted=False),
        # the temporal module over the three past months of a million nodes
        dict(name="temporal_1m", kind="temporal", d=64, dtype="f32", rows=1_000_000, window=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, max_nodes, max_edges, whole=False):
    """whole: the sizes of the subgraph's arrays are the same for every seed."""
    n = _log(rng, 1_000, max_nodes) | 1
    e = min(max_edges, int(n * rng.uniform(5, 30)))
    s, k0 = rng.choice([(1.1, 0.0), (1.2, 0.0), (1.3, 634e-7 * n), (1.6, 6339 / 5e6 * n)])
    if whole or rng.random() < 0.7:
        base, parts = int(n * rng.uniform(0.8, 0.95)), 0
        budget = max(1, int((n - base) * rng.uniform(0.3, 0.8 if whole else 1.2)))
    else:
        base, parts = 0, rng.randint(2, 8)
        budget = max(1, int(n / parts * rng.uniform(0.1, 0.6)))
    key = rng.choice([api.HG_KEY_OUTDEG, api.HG_KEY_OUTDEG, api.HG_KEY_HINDEX])
    theta = rng.choice([api.HG_THETA_NONE, api.HG_THETA_NONE, 2, 5])
    if whole:
        theta = api.HG_THETA_NONE
    return dict(nodes=n, edges=e, rels=rng.choice([2, 3, 4, 5, 8, 12, 24]), zipf_s=s, zipf_k0=k0, base=base,
                parts=parts, budget=budget, key=key, theta=theta)


def draw(rng):
    kind = rng.choice(["step", "build", "build", "mean_fwd", "mean_fwd", "mean_bwd", "mean_bwd", "hgt", "align",
                       "temporal"])
    if kind == "step":
        return dict(kind=kind, model=rng.choice(["full", "hgt"]), scale=round(math.exp(rng.uniform(-2.0, 1.2)), 3))
    if kind == "build":
        return dict(kind=kind, **_draw_graph(rng, 7_000_000, 150_000_000))
    if kind in ("mean_fwd", "mean_bwd"):
        d = rng.choice([64, 128, 256])
        bf16 = rng.random() < 0.4
        g = _draw_graph(rng, *((2_000_000, 40_000_000) if bf16 or d == 256 else (5_000_000, 100_000_000)), whole=True)
        return dict(kind=kind, d=d, dtype="bf16" if bf16 else "f32", weighted=not bf16 and rng.random() < 0.3, **g)
    if kind == "hgt":
        d = rng.choice([64, 64, 128])
        return dict(kind=kind, d=d, heads=rng.choice([1, 2, 4, 8]), lean=rng.random() < 0.3,
                    **_draw_graph(rng, 1_000_000, 64 * 20_000_000 // d, whole=True))
    if kind == "align":
        rows = _log(rng, 2_000, 5_000_000) | 1
        return dict(kind=kind, d=rng.choice([64, 128, 128, 256]), dtype=rng.choice(["f32", "f32", "bf16"]), rows=rows,
                    overlap=max(300, int(rows * rng.uniform(0.05, 0.15))), weighted=rng.random() < 0.3)
    return dict(kind=kind, d=64, dtype=rng.choice(["f32", "f32", "bf16"]), rows=_log(rng, 3_000, 3_000_000) | 1,
                window=rng.randint(0, 4))


# ---- inputs -----------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 64 + stream)
    return g


def _graph(case, seed):
    """Typed edges, node types and partition of a case, on the GPU."""
    n, e, rels = case["nodes"], case["edges"], case["rels"]
    g = _gen(seed, 1)
    node_of_rank = torch.randperm(n, generator=g, device=DEV)
    # ranks by the inverse of the continuous law's distribution function (elementwise, so the same on every run)
    lo, p = case["zipf_k0"] + 0.5, 1.0 - case["zipf_s"]
    src = torch.empty(e, dtype=torch.int32, device=DEV)
    for at in range(0, e, 1 << 25):
        u = torch.rand(min(1 << 25, e - at), dtype=F64, device=DEV, generator=g)
        rank = (lo**p + u * ((n + lo)**p - lo**p)).pow_(1.0 / p).sub_(lo).long().clamp_(0, n - 1)
        src[at:at + u.numel()] = node_of_rank[rank]
    dst = torch.randint(0, n, (e,), dtype=torch.int32, device=DEV, generator=g)
    rel = torch.randint(0, rels, (e,), dtype=torch.uint8, device=DEV, generator=g)
    ntype = torch.zeros(n, dtype=torch.uint8, device=DEV)
    ntype[node_of_rank[:max(1, n // 100)]] = 1
    if case["parts"]:
        part = torch.randint(0, case["parts"], (n,), dtype=torch.int32, device=DEV, generator=g)
    else:
        part = (torch.arange(n, device=DEV) >= case["base"]).to(torch.int32)
    w = None
    if case.get("weighted"):
        w = torch.rand(e, device=DEV, generator=g) * 1.9 + 0.1
    return dict(src=src, dst=dst, rel=rel, ntype=ntype, part=part, edge_w=w)


def _build(case, seed, g, **kw):
    return api.hg_build_csr(g["src"], g["dst"], g["rel"], g["ntype"], g["part"], 0, case["rels"], 2, case["budget"],
                            key=case["key"], theta=case["theta"], seed=seed, want_eid=False, edge_w=g["edge_w"], **kw)


def _uniform(g, shape, a):
    return torch.empty(shape, device=DEV).uniform_(-a, a, generator=g)


def _normal(g, shape, dtype=F32):
    return torch.randn(shape, device=DEV, generator=g).to(dtype)


def _dtype(case):
    return BF16 if case["dtype"] == "bf16" else F32


def _mean_inputs(case, seed, n):
    """Rows, weights, and for a backward the upstream gradient and the
    forward's ReLU mask (half of its bits set, as for random rows)."""
    d, R, dt = case["d"], case["rels"], _dtype(case)
    g = _gen(seed, 2)
    a = math.sqrt(6.0 / (2 * d))
    s = dict(H=_normal(g, (n, d), dt), W_rel=_uniform(g, (R, d, d), a), W_self=_uniform(g, (2, d, d), a),
             bias=_uniform(g, (2, d), 0.1))
    if case["kind"] == "mean_bwd":
        s["G"] = _normal(g, (n, d), dt)
        s["mask"] = torch.randint(-2**31, 2**31, (n, d // 32), dtype=torch.int32, device=DEV, generator=g)
    return s


def _hgt_inputs(case, seed, n):
    d, R, S = case["d"], case["rels"], case["heads"]
    g = _gen(seed, 3)
    a, ak = math.sqrt(6.0 / (2 * d)), math.sqrt(6.0 / (2 * (d // S)))
    W = {k: _uniform(g, (2, d, d), a) for k in ("W_K", "W_Q", "W_V", "W_agg")}
    W.update({k: _uniform(g, (R, S, d // S, d // S), ak) for k in ("W_att", "W_msg")})
    W["mu"] = _uniform(g, (2, R, 2), 0.5) + 1.0
    W.update({k: _uniform(g, (2, d), 0.1) for k in ("b_K", "b_Q", "b_V", "b_agg")})
    return dict(H=_normal(g, (n, d)), G=_normal(g, (n, d)), W=W)


def _align_inputs(case, seed):
    n, m, d, dt = case["rows"], case["overlap"], case["d"], _dtype(case)
    g = _gen(seed, 4)
    H = _normal(g, (n, d), dt)
    overlap = torch.randperm(n, device=DEV, generator=g)[:m].sort().values.to(torch.int32)
    # the other view of a node: its own row with as much noise
    ref = (H[overlap.long()].float() + _normal(g, (m, d))).to(dt)
    w = torch.rand(m, device=DEV, generator=g) + 0.5 if case["weighted"] else None
    return dict(H=H, overlap=overlap, ref=ref, base=_normal(g, (n, d), dt), w=w)


def _temporal_inputs(case, seed):
    n, d, w, dt = case["rows"], case["d"], case["window"], _dtype(case)
    g = _gen(seed, 5)
    a = 1.0 / math.sqrt(d)
    W = dict(Q=_uniform(g, (d, d), a), r=_uniform(g, (d,), 1.0), Wi=_uniform(g, (3, d, d), a),
             bi=_uniform(g, (3, d), 0.1), Wh=_uniform(g, (3, d, d), a), bh=_uniform(g, (3, d), 0.1))
    return dict(W=W, h=_normal(g, (n, d), dt), C=[(0.5 * _normal(g, (n, d))).to(dt) for _ in range(w)],
                dH=_normal(g, (n, d), dt))


def _step_workload(case, seed):
    wl = synth.WORKLOADS["tiny_" + case["model"]]
    return replace(wl, graph=replace(synth.scaled(wl.graph, case["scale"]), seed=seed),
                   model=replace(wl.model, seed=seed))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        wl = _step_workload(case, seed)
        return dict(kind=kind, inp=runner.make_inputs(wl, synth.make_graph(wl.graph), device=DEV))
    s = dict(kind=kind, case=case, seed=seed)
    if kind == "build":
        s["g"] = _graph(case, seed)
        s["sub"] = _build(case, seed, s["g"])
        s["ws"] = s["sub"].arrays["ws"]
        # arrays are returned to their capacity: zeros past the counts, which differ with the seed
        for k in BUILD_OUT:
            s["sub"].arrays[k].zero_()
    elif kind in ("mean_fwd", "mean_bwd"):
        sub = s["sub"] = _build(case, seed, _graph(case, seed))
        sub.arrays.pop("ws")
        s.update(_mean_inputs(case, seed, sub.n_sub))
        size = api.hg_layer_fwd_workspace_size if kind == "mean_fwd" else api.hg_layer_bwd_workspace_size
        s["ws"] = torch.empty(size(sub, case["d"], _dtype(case)), dtype=torch.uint8, device=DEV)
        s["out"] = torch.empty_like(s["H"])
        if kind == "mean_fwd":
            s["mask"] = torch.empty((sub.n_sub, case["d"] // 32), dtype=torch.int32, device=DEV)
        else:
            s["dW"] = [torch.empty_like(s[k]) for k in ("W_rel", "W_self", "bias")]
    elif kind == "hgt":
        sub = s["sub"] = _build(case, seed, _graph(case, seed))
        sub.arrays.pop("ws")
        s.update(_hgt_inputs(case, seed, sub.n_sub))
        d, S, lean = case["d"], case["heads"], case["lean"]
        s["out"], s["dH"] = torch.empty_like(s["H"]), torch.empty_like(s["H"])
        s["mask"] = torch.empty((sub.n_sub, d // 32), dtype=torch.int32, device=DEV)
        s["saved"] = torch.empty(api.hg_hgt_saved_size(sub, d, S, lean), dtype=torch.uint8, device=DEV)
        s["ws"] = torch.empty(max(api.hg_hgt_fwd_workspace_size(sub, d, S, lean),
                                  api.hg_hgt_bwd_workspace_size(sub, d, S, lean)), dtype=torch.uint8, device=DEV)
        s["grads"] = {k: torch.empty_like(v) for k, v in s["W"].items()}
    elif kind == "align":
        s.update(_align_inputs(case, seed))
        s["dH"] = s["base"].clone()  # the rows outside the overlap stay the upstream gradient's
        s["loss"] = torch.empty(3, device=DEV)
        s["ws"] = torch.empty(api.hg_align_workspace_size(case["overlap"], case["d"]), dtype=torch.uint8, device=DEV)
    else:
        s.update(_temporal_inputs(case, seed))
        s["out"], s["dh"] = torch.empty_like(s["h"]), torch.empty_like(s["h"])
        s["dC"] = [torch.empty_like(s["h"]) for _ in s["C"]]
        s["grads"] = {k: torch.empty_like(v) for k, v in s["W"].items()}
        s["ws"] = torch.empty(max(1, api.hg_temporal_bwd_workspace_size(case["rows"], case["d"], case["window"])),
                              dtype=torch.uint8, device=DEV)
    return s


# ---- one pass ---------------------------------------------------------------

BUILD_OUT = ("local2global", "global2local", "type_off", "overlap", "overlap_home", "overlap_rel", "csr_ptr",
             "csr_col", "csc_ptr", "csc_row", "csc_scale")


def run(s):
    kind = s["kind"]
    if kind == "step":
        inp = s["inp"]
        res = runner.run_step(inp)
        out = dict(loss=res.loss, dH0=res.dH0, grads=res.grads, weights=inp.weights)
        if inp.head is not None:
            out.update(loss_bce=inp.loss_bce, head=inp.head, head_grads=inp.head_grads)
        return out
    case, sub = s["case"], s.get("sub")
    if kind == "build":
        _build(case, s["seed"], s["g"], ws=s["ws"], out=sub)
        return dict({k: sub.arrays[k] for k in BUILD_OUT}, sizes=[sub.n_sub, sub.e_sub, sub.m_sel])
    if kind == "mean_fwd":
        H, mask = api.hg_layer_fwd(sub, s["H"], s["W_rel"], s["W_self"], s["bias"], H_out=s["out"], saved=s["mask"],
                                   ws=s["ws"])
        return dict(H=H, mask=mask)
    if kind == "mean_bwd":
        dH, dW_rel, dW_self, dbias = api.hg_layer_bwd(
            sub, s["H"], s["W_rel"], s["W_self"], s["mask"], s["G"], dH_in=s["out"], dW_rel=s["dW"][0],
            dW_self=s["dW"][1], dbias=s["dW"][2], ws=s["ws"])
        return dict(dH=dH, dW_rel=dW_rel, dW_self=dW_self, dbias=dbias)
    if kind == "hgt":
        # an output layer, without the ReLU: forward and backward of the pair
        lean = case["lean"]
        H, mask, saved = api.hg_hgt_fwd(sub, s["H"], s["W"], case["heads"], relu=False, H_out=s["out"],
                                        mask=s["mask"], saved=s["saved"], ws=s["ws"], lean=lean)
        dH, grads = api.hg_hgt_bwd(sub, s["H"], s["W"], case["heads"], mask, saved, s["G"], relu=False, dH_in=s["dH"],
                                   grads=s["grads"], ws=s["ws"], lean=lean)
        return dict(H=H, dH=dH, grads=grads)
    if kind == "align":
        api.hg_align_loss_fwd_bwd(s["H"], s["overlap"], s["ref"], s["dH"], w=s["w"], loss3=s["loss"], ws=s["ws"],
                                  dH_base=s["base"])
        return dict(loss=s["loss"], dH=s["dH"])
    H = api.hg_temporal_fwd(s["h"], s["C"], s["W"], H=s["out"])
    for t in s["dC"]:
        t.zero_()  # the state gradients are added into
    dh, grads = api.hg_temporal_bwd(s["h"], s["C"], s["W"], s["dH"], dh=s["dh"], dstates=s["dC"], grads=s["grads"],
                                    ws=s["ws"])
    return dict(H=H, dh=dh, dC=s["dC"], grads=grads)


# ---- what a pass cannot do without -------------------------------------------

def _sub_size(case):
    """(nodes, edges) that the subgraph keeps, about: every edge with both ends
    in the base set or its overlap (the overlap's nodes have few out-edges)."""
    n, e = case["nodes"], case["edges"]
    base = n / case["parts"] if case["parts"] else case["base"]
    ns = min(n, base + case["budget"])
    return ns, e * ns / n * (base / n if case["parts"] else 1.0)


def work(case):
    """Inputs read once and outputs written once; a multiply and an add per
    product of the transforms that are needed at least (one relation per row
    beside its own) and per edge and column."""
    kind = case["kind"]
    if kind == "step":
        cfg = synth.scaled(synth.WORKLOADS["tiny_" + case["model"]].graph, case["scale"])
        n, e, d = cfg.n_nodes, cfg.n_edges, 64
        return {"bytes": 9 * e + 5 * n + 2 * (4 * e + 6 * n * d * 4), "flops": 2 * 3 * (4 * n * d * d + 2 * e * d)}
    if kind == "build":
        n, e = case["nodes"], case["edges"]
        ns, es = _sub_size(case)
        return {"bytes": 9 * e + 9 * n + 4 * ns + 8 * ns * case["rels"] + 12 * es, "flops": 0}
    if kind in ("mean_fwd", "mean_bwd", "hgt"):
        d, R = case["d"], case["rels"]
        b = 2 if case.get("dtype") == "bf16" else 4
        n, e = _sub_size(case)
        row = n * d * b
        if kind == "mean_fwd":
            return {"bytes": 2 * row + n * d / 8 + 4 * (e + n * R) + 4 * (R + 2) * d * d,
                    "flops": 4 * n * d * d + 2 * e * d}
        if kind == "mean_bwd":
            return {"bytes": 3 * row + n * d / 8 + 8 * e + 4 * n * R + 8 * (R + 2) * d * d,
                    "flops": 8 * n * d * d + 2 * e * d}
        # projections and the aggregation forward, twice that backward; score and message per edge
        return {"bytes": 2 * row + 3 * row + 12 * e + 8 * n * R, "flops": 3 * (12 * n * d * d + 4 * e * d)}
    b = 2 if case["dtype"] == "bf16" else 4
    if kind == "align":
        m, d = case["overlap"], case["d"]
        return {"bytes": 4 * m * d * b + 4 * m, "flops": 6 * m * d * d}
    n, d, w = case["rows"], case["d"], case["window"]
    return {"bytes": n * d * b * ((w + 2) + (w + 3 + w)), "flops": 2 * n * d * d * ((w + 6) + 2 * (w + 6))}


# ---- outputs in float64 -------------------------------------------------------

def _splitmix(x):
    """First output of the SplitMix64 generator from state x (int64 bits)."""
    def i64(v):
        return v - (1 << 64) if v >> 63 else v

    def shift(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)
    z = x + i64(0x9E3779B97F4A7C15)
    z = (z ^ shift(z, 30)) * i64(0xBF58476D1CE4E5B9)
    z = (z ^ shift(z, 27)) * i64(0x94D049BB133111EB)
    return z ^ shift(z, 31)


def _select(src, dst, part, ntype, key, theta, budget, seed):
    """Global ids of the subgraph in local order, and which are overlap."""
    n = part.numel()
    deg = torch.bincount(src, minlength=n)
    base = part == 0
    keys = deg
    if key == api.HG_KEY_HINDEX:
        order = torch.argsort(src * (deg.max() + 1) + (deg.max() - deg[dst]))
        s, a = src[order], deg[dst][order]
        first = deg.cumsum(0) - deg
        rank = torch.arange(s.numel(), device=DEV) - first[s] + 1
        keys = torch.bincount(s[a >= rank], minlength=n)
    cand = torch.zeros(n, dtype=torch.bool, device=DEV)
    cand[src[base[dst]]] = True
    cand[dst[base[src]]] = True
    gid = torch.nonzero(cand & ~base & (keys <= theta)).flatten()
    h = _splitmix(seed ^ gid) ^ (-1 << 63)  # unsigned order
    order = torch.argsort(h, stable=True)
    order = order[torch.argsort(keys[gid][order], stable=True)]
    member = base.clone()
    member[gid[order[:budget]]] = True
    ids = torch.nonzero(member).flatten()
    ids = ids[torch.argsort(ntype[ids], stable=True)]
    return ids, ~base[ids]


def _local(case, seed, g=None):
    """The subgraph's nodes and edges (local ids, original edge order)."""
    g = _graph(case, seed) if g is None else g
    ids, over = _select(g["src"].long(), g["dst"].long(), g["part"], g["ntype"], case["key"], case["theta"],
                        case["budget"], seed)
    loc = torch.full((g["part"].numel(),), -1, dtype=torch.int64, device=DEV)
    loc[ids] = torch.arange(ids.numel(), device=DEV)
    src, dst = loc[g["src"].long()], loc[g["dst"].long()]
    keep = (src >= 0) & (dst >= 0)
    w = None if g["edge_w"] is None else g["edge_w"][keep].double()
    return dict(ids=ids, over=over, n=ids.numel(), src=src[keep], dst=dst[keep], rel=g["rel"][keep].long(), w=w,
                ntype=g["ntype"][ids].long(), R=case["rels"])


def _scale(L):
    """Mean weight of every edge, float64."""
    q = L["dst"] * L["R"] + L["rel"]
    deg = torch.bincount(q, minlength=L["n"] * L["R"])
    s = 1.0 / deg[q].double()
    return s if L["w"] is None else s * L["w"]


def _scatter(n, to, frm, scale, X):
    """out[to[e]] += scale[e] X[frm[e]] in float64."""
    out = torch.zeros((n, X.shape[1]), dtype=F64, device=DEV)
    step = max(1, (1 << 29) // X.shape[1])
    for at in range(0, to.numel(), step):
        c = slice(at, at + step)
        out.index_add_(0, to[c], X[frm[c]].double() * scale[c, None])
    return out


def _per_type(X, ntype, W, b=None):
    out = torch.empty((X.shape[0], W.shape[2]), dtype=F64, device=DEV)
    for t in range(W.shape[0]):
        rows = torch.nonzero(ntype == t).flatten()
        y = X[rows].double() @ W[t].double()
        out = out.index_copy(0, rows, y if b is None else y + b[t].double())
    return out


def _mean_fwd(L, H, W_rel, W_self, bias):
    scale = _scale(L)
    z = _per_type(H, L["ntype"], W_self, bias)
    for r in range(L["R"]):
        e = torch.nonzero(L["rel"] == r).flatten()
        z += _scatter(L["n"], L["dst"][e], L["src"][e], scale[e], H) @ W_rel[r].double()
    return z.clamp_(min=0) + H.double(), None


def _mean_bwd(L, s):
    H, G, R = s["H"], s["G"], L["R"]
    d = H.shape[1]
    bits = (s["mask"][:, :, None] >> torch.arange(32, dtype=torch.int32, device=DEV)) & 1
    dZ = G.double() * bits.reshape(-1, d)
    del bits
    scale = _scale(L)
    dH = G.double() + _per_type(dZ, L["ntype"], s["W_self"].transpose(1, 2))
    dW_rel = []
    for r in range(R):
        e = torch.nonzero(L["rel"] == r).flatten()
        src, dst, sc = L["src"][e], L["dst"][e], scale[e]
        dY = _scatter(L["n"], src, dst, sc, dZ)
        dW_rel.append(H.double().T @ dY)
        dH += dY @ s["W_rel"][r].double().T
        del dY
    dW_self, dbias = [], []
    for t in range(2):
        rows = torch.nonzero(L["ntype"] == t).flatten()
        dW_self.append(H[rows].double().T @ dZ[rows])
        dbias.append(dZ[rows].sum(0))
    return dict(dH=dH, dW_rel=torch.stack(dW_rel), dW_self=torch.stack(dW_self), dbias=torch.stack(dbias))


def _hgt_fwd(L, H, W, S, relu):
    """Attention layer in float64; differentiable."""
    n, d = H.shape
    dk = d // S
    K, Q, V = (_per_type(H, L["ntype"], W["W_" + k], W["b_" + k]) for k in "KQV")
    score, msg, dst = [], [], []
    for r in range(L["R"]):
        e = torch.nonzero(L["rel"] == r).flatten()
        i, j = L["src"][e], L["dst"][e]
        kt = torch.stack([K[:, h * dk:(h + 1) * dk] @ W["W_att"][r, h] for h in range(S)], 1)
        vt = torch.stack([V[:, h * dk:(h + 1) * dk] @ W["W_msg"][r, h] for h in range(S)], 1)
        mu = W["mu"][L["ntype"][i], r, L["ntype"][j]]
        score.append((kt[i] * Q.view(n, S, dk)[j]).sum(-1) * (mu / math.sqrt(dk))[:, None])
        msg.append(vt[i])
        dst.append(j)
    score, dst = torch.cat(score), torch.cat(dst)
    top = torch.full((n, S), -math.inf, dtype=F64, device=DEV)
    top = top.scatter_reduce(0, dst[:, None].expand(-1, S), score.detach(), "amax")
    ex = torch.exp(score - top[dst])
    den = torch.zeros((n, S), dtype=F64, device=DEV).index_add(0, dst, ex)
    alpha = ex / den[dst]
    ht = torch.zeros((n, S, dk), dtype=F64, device=DEV)
    at = 0
    for m in msg:
        c = slice(at, at + m.shape[0])
        ht = ht.index_add(0, dst[c], m * alpha[c][:, :, None])
        at += m.shape[0]
    z = _per_type(ht.view(n, d), L["ntype"], W["W_agg"], W["b_agg"])
    return (z.clamp(min=0) if relu else z) + H


def _align(H, overlap, ref, w, lambda_n=2e-4, eps=1e-5):
    """(L_inv, L_dec, L) with variances of divisor M."""
    m, d = ref.shape
    views = []
    for V in (H[overlap], ref):
        c = V - V.mean(0)
        views.append(c / torch.sqrt((c * c).mean(0) + eps) / math.sqrt(m))
    x, y = views
    diff = ((x - y) ** 2).sum(1)
    inv = diff.sum() if w is None else (diff * w.double()).sum()
    eye = torch.eye(d, dtype=F64, device=DEV)
    dec = ((x.T @ x - eye) ** 2).sum() + ((y.T @ y - eye) ** 2).sum()
    return torch.stack([inv, dec, inv + lambda_n * dec])


def _leaf(x):
    return {k: _leaf(v) for k, v in x.items()} if isinstance(x, dict) else x.double().requires_grad_()


def _exact_step(case, seed):
    """The losses of the step. A ReLU decision within rounding of zero may fall
    either way, and the gradients jump with it: they have no exact value."""
    wl = _step_workload(case, seed)
    cfg, mc = wl.graph, wl.model
    graph = synth.make_graph(cfg)
    g = {k: torch.from_numpy(getattr(graph, k)).to(DEV) for k in ("src", "dst", "rel", "ntype", "part")}
    L = _local(dict(rels=cfg.n_rel, key=cfg.key, theta=cfg.theta, budget=cfg.budget), cfg.seed, dict(g, edge_w=None))
    H = torch.from_numpy(synth.features(mc.seed, graph.n_nodes, mc.d)).to(DEV)[L["ids"]].double()
    for li in range(mc.n_layers):
        if mc.kind == "hgt":
            W = synth.hgt_weights(mc.seed, li, cfg.n_rel, 2, mc.d, mc.heads, mc.bias_range)
            H = _hgt_fwd(L, H, {k: torch.from_numpy(v).to(DEV).double() for k, v in W.items()}, mc.heads, True)
        else:
            W = synth.layer_weights(mc.seed, li, cfg.n_rel, 2, mc.d, mc.bias_range)
            H, _ = _mean_fwd(L, H, *(torch.from_numpy(w).to(DEV) for w in (W.w_rel, W.w_self, W.bias)))
    overlap = torch.nonzero(L["over"]).flatten()
    ref = torch.from_numpy(synth.reference_embeddings(mc.seed, max(1, overlap.numel()), mc.d)).to(DEV).double()
    out = dict(loss=_align(H, overlap, ref[:overlap.numel()], None))
    if mc.objective == "bce":
        y = torch.from_numpy(synth.labels(mc.seed, graph.ntype)).to(DEV)[L["ids"]]
        hw = {k: torch.from_numpy(v).to(DEV).double() for k, v in synth.head_weights(mc.seed, mc.d).items()}
        o = ((H @ hw["W1"] + hw["b1"]).clamp(min=0) @ hw["W2"] + hw["b2"])[:, 0]
        lab = y >= 0
        terms = torch.nn.functional.softplus(o[lab]) - y[lab].double() * o[lab]
        out["loss_bce"] = terms.mean()[None] if terms.numel() else torch.zeros(1, dtype=F64, device=DEV)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        return _exact_step(case, seed)
    if kind == "build":
        # the one computed number: w / deg in the order (source, relation, destination, edge)
        L = _local(case, seed)
        scale = _scale(L)
        row = L["src"] * L["R"] + L["rel"]
        order = torch.argsort(row * L["n"] + L["dst"], stable=True)
        out = torch.zeros(case["edges"], dtype=F64, device=DEV)
        out[:order.numel()] = scale[order]
        return dict({k: out if k == "csc_scale" else None for k in BUILD_OUT}, sizes=None)
    if kind in ("mean_fwd", "mean_bwd"):
        L = _local(case, seed)
        s = _mean_inputs(case, seed, L["n"])
        if kind == "mean_bwd":
            return _mean_bwd(L, s)
        H, mask = _mean_fwd(L, s["H"], s["W_rel"], s["W_self"], s["bias"])
        return dict(H=H, mask=mask)
    if kind == "hgt":
        L = _local(case, seed)
        s = _hgt_inputs(case, seed, L["n"])
        H, W = _leaf(s["H"]), _leaf(s["W"])
        out = _hgt_fwd(L, H, W, case["heads"], False)
        out.backward(s["G"].double())
        return dict(H=out.detach(), dH=H.grad, grads={k: v.grad for k, v in W.items()})
    if kind == "align":
        s = _align_inputs(case, seed)
        H = _leaf(s["H"])
        loss = _align(H, s["overlap"].long(), s["ref"].double(), s["w"])
        (dH,) = torch.autograd.grad(loss[2], H)
        return dict(loss=loss.detach(), dH=s["base"].double() + 0.1 * dH)
    s = _temporal_inputs(case, seed)
    h, C, W = _leaf(s["h"]), [_leaf(c) for c in s["C"]], _leaf(s["W"])
    Ht = torch.zeros_like(h)
    if C:
        sc = torch.stack([torch.tanh(c @ W["Q"].T) @ W["r"] for c in C], 1).softmax(1)
        Ht = sum(sc[:, k:k + 1] * c for k, c in enumerate(C))
    gi = [h @ W["Wi"][k] + W["bi"][k] for k in range(3)]
    gh = [Ht @ W["Wh"][k] + W["bh"][k] for k in range(3)]
    r, z = torch.sigmoid(gi[0] + gh[0]), torch.sigmoid(gi[1] + gh[1])
    H = (1 - z) * torch.tanh(gi[2] + r * gh[2]) + z * Ht
    H.backward(s["dH"].double())
    zero = torch.zeros_like
    return dict(H=H.detach(), dh=h.grad, dC=[c.grad for c in C],
                grads={k: v.grad if v.grad is not None else zero(v) for k, v in W.items()})


def tolerance(case):
    """Floats of 32 bits: sums in another order and products of another split.
    bfloat16: one rounding of a result. A step: a ReLU decision within rounding
    of zero that falls the other way changes a few gradient rows."""
    if case["kind"] == "build":
        return "exact"
    if case["kind"] == "step":
        return {"rel": 5e-3, "max": 0.5}
    if case.get("dtype") == "bf16":
        return {"rel": 5e-3, "max": 3e-2, "differ": 5e-3}
    # weight gradients are float32 sums over the rows: their error grows with them (1.7e-5 at 10M rows)
    rows = case["nodes"] if case["kind"] == "mean_bwd" else 0
    return {"rel": 1e-5 * max(1.0, rows / 1.5e6), "max": 1e-3, "differ": 1e-4}
