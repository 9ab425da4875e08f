"""The measured work of the framework: graph steps as a user's program makes them.

Each case names a kind of call sequence, its sizes and its options:

* ``step``       graph build + GCN normalisation + sum aggregation (a new graph every pass)
* ``train``      aggregation and its gradients on a cached graph (sum, mean or max)
* ``propagate``  K steps of APPNP on a cached graph
* ``gat``        the fused additive attention layer on a cached graph (inference)
* ``gat_train``  the attention layer with its coefficients kept, and its gradients
* ``dot``        the fused scaled dot-product attention layer
* ``batch``      a mini-batch training step over many small graphs

Graphs are drawn on the device from the seed: ``uniform`` (random endpoint pairs, both
directions), ``power`` (Chung-Lu with weight 1 / (i + 850.2), both directions) and ``attach``
(preferential attachment: every new node links to m older ones, node i of the first v being
picked with density ~ i^-1/2). Node ids are relabelled and edges shuffled.
"""

import math

import torch

import paper_2101_11552_amd as tfg

DEV = "cuda"
SLOPE = 0.2  # LeakyReLU slope of the additive attention score


def listed():
    return [
        # a citation-graph-sized GCN layer, its graph new on every call: launches and latency
        {"name": "step_small", "kind": "step", "graph": "uniform", "N": 2708, "E": 10556, "F": 64,
         "index": "int64", "weighted": False},
        # a citation graph with edge weights and its raw bag-of-words features (500 columns)
        {"name": "step_weighted", "kind": "step", "graph": "uniform", "N": 19717, "E": 88648,
         "F": 500, "index": "int64", "weighted": True},
        # the headline workload: a social graph of 114.6M edges, build + normalise + aggregate
        {"name": "step_large", "kind": "step", "graph": "power", "N": 232965, "E": 114600000,
         "F": 128, "index": "int32", "weighted": False},
        # the hidden layer (16 columns) of a GCN trained on a cached citation graph
        {"name": "train_small", "kind": "train", "graph": "uniform", "N": 2708, "E": 10556,
         "F": 16, "reduce": "sum", "weighted": True, "dw": False, "index": "int64"},
        # a mean-aggregating layer on a co-purchase-like graph with 100 features
        {"name": "train_mean", "kind": "train", "graph": "power", "N": 400000, "E": 10000000,
         "F": 100, "reduce": "mean", "weighted": False, "dw": False, "index": "int64"},
        # a max-aggregating layer (with its argmax) on a social graph
        {"name": "train_max", "kind": "train", "graph": "power", "N": 232965, "E": 23000000,
         "F": 64, "reduce": "max", "weighted": False, "dw": False, "index": "int32"},
        # APPNP smooths class scores (40 classes) over a paper-citation graph, 10 steps
        {"name": "propagate_classes", "kind": "propagate", "graph": "uniform", "N": 169343,
         "E": 2315598, "F": 40, "K": 10, "index": "int64"},
        # attention inference on a preferential-attachment graph, 8 heads of 16
        {"name": "gat_medium", "kind": "gat", "graph": "attach", "N": 169343, "E": 1185352,
         "H": 8, "D": 16, "index": "int64"},
        # attention inference on the social graph, 8 heads of 8
        {"name": "gat_large", "kind": "gat", "graph": "power", "N": 232965, "E": 114600000,
         "H": 8, "D": 8, "index": "int32"},
        # one attention layer of a training step, coefficients and their gradients kept
        {"name": "gat_train", "kind": "gat_train", "graph": "attach", "N": 169343, "E": 1185352,
         "H": 8, "D": 16, "index": "int64"},
        # Transformer-style attention on a denser graph, 4 heads of 32
        {"name": "dot_medium", "kind": "dot", "graph": "power", "N": 100000, "E": 3000000,
         "H": 4, "D": 32, "index": "int64"},
        # graph classification: 4,096 small graphs batched, three layers, three pools, gradients
        {"name": "batch_train", "kind": "batch", "G": 4096, "F": 64, "index": "int64"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _features(rng, lo, hi):
    """Feature counts: any in the range, half of them a multiple of 8 as hidden layers have."""
    f = _log(rng, lo, hi)
    return f if rng.random() < 0.5 else max(8, f // 8 * 8)


def draw(rng):
    kind = rng.choice(["step", "step", "train", "train", "train", "propagate", "gat", "gat_train",
                       "dot", "batch"])
    index = rng.choice(["int32", "int64"])
    graph = rng.choice(["uniform", "power"])
    if kind == "batch":
        return {"kind": kind, "G": _log(rng, 64, 4096), "F": _features(rng, 16, 64),
                "index": index}
    N = _log(rng, 2000, 232965)
    E = int(N * math.exp(rng.uniform(math.log(3.0), math.log(200.0)))) // 2 * 2
    if kind == "step":
        return {"kind": kind, "graph": graph, "N": N, "E": E, "F": _features(rng, 16, 128),
                "index": index, "weighted": rng.random() < 0.4}
    if kind == "train":
        reduce = rng.choice(["sum", "mean", "max"])
        weighted = reduce == "sum" and rng.random() < 0.7
        return {"kind": kind, "graph": graph, "N": N, "E": E // 2, "F": _features(rng, 16, 128),
                "reduce": reduce, "weighted": weighted, "dw": weighted and rng.random() < 0.5,
                "index": index}
    if kind == "propagate":
        return {"kind": kind, "graph": graph, "N": N, "E": N * rng.randint(3, 40) // 2 * 2,
                "F": _log(rng, 7, 70), "K": rng.randint(2, 10), "index": index}
    H = rng.choice([1, 2, 4, 8])
    if kind == "gat":
        return {"kind": kind, "graph": rng.choice(["uniform", "power", "attach"]), "N": N, "E": E,
                "H": H, "D": rng.choice([7, 8, 16, 16, 24, 32]), "index": index}
    if kind == "gat_train":  # at most 13 edges a node: the graph order is the plain CSR
        return {"kind": kind, "graph": rng.choice(["uniform", "power", "attach"]), "N": N,
                "E": N * rng.randint(2, 13) // 2 * 2, "H": H,
                "D": rng.choice([8, 16, 16, 32]), "index": index}
    return {"kind": kind, "graph": graph, "N": N, "E": E // 2, "H": H,
            "D": rng.choice([8, 16, 32]), "index": index}


# ---- inputs -------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 101)
    return g


def _endpoints(case, n, gen):
    u = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64)
    N = case["N"]
    if case["graph"] == "power":  # inverse of the weights' cumulative log
        off = 850.2
        i = off * ((N + off) / off) ** u - off
    else:
        i = u * N
    return i.to(torch.int64).clamp_(0, N - 1).to(torch.int32)


def _edges(case, gen):
    N, E = case["N"], case["E"]
    if case["graph"] == "attach":
        m = max(1, round(E / N))
        v = torch.arange(E, device=DEV) // m + m  # the new node of each link
        v.clamp_(max=N - 1)
        u = torch.rand(E, generator=gen, device=DEV, dtype=torch.float64)
        s, t = v.to(torch.int32), (v * u * u).to(torch.int64).clamp_(max=N - 1).to(torch.int32)
    else:
        a, b = _endpoints(case, E // 2, gen), _endpoints(case, E // 2, gen)
        s, t = torch.cat([a, b]), torch.cat([b, a])
    relabel = torch.randperm(N, generator=gen, device=DEV).to(torch.int32)
    order = torch.randperm(s.numel(), generator=gen, device=DEV)
    ei = torch.stack([relabel[s[order]], relabel[t[order]]])
    return ei.to(getattr(torch, case["index"]))


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float32)


def _batch(case, gen):
    """Local edge lists of G graphs of 10..60 nodes (every size as often, in a random order),
    one pair in ten, both directions."""
    G = case["G"]
    n = 10 + torch.randperm(G, generator=gen, device=DEV) % 51
    pairs = (n * (n - 1) // 20).clamp_(min=1)
    each = torch.repeat_interleave(n, pairs).to(torch.float64)
    u = torch.rand(2, each.numel(), generator=gen, device=DEV, dtype=torch.float64)
    a = (u[0] * each).to(torch.int64)
    b = (a + 1 + (u[1] * (each - 1)).to(torch.int64)) % each.to(torch.int64)
    local = torch.stack([torch.stack([a, b], 1).reshape(-1), torch.stack([b, a], 1).reshape(-1)])
    dt = getattr(torch, case["index"])
    return n.to(dt), (2 * pairs).to(dt), local.to(dt)


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    gen, kind = _gen(seed), case["kind"]
    if kind == "batch":
        nc, ec, local = _batch(case, gen)
        F, nb = case["F"], int(nc.sum())
        return {"nc": nc, "ec": ec, "local": local, "x": _normal(gen, nb, F),
                "dp": [_normal(gen, case["G"], F) for _ in range(3)]}
    d, N = {"ei": _edges(case, gen)}, case["N"]
    if kind in ("step", "train", "propagate"):
        d["x"] = _normal(gen, N, case["F"])
    if case.get("weighted"):
        d["w"] = torch.rand(d["ei"].shape[1], generator=gen, device=DEV) + 0.1
    if kind == "train":
        d["dy"] = _normal(gen, N, case["F"])
    if kind in ("gat", "gat_train"):
        H, D = case["H"], case["D"]
        d["x"] = _normal(gen, N, H * D)
        d["a_src"], d["a_dst"] = (0.3 * _normal(gen, H, D) for _ in range(2))
        if kind == "gat_train":
            d["dy"] = _normal(gen, N, H * D)
    if kind == "dot":
        F = case["H"] * case["D"]
        d["q"], d["k"], d["x"] = (_normal(gen, N, F) for _ in range(3))
    return d


def _cached(g):
    """A program that keeps the handle no longer needs the edge list it came from."""
    torch.cuda.synchronize()
    return g


def prepare(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    d["case"] = dict(case)
    if kind in ("step", "batch"):  # the graph itself is new on every pass
        return d
    N, ei = case["N"], d.pop("ei")
    loops = kind in ("propagate", "gat_train")
    d["g"] = _cached(tfg.tfg_graph_create(ei, N, add_self_loops=loops))
    if kind in ("train", "gat_train"):
        d["gt"] = _cached(tfg.tfg_graph_create_transposed(ei, N, add_self_loops=loops))
    if kind == "propagate":
        d["w"] = tfg.tfg_gcn_norm(ei, N, graph=d["g"], out_edge_index=False,
                                  out_edge_weight=False, out_deg=False)["edge_weight_csr"]
    elif case.get("weighted"):
        w = d.pop("w")
        d["w"] = tfg.tfg_edge_reorder(w, None, d["g"])
        d["wt"] = tfg.tfg_edge_reorder(w, None, d["gt"])
    return d


# ---- the measured pass --------------------------------------------------------------------------

def run(state):
    return _RUN[state["case"]["kind"]](state, state["case"])


def _run_step(s, case):
    N = case["N"]
    g = tfg.tfg_graph_create(s["ei"], N, add_self_loops=True)
    norm = tfg.tfg_gcn_norm(s["ei"], N, edge_weight=s.get("w"), graph=g)
    y = tfg.tfg_aggregate(norm["edge_index"], s["x"], N, edge_weight=norm["edge_weight_csr"],
                          weight_order="csr", graph=g)
    return {"edge_index": norm["edge_index"], "edge_weight": norm["edge_weight"],
            "edge_weight_csr": norm["edge_weight_csr"], "deg": norm["deg"], "y": y}


def _run_train(s, case):
    N, red = case["N"], case["reduce"]
    r = tfg.tfg_aggregate(None, s["x"], N, red, edge_weight=s.get("w"), weight_order="csr",
                          graph=s["g"])
    y, arg = r if red == "max" else (r, None)
    dx, dw = tfg.tfg_aggregate_backward(s["g"], s["dy"], red, graph_t=s["gt"], x=s["x"],
                                        edge_weight=s.get("wt"), weight_order="csr_t",
                                        argmax=arg, want_dw=case["dw"])
    return {"y": y, "argmax": arg, "dx": dx, "dw": dw}


def _run_propagate(s, case):
    return tfg.tfg_propagate(s["g"], s["x"], case["K"], alpha=0.1, h=s["x"], edge_weight=s["w"])


def _run_gat(s, case):
    return tfg.tfg_gat_aggregate(s["g"], s["x"], s["a_src"], s["a_dst"], SLOPE)


def _run_gat_train(s, case):
    g, x = s["g"], s["x"]
    scores = tfg.tfg_gat_graph_scores(g, x, s["a_src"], s["a_dst"], SLOPE)
    alpha = tfg.tfg_segment_softmax_graph(g, scores)
    y = tfg.tfg_aggregate(None, x, case["N"], edge_weight=alpha, heads=case["H"],
                          weight_order="csr", graph=g)
    dx, dalpha = tfg.tfg_aggregate_backward(g, s["dy"], graph_t=s["gt"], x=x, edge_weight=alpha,
                                            heads=case["H"], weight_order="csr", want_dw=True,
                                            dw_order="csr")
    ds = tfg.tfg_segment_softmax_graph_backward(g, alpha, dalpha)
    return {"alpha": alpha, "y": y, "dx": dx, "dalpha": dalpha, "ds": ds}


def _run_dot(s, case):
    return tfg.tfg_gat_dot_aggregate(s["g"], s["q"], s["k"], s["x"], case["H"])


def _run_batch(s, case):
    ei, gi, _, _ = tfg.tfg_batch_graphs(s["nc"], s["ec"], s["local"])
    N, G = gi.shape[0], case["G"]
    g = tfg.tfg_graph_create(ei, N, add_self_loops=True)
    gt = tfg.tfg_graph_create_transposed(ei, N, add_self_loops=True)
    norm = tfg.tfg_gcn_norm(ei, N, graph=g, out_edge_index=False, out_deg=False)
    wt = tfg.tfg_edge_reorder(norm["edge_weight"], None, gt)
    # the readout joins the input's maximum, the second layer's mean and the last layer's sum
    top, arg = tfg.tfg_segment_pool(s["x"], gi, G, "max", validate=False)
    hs = [s["x"]]
    for _ in range(3):
        hs.append(tfg.tfg_aggregate(None, hs[-1], N, edge_weight=norm["edge_weight_csr"],
                                    weight_order="csr", graph=g))
    pools = [top, tfg.tfg_segment_pool(hs[2], gi, G, "mean", validate=False),
             tfg.tfg_segment_pool(hs[3], gi, G, "sum", validate=False)]

    def back(d):
        return tfg.tfg_aggregate_backward(g, d, graph_t=gt, edge_weight=wt,
                                          weight_order="csr_t")[0]

    dtop, dmean, dsum = s["dp"]
    d = back(tfg.tfg_segment_pool_backward(dsum, gi, "sum", validate=False))
    d = back(back(d + tfg.tfg_segment_pool_backward(dmean, gi, "mean", validate=False)))
    d = d + tfg.tfg_segment_pool_backward(dtop, gi, "max", argmax=arg, validate=False)
    return {"edge_index": ei, "graph_index": gi, "h": hs[3], "pools": pools, "argmax": arg,
            "dx": d}


_RUN = {"step": _run_step, "train": _run_train, "propagate": _run_propagate, "gat": _run_gat,
        "gat_train": _run_gat_train, "dot": _run_dot, "batch": _run_batch}


# ---- what a pass cannot do without --------------------------------------------------------------

def work(case):
    """Bytes: every input read once and every output written once (a cached graph is two words
    an edge: the source id and the row it belongs to, counted as one word plus row starts)."""
    kind = case["kind"]
    if kind == "batch":
        n, e, F = 35 * case["G"], 140 * case["G"], case["F"]
        i = 8 if case["index"] == "int64" else 4
        return {"bytes": 4 * e * i + n * i + 4 * F * (3 * n + 6 * case["G"]) + 4 * F * case["G"],
                "flops": 12 * (e + n) * F + 6 * n * F}
    N, E = case["N"], case["E"]
    i = 8 if case["index"] == "int64" else 4
    if kind == "step":
        F, Ep = case["F"], E + N
        w = 4 * E if case["weighted"] else 0
        return {"bytes": 2 * i * E + w + 16 * Ep + 4 * N + 8 * N * F, "flops": 2 * Ep * (F + 1)}
    if kind == "train":
        F = case["F"]
        per_edge = 8 + (8 if case["weighted"] else 0) + (4 if case["dw"] else 0)
        arg = 4 * N * F if case["reduce"] == "max" else 0
        return {"bytes": per_edge * E + 8 * N + 16 * N * F + arg,
                "flops": (4 + (2 if case["dw"] else 0)) * E * F}
    if kind == "propagate":
        F, Ep = case["F"], E + N
        return {"bytes": 8 * Ep + 4 * N + 8 * N * F, "flops": case["K"] * (2 * Ep * F + 3 * N * F)}
    H, F = case["H"], case["H"] * case["D"]
    if kind == "gat":
        return {"bytes": 4 * E + 4 * N + 8 * N * F, "flops": E * (2 * F + 6 * H) + 4 * N * F}
    if kind == "dot":
        return {"bytes": 4 * E + 4 * N + 16 * N * F, "flops": E * (4 * F + 6 * H)}
    Ep = E + N
    return {"bytes": 8 * Ep + 12 * Ep * H + 16 * N * F,
            "flops": Ep * (6 * F + 12 * H) + 4 * N * F}


def tolerance(case):
    """About four times the difference from the same sums in 64 bits (whole values are exact)."""
    return _TOLERANCE[case["kind"]]


# Measured against exact() over the listed cases and drawn ones: relative error of up to 1e-7 in
# every kind; where a score's rounding passes through the exponential it grows with the scores.
# The largest single difference is at hub rows, whose many terms nearly cancel in a few columns.
_TOLERANCE = {
    "step": {"rel": 5e-7, "max": 2e-5},
    "train": {"rel": 5e-7, "max": 2e-5},
    "propagate": {"rel": 5e-7, "max": 2e-5},
    "gat": {"rel": 1e-6, "max": 4e-5},
    "gat_train": {"rel": 1e-6, "max": 4e-5},
    "dot": {"rel": 1e-6, "max": 4e-5},
    "batch": {"rel": 5e-7, "max": 2e-5},
}


# ---- the same results in 64 bits ----------------------------------------------------------------

def exact(case, seed):
    d = _inputs(case, seed)
    return _EXACT[case["kind"]](d, case)


def _columns(E, F):
    """Column ranges whose per-edge products fit comfortably."""
    c = max(1, min(F, int(1.5e9) // max(E, 1)))
    return [(f, min(f + c, F)) for f in range(0, F, c)]


def _sum64(s, t, w, x, N):
    """out[t] += w * x[s]; w [E], [E, H] (one weight per head) or None."""
    F = x.shape[1]
    out = torch.zeros(N, F, dtype=torch.float64, device=DEV)
    for a, b in _columns(s.numel(), F):
        m = x[:, a:b].double()[s]
        if w is not None and w.dim() == 1:
            m *= w[:, None]
        elif w is not None:
            m *= w[:, torch.arange(a, b, device=DEV) // (F // w.shape[1])]
        out[:, a:b] = torch.zeros(N, b - a, dtype=torch.float64, device=DEV).index_add_(0, t, m)
    return out


def _dot64(s, t, x, y, H):
    """<y[t], x[s]> per edge and head."""
    D = x.shape[1] // H
    out = torch.empty(s.numel(), H, dtype=torch.float64, device=DEV)
    step = max(1, int(1e9) // x.shape[1])
    for a in range(0, s.numel(), step):
        b = min(a + step, s.numel())
        out[a:b] = (x[s[a:b]].double() * y[t[a:b]].double()).view(b - a, H, D).sum(2)
    return out


def _softmax64(t, sc, N):
    H = sc.shape[1]
    m = torch.full((N, H), -math.inf, dtype=torch.float64, device=DEV)
    m.scatter_reduce_(0, t[:, None].expand(-1, H), sc, "amax")
    e = torch.exp(sc - m[t])
    den = torch.zeros(N, H, dtype=torch.float64, device=DEV).index_add_(0, t, e)
    return e / den[t]


def _ends(d, N, loops):
    s, t = d["ei"][0].long(), d["ei"][1].long()
    if loops:
        i = torch.arange(N, device=DEV)
        s, t = torch.cat([s, i]), torch.cat([t, i])
    return s, t


def _norm64(s, t, N, w=None):
    w = torch.ones(s.numel(), dtype=torch.float64, device=DEV) if w is None else w
    deg = torch.zeros(N, dtype=torch.float64, device=DEV).index_add_(0, t, w)
    inv = torch.where(deg > 0, deg.rsqrt(), torch.zeros_like(deg))
    return deg, inv[s] * w * inv[t]


def _exact_step(d, case):
    N = case["N"]
    s, t = _ends(d, N, True)
    w = None
    if "w" in d:
        w = torch.cat([d["w"].double(), torch.ones(N, dtype=torch.float64, device=DEV)])
    deg, w = _norm64(s, t, N, w)
    return {"edge_index": None, "edge_weight": w, "edge_weight_csr": None, "deg": deg,
            "y": _sum64(s, t, w, d["x"], N)}


def _exact_train(d, case):
    N, red = case["N"], case["reduce"]
    s, t = _ends(d, N, False)
    E, F = s.numel(), case["F"]
    if red == "max":
        y, dx = (torch.zeros(N, F, dtype=torch.float64, device=DEV) for _ in range(2))
        ids = torch.arange(E, device=DEV)
        for a, b in _columns(2 * E, F):
            m, tt = d["x"][:, a:b][s], t[:, None].expand(-1, b - a)
            top = torch.full((N, b - a), -math.inf, device=DEV).scatter_reduce_(0, tt, m, "amax")
            won = torch.where(m == top[t], ids[:, None].expand(-1, b - a), E)
            arg = torch.full((N, b - a), E, device=DEV).scatter_reduce_(0, tt, won, "amin")
            has = arg < E
            y[:, a:b] = torch.where(has, top.double(), 0.0)
            dx[:, a:b].scatter_add_(0, s[arg.clamp(max=E - 1)],
                                    torch.where(has, d["dy"][:, a:b].double(), 0.0))
        return {"y": y, "argmax": None, "dx": dx, "dw": None}
    w = d["w"].double() if "w" in d else None
    y, dy = _sum64(s, t, w, d["x"], N), d["dy"].double()
    if red == "mean":
        deg = torch.bincount(t, minlength=N).clamp_(min=1).double()[:, None]
        y, dy = y / deg, dy / deg
    dw = _dot64(s, t, d["x"], dy, 1) if case["dw"] else None
    return {"y": y, "argmax": None, "dx": _sum64(t, s, w, dy, N), "dw": dw}


def _exact_propagate(d, case):
    N = case["N"]
    s, t = _ends(d, N, True)
    _, w = _norm64(s, t, N)
    h = d["x"].double()
    z = h
    for _ in range(case["K"]):
        z = 0.9 * _sum64(s, t, w, z, N) + 0.1 * h
    return z


def _gat_alpha64(d, case, s, t):
    N, H, D = case["N"], case["H"], case["D"]
    h = d["x"].double().view(N, H, D)
    z = (h * d["a_src"].double()).sum(2)[s] + (h * d["a_dst"].double()).sum(2)[t]
    return _softmax64(t, torch.where(z >= 0, z, z * float(torch.tensor(SLOPE))), N)


def _exact_gat(d, case):
    s, t = _ends(d, case["N"], False)
    return _sum64(s, t, _gat_alpha64(d, case, s, t), d["x"], case["N"])


def _exact_gat_train(d, case):
    N, H = case["N"], case["H"]
    s, t = _ends(d, N, True)
    t, order = torch.sort(t, stable=True)  # the graph order: targets, input order in each
    s = s[order]
    alpha = _gat_alpha64(d, case, s, t)
    dalpha = _dot64(s, t, d["x"], d["dy"], H)
    mean = torch.zeros(N, H, dtype=torch.float64, device=DEV).index_add_(0, t, alpha * dalpha)
    return {"alpha": alpha, "y": _sum64(s, t, alpha, d["x"], N),
            "dx": _sum64(t, s, alpha, d["dy"], N), "dalpha": dalpha,
            "ds": alpha * (dalpha - mean[t])}


def _exact_dot(d, case):
    s, t = _ends(d, case["N"], False)
    sc = _dot64(s, t, d["k"], d["q"], case["H"]) / math.sqrt(case["D"])
    return _sum64(s, t, _softmax64(t, sc, case["N"]), d["x"], case["N"])


def _exact_batch(d, case):
    n, e, G = d["nc"].long(), d["ec"].long(), case["G"]
    ids = torch.arange(G, device=DEV)
    gi, ge = torch.repeat_interleave(ids, n), torch.repeat_interleave(ids, e)
    N = gi.numel()
    off = torch.cumsum(n, 0) - n
    loops = torch.arange(N, device=DEV)
    s = torch.cat([d["local"][0].long() + off[ge], loops])
    t = torch.cat([d["local"][1].long() + off[ge], loops])
    _, w = _norm64(s, t, N)
    h2 = _sum64(s, t, w, _sum64(s, t, w, d["x"], N), N)
    h3 = _sum64(s, t, w, h2, N)
    F, cnt, x = case["F"], n.double()[:, None], d["x"].double()
    zero = torch.zeros(G, F, dtype=torch.float64, device=DEV)
    top = torch.full((G, F), -math.inf, dtype=torch.float64, device=DEV)
    top = top.scatter_reduce_(0, gi[:, None].expand(-1, F), x, "amax")
    dtop, dmean, dsum = (p.double() for p in d["dp"])
    dh = _sum64(t, s, w, dsum[gi], N) + (dmean / cnt)[gi]
    dh = _sum64(t, s, w, _sum64(t, s, w, dh, N), N)
    # (equal maxima in one graph and column are left to the whole-value comparison of argmax)
    dh = dh + torch.where(x == top[gi], dtop[gi], 0.0)
    return {"edge_index": None, "graph_index": None, "h": h3, "argmax": None,
            "pools": [top, zero.index_add(0, gi, h2) / cnt, zero.index_add(0, gi, h3)], "dx": dh}


_EXACT = {"step": _exact_step, "train": _exact_train, "propagate": _exact_propagate,
          "gat": _exact_gat, "gat_train": _exact_gat_train, "dot": _exact_dot,
          "batch": _exact_batch}
