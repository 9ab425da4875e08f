"""The slot aggregation at the sizes where it can go wrong: every row length around its lists'
and rounds' edges, every width around its lane layouts, both plans, with a leading dimension
that leaves rows at dword alignment only. Sums against the oracle at the scaled 1e-5 bound of
float32 chains (a few hundred units of 2^-24), maxima and argmax bit for bit."""

import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 127, 128, 129, 200,
           256, 257, 700]
WIDTHS = [1, 2, 3, 4, 5, 7, 15, 16, 17, 31, 33, 40, 63, 64, 65, 100, 128, 130, 255, 257, 300]


@pytest.fixture(scope="module")
def tfg():
    import paper_2101_11552_amd as m
    m.load()
    return m


def _graph(seed, n_src, repeat):
    """Rows of every length in LENGTHS, `repeat` times, in a random order of rows and edges."""
    r = np.random.default_rng(seed)
    deg = r.permutation(np.repeat(LENGTHS, repeat))
    tgt = np.repeat(np.arange(deg.size), deg)
    src = r.integers(0, n_src, tgt.size)
    order = r.permutation(tgt.size)
    return np.stack([src[order], tgt[order]]).astype(np.int64), deg.size


def _check(orc, ei, x, n, res, reduce, w, heads):
    if reduce == "max":
        ref, arg = orc.aggregate(ei, x, n, "max", edge_weight=w, heads=heads)
        assert np.array_equal(res[0].cpu().numpy().view(np.uint32), ref.view(np.uint32))
        assert np.array_equal(res[1].cpu().numpy(), arg)
    else:
        ref, scale = orc.aggregate(ei, x, n, reduce, edge_weight=w, heads=heads)
        err = np.abs(res.cpu().numpy().astype(np.float64) - ref) / np.maximum(scale, 1e-300)
        assert float(err.max()) <= 1e-5


@pytest.mark.parametrize("plan", ["0", "1"])
@pytest.mark.parametrize("F", WIDTHS)
def test_row_lengths_and_widths(tfg, orc, monkeypatch, F, plan):
    monkeypatch.setenv("TFG_PART_PLAN", plan)
    ei, n = _graph(F, 500, 3)
    r = np.random.default_rng([7, F])
    big = r.standard_normal((500, F + 3)).astype(np.float32)
    big[:, :F][r.random((500, F)) < 0.2] = 0.0  # equal maxima
    x = np.ascontiguousarray(big[:, :F])
    xd = torch.from_numpy(big).cuda()[:, :F]
    w = r.standard_normal(ei.shape[1]).astype(np.float32)
    g = tfg.tfg_graph_create(torch.from_numpy(ei).cuda(), n, N_src=500,
                             src_parts=4 if plan == "1" else 3)
    for reduce in ("sum", "mean", "max"):
        for weight in (None, w):
            wd = None if weight is None else torch.from_numpy(weight).cuda()
            res = tfg.tfg_aggregate(None, xd, n, reduce, edge_weight=wd, graph=g)
            _check(orc, ei, x, n, res, reduce, weight, 1)


@pytest.mark.parametrize("plan", ["0", "1"])
@pytest.mark.parametrize("H,D", [(2, 1), (2, 6), (3, 7), (4, 4), (8, 8), (8, 16), (5, 20), (16, 32)])
def test_heads(tfg, orc, monkeypatch, H, D, plan):
    monkeypatch.setenv("TFG_PART_PLAN", plan)
    ei, n = _graph(100 + H * D, 400, 2)
    r = np.random.default_rng([8, H, D])
    x = r.standard_normal((400, H * D)).astype(np.float32)
    w = r.standard_normal((ei.shape[1], H)).astype(np.float32)
    g = tfg.tfg_graph_create(torch.from_numpy(ei).cuda(), n, N_src=400, src_parts=2)
    wd = torch.from_numpy(w).cuda()
    for order, weight in (("coo", wd), ("csr", tfg.tfg_edge_reorder(wd, None, g))):
        for reduce in ("sum", "max"):
            res = tfg.tfg_aggregate(None, torch.from_numpy(x).cuda(), n, reduce,
                                    edge_weight=weight, heads=H, weight_order=order, graph=g)
            _check(orc, ei, x, n, res, reduce, w, H)


@pytest.mark.parametrize("plan", ["0", "1"])
@pytest.mark.parametrize("F", [1, 3, 4, 7, 16, 33, 64, 100, 130, 257])
def test_max_gradient(tfg, orc, monkeypatch, F, plan):
    monkeypatch.setenv("TFG_PART_PLAN", plan)
    ei, n = _graph(300 + F, 300, 2)
    r = np.random.default_rng([9, F])
    x = r.standard_normal((300, F)).astype(np.float32)
    dy = r.standard_normal((n, F)).astype(np.float32)
    w = r.standard_normal(ei.shape[1]).astype(np.float32)
    eid = torch.from_numpy(ei).cuda()
    g = tfg.tfg_graph_create(eid, n, N_src=300, src_parts=2)
    gt = tfg.tfg_graph_create_transposed(eid, n, N_src=300, src_parts=2)
    wd = torch.from_numpy(w).cuda()
    _, arg = tfg.tfg_aggregate(None, torch.from_numpy(x).cuda(), n, "max", edge_weight=wd, graph=g)
    dx, _ = tfg.tfg_aggregate_backward(g, torch.from_numpy(dy).cuda(), "max", graph_t=gt,
                                       edge_weight=wd, argmax=arg)
    a = arg.cpu().numpy()
    ref, _ = orc.aggregate_backward(ei, x, n, dy, "max", edge_weight=w, arg=a)
    # the scale of a masked sum: the same winners, with |w| and |dy|
    m = np.zeros_like(ref)
    for c in range(F):
        ok = a[:, c] >= 0
        e = a[ok, c]
        np.add.at(m[:, c], ei[0][e], np.abs(w[e].astype(np.float64) * dy[ok, c]))
    err = np.abs(dx.cpu().numpy() - ref) / np.maximum(m, 1e-300)
    assert float(np.where(m > 0, err, np.abs(ref)).max()) <= 1e-5


@pytest.mark.parametrize("plan", ["0", "1"])
@pytest.mark.parametrize("H,D", [(1, 1), (1, 2), (1, 4), (1, 8), (1, 16), (1, 32), (1, 64), (2, 2),
                                 (2, 8), (3, 8), (8, 8), (4, 32), (8, 16), (2, 64), (5, 24),
                                 (3, 6), (3, 7), (16, 32)])
def test_attention_rows(tfg, orc, monkeypatch, H, D, plan):
    """Both fused layers over rows of every length, whole or by source part, with the
    coefficients. Scores of about one unit: their float32 error (a few 1e-7) passes through
    the exponential unamplified and stays inside the 1e-5 bar of the sums and of alpha."""
    monkeypatch.setenv("TFG_PART_PLAN", plan)
    ei, n = _graph(500 + 70 * H + D, 30, 2)
    ei[0] = np.random.default_rng(D).integers(0, n, ei.shape[1])  # square
    r = np.random.default_rng([10, H, D])
    q, k, h = (r.standard_normal((n, H * D)).astype(np.float32) for _ in range(3))
    a_s, a_d = (0.5 * r.standard_normal((H, D)).astype(np.float32) for _ in range(2))
    g = tfg.tfg_graph_create(torch.from_numpy(ei).cuda(), n, src_parts=3)
    dv = [torch.from_numpy(t).cuda() for t in (q, k, h, a_s, a_d)]

    def check(res, ref):
        out, alpha, scale = ref
        err = np.abs(res[0].cpu().numpy() - out) / np.maximum(scale, 1e-300)
        assert float(err.max()) <= 1e-5
        rel = np.abs(res[1].cpu().numpy() - alpha) / np.maximum(alpha, 1e-30)
        assert float(rel.max()) <= 1e-5

    check(tfg.tfg_gat_aggregate(g, dv[2], dv[3], dv[4], 0.2, want_alpha=True),
          orc.gat_layer(ei, h, a_s, a_d, H, slope=np.float32(0.2)))
    if D & (D - 1) == 0:
        sc = np.float32(0.5 / np.sqrt(D))
        check(tfg.tfg_gat_dot_aggregate(g, *dv[:3], H, scale=float(sc), want_alpha=True),
              orc.dot_layer(ei, q, k, h, H, sc))


@pytest.mark.parametrize("plan", ["0", "1"])
@pytest.mark.parametrize("H,D", [(1, 1), (1, 3), (1, 7), (1, 16), (1, 33), (1, 64), (1, 100),
                                 (1, 256), (1, 300), (2, 2), (3, 5), (8, 16), (4, 24), (5, 20),
                                 (16, 32), (2, 258)])
def test_edge_gradients(tfg, orc, monkeypatch, H, D, plan):
    monkeypatch.setenv("TFG_PART_PLAN", plan)
    ei, n = _graph(700 + 11 * H + D, 200, 1)
    r = np.random.default_rng([11, H, D])
    F = H * D
    big = r.standard_normal((200, F + 1)).astype(np.float32)
    x = np.ascontiguousarray(big[:, :F])
    dy = r.standard_normal((n, F)).astype(np.float32)
    w = r.standard_normal((ei.shape[1], H)).astype(np.float32)
    g = tfg.tfg_graph_create(torch.from_numpy(ei).cuda(), n, N_src=200, src_parts=2)
    xd, dyd, wd = torch.from_numpy(big).cuda()[:, :F], torch.from_numpy(dy).cuda(), torch.from_numpy(w).cuda()
    perm = tfg.tfg_graph_csr(g)[2].cpu().numpy()
    for reduce in ("sum", "mean", "max"):
        a = ad = None
        if reduce == "max":
            _, ad = tfg.tfg_aggregate(None, xd, n, "max", edge_weight=wd, heads=H, graph=g)
            a = ad.cpu().numpy()
        _, ref = orc.aggregate_backward(ei, x, n, dy, reduce, edge_weight=w, heads=H, arg=a)
        _, scale = orc.aggregate_backward(ei, np.abs(x), n, np.abs(dy), reduce, edge_weight=w,
                                          heads=H, arg=a)
        for order in ("coo", "csr"):
            _, dw = tfg.tfg_aggregate_backward(g, dyd, reduce, x=xd, edge_weight=wd, heads=H,
                                               argmax=ad, want_dx=False, want_dw=True,
                                               dw_order=order)
            got = dw.cpu().numpy()
            want, s = (ref, scale) if order == "coo" else (ref[perm], scale[perm])
            err = np.abs(got - want) / np.maximum(s, 1e-300)
            assert float(np.where(s > 0, err, np.abs(got)).max()) <= 1e-5


@pytest.mark.parametrize("plan", ["0", "1"])
@pytest.mark.parametrize("H,D", [(1, 7), (1, 64), (4, 8)])
def test_max_weight_gradient_beside_infinities(tfg, monkeypatch, H, D, plan):
    """Entries of -inf, the usual filler before a maximum, lose and add nothing to the gradient
    of the weights: the same bits as with finite losers in their place."""
    monkeypatch.setenv("TFG_PART_PLAN", plan)
    ei, n = _graph(900 + D, 100, 1)
    r = np.random.default_rng([12, H, D])
    x = r.standard_normal((100, H * D)).astype(np.float32)
    drop = r.random(x.shape) < 0.3
    drop[ei[0][:: 7]] = False
    dy = torch.from_numpy(r.standard_normal((n, H * D)).astype(np.float32)).cuda()
    w = torch.from_numpy(r.uniform(0.5, 1.5, (ei.shape[1], H)).astype(np.float32)).cuda()
    g = tfg.tfg_graph_create(torch.from_numpy(ei).cuda(), n, N_src=100, src_parts=2)
    res = []
    for filler in (-np.inf, -1e4):
        xd = torch.from_numpy(np.where(drop, np.float32(filler), x)).cuda()
        y, a = tfg.tfg_aggregate(None, xd, n, "max", edge_weight=w, heads=H, graph=g)
        a = torch.where(y < -1e3, -1, a)  # rows that hold fillers alone: no winner
        res.append((a, tfg.tfg_aggregate_backward(g, dy, "max", x=xd, edge_weight=w, heads=H,
                                                  argmax=a, want_dx=False, want_dw=True)[1]))
    assert torch.equal(res[0][0], res[1][0])
    assert torch.equal(res[0][1], res[1][1])
    assert bool(torch.isfinite(res[0][1]).all())


def test_head_weights_beyond_2_gib(tfg):
    """Per-head weights whose byte offsets pass 2^31 (they stay below 2^32, the 32-bit path's
    limit): the last targets, whose weights lie there, against sums in 64 bits."""
    H, n, deg = 64, 1 << 16, 130
    E = n * deg  # 8.5M edges, 2.18 GB of weights
    assert 2**31 < 4 * E * H < 2**32
    gen = torch.Generator(device="cuda").manual_seed(13)
    src = torch.randint(0, 1000, (E,), generator=gen, device="cuda", dtype=torch.int32)
    tgt = torch.arange(n, device="cuda", dtype=torch.int32).repeat_interleave(deg)
    g = tfg.tfg_graph_create(torch.stack([src, tgt]), n, N_src=1000)
    x = torch.randn(1000, H, generator=gen, device="cuda")
    w = torch.rand(E, H, generator=gen, device="cuda")
    for order in ("csr", "coo"):  # the input is grouped by target: both orders are one
        y = tfg.tfg_aggregate(None, x, n, edge_weight=w, heads=H, weight_order=order, graph=g)
        last = slice(E - 50 * deg, E)
        m = w[last].double() * x[src[last].long()].double()
        ref = m.view(50, deg, H).sum(1)
        scale = m.abs().view(50, deg, H).sum(1)
        assert float(((y[-50:].double() - ref).abs() / scale).max()) <= 1e-5


@pytest.mark.parametrize("F", [1, 3, 4, 16, 33, 64, 130, 260])
@pytest.mark.parametrize("chunks", [[2, 3], [4, 5, 9], [2] * 40 + [70], [33, 65]])
def test_split_rows(tfg, orc, F, chunks):
    """Rows of many chunks (128 edges each), whose partials go over 4 to 16 slots of a wavefront by
    their average number, beside short ones: sums, means and maxima with their edges."""
    r = np.random.default_rng([14, F, len(chunks)])
    deg = np.array([128 * c - int(r.integers(0, 127)) for c in chunks] + [0, 3, 20])
    tgt = np.repeat(np.arange(deg.size), deg)
    ei = np.stack([r.integers(0, 300, tgt.size), tgt])[:, r.permutation(tgt.size)].astype(np.int64)
    x = r.standard_normal((300, F)).astype(np.float32)
    x[r.random(x.shape) < 0.2] = 0.0
    w = r.standard_normal(tgt.size).astype(np.float32)
    g = tfg.tfg_graph_create(torch.from_numpy(ei).cuda(), deg.size, N_src=300)
    for reduce in ("sum", "mean", "max"):
        res = tfg.tfg_aggregate(None, torch.from_numpy(x).cuda(), deg.size, reduce,
                                edge_weight=torch.from_numpy(w).cuda(), graph=g)
        _check(orc, ei, x, deg.size, res, reduce, w, 1)
