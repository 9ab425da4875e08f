"""Segment softmax and its gradient at the row lengths and head counts where their lane groups
can go wrong: every length around the lists' edges and the chunks' (128 edges), hubs of 17 and 65
chunks, one of over 2,048 (its statistics combined by a block), heads in one and in several
passes, and rows with scores of -inf. Against 64-bit sums, at 1e-5: a few float32 roundings of the
exponential and the division (2^-24 each, times the scores' size of up to about 25)."""

import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 7, 8, 9, 10, 15, 16, 17, 23, 31, 32, 33, 47, 63, 64, 65, 100, 127, 128, 129,
           255, 256, 257, 700]


@pytest.fixture(scope="module")
def tfg():
    import paper_2101_11552_amd as m
    m.load()
    return m


def _case(tfg, seed, H, hubs, masked):
    r = np.random.default_rng(seed)
    deg = r.permutation(np.concatenate([np.repeat(LENGTHS, 6), np.array(hubs, dtype=np.int64)]))
    tgt = np.repeat(np.arange(deg.size), deg)[r.permutation(int(deg.sum()))]
    ei = np.stack([r.integers(0, deg.size, tgt.size), tgt]).astype(np.int64)
    s = (6 * r.standard_normal((tgt.size, H))).astype(np.float32)
    if masked:  # the first edges of the input order among them: whole chunks and leading slots
        s[r.random(s.shape) < 0.6] = -np.inf
        s[: tgt.size // 3] = -np.inf
    g = tfg.tfg_graph_create(torch.from_numpy(ei).cuda(), deg.size)
    return r, tgt, deg.size, s, g


def _softmax64(s, tgt, n):
    m = np.full((n, s.shape[1]), -np.inf)
    np.maximum.at(m, tgt, s.astype(np.float64))
    with np.errstate(invalid="ignore"):
        x = np.exp(s - m[tgt])  # NaN where every score of the row is -inf
    d = np.zeros((n, s.shape[1]))
    np.add.at(d, tgt, x)
    return x / d[tgt]


@pytest.mark.parametrize("H,hubs,masked", [
    (1, [2100, 8300, 300_000], False), (8, [2100, 8300, 300_000], False), (2, [2100], False),
    (3, [2100], False), (4, [2100], True), (5, [8300], False), (8, [2100, 8300], True),
    (16, [2100], False), (17, [2100], False), (32, [2100], True), (64, [2100], False),
    (80, [2100], True)])
def test_softmax_rows(tfg, H, hubs, masked):
    r, tgt, n, s, g = _case(tfg, H + masked, H, hubs, masked)
    perm = np.argsort(tgt, kind="stable")
    ref = _softmax64(s, tgt, n)
    t = torch.from_numpy(tgt).cuda()
    a, a_csr = tfg.tfg_segment_softmax(torch.from_numpy(s).cuda(), t, n, graph=g, out_csr=True)
    ordered = tfg.tfg_segment_softmax_graph(g, torch.from_numpy(s[perm]).cuda())
    a, a_csr, ordered = a.cpu().numpy(), a_csr.cpu().numpy(), ordered.cpu().numpy()
    np.testing.assert_array_equal(a_csr, a[perm])
    np.testing.assert_array_equal(ordered, a[perm])
    np.testing.assert_allclose(a, ref, rtol=1e-5, atol=1e-30, equal_nan=True)

    al = np.nan_to_num(a)
    da = r.standard_normal(s.shape).astype(np.float32)
    ds = tfg.tfg_segment_softmax_graph_backward(g, torch.from_numpy(al[perm]).cuda(),
                                                torch.from_numpy(da[perm]).cuda())
    dot, size = (np.zeros((n, H)) for _ in range(2))
    np.add.at(dot, tgt, al.astype(np.float64) * da)
    np.add.at(size, tgt, al.astype(np.float64) * np.abs(da))
    want, scale = al * (da - dot[tgt]), al * (np.abs(da) + size[tgt])
    err = np.abs(ds.cpu().numpy() - want[perm]) / np.maximum(scale[perm], 1e-30)
    assert float(err.max()) <= 1e-5


def _alpha_error(tfg, n, H):
    """Relative error (root mean square) of the coefficients of rows of n edges against 64 bits."""
    rows = max(4, 400_000 // (n * H))
    r = np.random.default_rng([12, n, H])
    tgt = np.repeat(np.arange(rows), n)
    s = r.standard_normal((tgt.size, H)).astype(np.float32)
    g = tfg.tfg_graph_create(torch.from_numpy(np.stack([tgt, tgt])).cuda(), rows)
    a = tfg.tfg_segment_softmax_graph(g, torch.from_numpy(s).cuda()).cpu().numpy()
    ref = _softmax64(s, tgt, rows)
    return float(np.sqrt(np.mean((a / ref - 1.0) ** 2)))


@pytest.mark.parametrize("n", [100, 2200])
def test_rows_from_registers_are_as_exact_as_swept_ones(tfg, n):
    """Rows of over 64 edges, whole and in chunks, keep their exponentials in registers at 8 heads
    and load the scores again at 5: both divide by the sum in double (2% for the sample)."""
    assert _alpha_error(tfg, n, 8) <= 1.02 * _alpha_error(tfg, n, 5)


def _check_edge_order_gradient(tfg, H, E, hubs):
    """Rows of the given lengths among E edges: the gradient in the caller's order against the
    graph order (the same products, added in double)."""
    r = np.random.default_rng([15, H])
    n = 20_000
    tgt = np.concatenate([np.repeat(np.arange(len(hubs)), hubs),
                          r.integers(len(hubs), n, E - sum(hubs) - 600),
                          r.integers(n, n + 2, 600)])
    r.shuffle(tgt)
    g = tfg.tfg_graph_create(torch.from_numpy(np.stack([tgt, tgt])).cuda(), n + 2)
    s, da = (torch.from_numpy(r.standard_normal((E, H)).astype(np.float32)).cuda() for _ in range(2))
    al = tfg.tfg_segment_softmax_graph(g, s, order="coo")
    ds = tfg.tfg_segment_softmax_graph_backward(g, al, da, order="coo")
    move = lambda t: tfg.tfg_edge_reorder(t, None, g)
    want = tfg.tfg_segment_softmax_graph_backward(g, move(al), move(da))
    scale = move(al) * (move(da).abs() + 4)
    assert float(((move(ds) - want).abs() / scale).max()) <= 2 ** -23


@pytest.mark.parametrize("H,E", [(1, 4_200_000), (2, 2_100_000), (3, 1_400_001), (4, 1_050_000)])
def test_gradient_of_split_rows_in_edge_order(tfg, H, E):
    """Arrays beyond the L2s in the caller's order: split rows of up to 16 chunks by a block each,
    of more by the chunk launches."""
    hubs = [129, 256, 257, 15 * 128, 16 * 128, 16 * 128 + 1, 17 * 128, 9000]
    _check_edge_order_gradient(tfg, H, E, hubs)


@pytest.mark.parametrize("H,E", [(1, 4_200_000), (4, 1_050_000)])
def test_gradient_of_giant_rows_in_edge_order(tfg, H, E):
    """Beside them, rows of 2,048 chunks (by the chunk launch) and of more (by a block each)."""
    _check_edge_order_gradient(tfg, H, E, [257, 2048 * 128, 2048 * 128 + 1])
