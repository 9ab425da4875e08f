"""The graph build and the one-launch normalisation around the edges of their size rules: sort
tiles of 2048, 4096 and 8192 edges, digit tables read in the scatter blocks or scanned, one to
three passes of 4 to 8 bits, and the largest graph of the one-launch normalisation. The
permutation is the unique stable one and the weights are float32 expressions of exact degrees,
so everything is compared bit for bit."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tfg():
    import paper_2101_11552_amd as m
    m.load()
    return m


def _edges(n, e, dtype):
    r = np.random.default_rng([21, n, e])
    return np.stack([r.integers(0, n, e), r.integers(0, n, e)]).astype(dtype)


# (nodes, edges): nodes set the digits, edges the tile and whether its table is scanned
SIZES = [(10, 1), (16, 2047), (16, 2048), (255, 2049), (300, 8192), (300, 65537), (2708, 13264),
         (4096, 131073), (5000, 262145), (19717, 65536), (65536, 131073), (65536, 524288),
         (65536, 524289), (70000, 2048), (70000, 600000), (140000, 2097153),
         # fewer than 16 digits: 64 threads each, in 1,024 tiles and one more
         (1, 8191), (3, 600001), (7, 8388608), (8, 8388609)]


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("n,e", SIZES)
def test_build(tfg, n, e, dtype):
    ei = _edges(n, e, dtype)
    d = torch.from_numpy(ei).cuda()
    g = tfg.tfg_graph_create(d, n, src_parts=1)
    rowptr, col, perm = (t.cpu().numpy() for t in tfg.tfg_graph_csr(g))
    want = np.argsort(ei[1], kind="stable")
    assert np.array_equal(perm, want)
    assert np.array_equal(col, ei[0][want])
    assert np.array_equal(rowptr, np.searchsorted(ei[1][want], np.arange(n + 1)))
    bad = d.clone()
    bad[0, e - 1] = n  # the last edge's source, in the last tile
    with pytest.raises(IndexError):
        tfg.tfg_graph_create(bad, n, src_parts=1)
    tfg.tfg_graph_create(d, n, src_parts=1)  # and the flag does not stick


@pytest.mark.parametrize("n", [3, 5000])  # work lists by one block, and by several
@pytest.mark.parametrize("deg", [64 * 128 - 1, 64 * 128, 64 * 128 + 1, 65 * 128, 300 * 128 + 5])
def test_chunks_of_hub_rows(tfg, n, deg):
    """Rows of up to 64 chunks, whose items their own thread writes, and of more, which the
    wavefront does, two of them side by side: every chunk is summed once (integers: exact)."""
    tgt = np.concatenate([np.full(deg, 1), np.full(deg + 200, 2), np.arange(n)])
    r = np.random.default_rng([22, n, deg])
    src = r.integers(0, 50, tgt.size)
    x = r.integers(-8, 9, (50, 4)).astype(np.float32)
    order = r.permutation(tgt.size)
    ei = torch.from_numpy(np.stack([src, tgt])[:, order].astype(np.int64)).cuda()
    g = tfg.tfg_graph_create(ei, n, N_src=50)
    y = tfg.tfg_aggregate(None, torch.from_numpy(x).cuda(), n, graph=g).cpu().numpy()
    ref = np.zeros((n, 4))
    np.add.at(ref, tgt, x[src])
    assert np.array_equal(y, ref)


@pytest.mark.parametrize("n,e,loops", [(7, 0, True), (5000, 10, False), (2708, 10556, True),
                                       (3000, 2 ** 20 - 3000, True), (3000, 2 ** 20 - 2999, True),
                                       (100000, 2 ** 20, False)])
def test_unit_normalisation(tfg, orc, n, e, loops):
    for dtype in (np.int32, np.int64):
        ei = _edges(n, e, dtype) if e else np.zeros((2, 0), dtype)
        d = torch.from_numpy(ei).cuda()
        g = tfg.tfg_graph_create(d, n, add_self_loops=loops)
        r = tfg.tfg_gcn_norm(d, n, add_self_loops=loops, graph=g)
        oei, ow, odeg = orc.gcn_norm(ei.astype(np.int64), n, add_self_loops=loops)
        assert np.array_equal(r["edge_index"].cpu().numpy(), oei)
        assert np.array_equal(r["edge_weight"].cpu().numpy(), ow)
        assert np.array_equal(r["deg"].cpu().numpy(), odeg)
        perm = tfg.tfg_graph_csr(g)[2].cpu().numpy()
        assert np.array_equal(r["edge_weight_csr"].cpu().numpy(), ow[perm])
