"""How far float32 sums are from the same sums in 64 bits, at one row length at a time: no
further (2-norm over many rows and columns) than sums in a stated order of float32
multiply-adds, emulated here. Rows of up to 4 edges against one chain, rows of 128 edges
against eight interleaved chains added up in pairs (four for the attention layer). The bound is
that order's own error with 2% for the sample (60,000 sums or more)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tfg():
    import paper_2101_11552_amd as m
    m.load()
    return m


def _chains(w, x, k):
    """Sum over axis 1 in k interleaved chains of float32 multiply-adds, then pairwise."""
    acc = np.zeros((k, w.shape[0], x.shape[2]), np.float32)
    for j in range(x.shape[1]):
        a = acc[j % k]
        acc[j % k] = (w[:, j, None].astype(np.float64) * x[:, j] + a).astype(np.float32)
    parts = list(acc)
    while len(parts) > 1:
        parts = [parts[i] + parts[i + 1] for i in range(0, len(parts), 2)]
    return parts[0]


def _rows(seed, n, F):
    rows = max(256, 60000 // F)
    r = np.random.default_rng([seed, n, F])
    src = r.integers(0, 5000, (rows, n))
    x = r.standard_normal((5000, F)).astype(np.float32)
    ei = np.stack([src.ravel(), np.repeat(np.arange(rows), n)]).astype(np.int64)
    return r, rows, src, x, torch.from_numpy(ei).cuda()


def _err(y, ref):
    return np.linalg.norm(y - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,F,chains", [(2, 64, 1), (3, 16, 1), (3, 64, 1), (4, 256, 1),
                                        (128, 200, 8), (128, 256, 8)])
def test_sums(tfg, n, F, chains, weighted):
    r, rows, src, x, ei = _rows(1, n, F)
    w = r.uniform(0.5, 1.5, src.size).astype(np.float32) if weighted else np.ones(src.size, np.float32)
    y = tfg.tfg_aggregate(ei, torch.from_numpy(x).cuda(), rows,
                          edge_weight=torch.from_numpy(w).cuda() if weighted else None)
    w = w.reshape(rows, n)
    ref = (w[:, :, None].astype(np.float64) * x[src]).sum(1)
    assert _err(y.cpu().numpy(), ref) <= 1.02 * _err(_chains(w, x[src], chains), ref)


@pytest.mark.parametrize("n,H,D,chains", [(3, 8, 8, 1), (128, 4, 64, 4)])
def test_attention_sums(tfg, n, H, D, chains):
    """Equal scores: every coefficient is 1 / n, and the rows are means."""
    _, rows, src, x, ei = _rows(2, n, H * D)
    N = 5000
    g = tfg.tfg_graph_create(ei, N)
    zero = torch.zeros(H, D, device="cuda")
    y = tfg.tfg_gat_aggregate(g, torch.from_numpy(x).cuda(), zero, zero, 0.2).cpu().numpy()[:rows]
    ref = x[src].astype(np.float64).mean(1)
    emu = (_chains(np.ones((rows, n), np.float32), x[src], chains).astype(np.float64) / n).astype(np.float32)
    assert _err(y, ref) <= 1.02 * _err(emu, ref)
