"""Pooling and its gradient at every width around the lane layouts, with a leading dimension that
leaves rows at dword alignment only and empty graphs at both ends, without the index check: sums
and means within the scaled 1e-5 bound of float32 sums, maxima, argmax and gradients exactly."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 7, 8, 15, 17, 30, 31, 33, 62, 63, 65, 130, 255, 256,
                               257, 300, 500, 602, 1030])
@pytest.mark.parametrize("most", [40, 5])  # nodes: four columns a lane, and one where F % 4 != 0
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
def test_pool_widths(F, most, dtype):
    import paper_2101_11552_amd as tfg
    tfg.load()
    r = np.random.default_rng(F)
    sizes = np.concatenate([[0, 0], r.integers(0, most, 60), [1, 5 * most, 0]])
    G, Nb = sizes.size, int(sizes.sum())
    gi = np.repeat(np.arange(G), sizes).astype(dtype)
    wide = torch.from_numpy(r.standard_normal((Nb, F + 1)).astype(np.float32)).cuda()
    x, index = wide[:, 1:], torch.from_numpy(gi).cuda()
    xh, dy = x.cpu().numpy(), r.standard_normal((G, F)).astype(np.float32)
    tot, mag = np.zeros((G, F)), np.zeros((G, F))
    np.add.at(tot, gi, xh.astype(np.float64))
    np.add.at(mag, gi, np.abs(xh.astype(np.float64)))
    cnt = np.maximum(sizes, 1)[:, None]
    for reduce, div in (("sum", 1), ("mean", cnt)):
        y = tfg.tfg_segment_pool(x, index, G, reduce, validate=False).cpu().numpy()
        assert float((np.abs(y - tot / div) / np.maximum(mag / div, 1e-30)).max()) <= 1e-5
        dx = tfg.tfg_segment_pool_backward(torch.from_numpy(dy).cuda(), index, reduce,
                                           validate=False)
        want = dy if reduce == "sum" else dy / cnt.astype(np.float32)
        np.testing.assert_array_equal(dx.cpu().numpy(), want[gi])
    y, arg = tfg.tfg_segment_pool(x, index, G, "max", validate=False)
    dx = tfg.tfg_segment_pool_backward(torch.from_numpy(dy).cuda(), index, "max", argmax=arg,
                                       validate=False).cpu().numpy()
    want = np.zeros((Nb, F), np.float32)
    off = np.concatenate([[0], np.cumsum(sizes)])
    for g in range(G):
        rows = xh[off[g]:off[g + 1]]
        if rows.shape[0] == 0:
            assert np.all(arg[g].cpu().numpy() == -1) and np.all(y[g].cpu().numpy() == 0)
            continue
        a = rows.argmax(0)
        np.testing.assert_array_equal(arg[g].cpu().numpy(), a + off[g])
        np.testing.assert_array_equal(y[g].cpu().numpy(), rows.max(0))
        want[off[g] + a, np.arange(F)] = dy[g]
    np.testing.assert_array_equal(dx, want)
