"""DBSCAN where most cells hold one or two points, so that every point looks its
cells up by itself: on both sides of that rule, with clusters among the lone
points, cells at and beyond the ends of the key range, coincident points and a
NaN, against the oracle."""
import numpy as np
import pytest

from gpu_common import torch
from oracle import geometry as og

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("segs,clustered,min_pts", [(60, 0.1, 4), (60, 0.1, 2), (60, 0.9, 4), (14, 0.3, 1), (60, 0.0, 12)])
def test_sparse_cells(segs, clustered, min_pts):
    cells, n = check(segs, clustered, min_pts)
    assert (cells > (10000 if min_pts == 1 else 30000 + n // 4)) == (clustered < 0.5)


@pytest.mark.parametrize("clustered,min_pts", [(0.1, 4), (0.1, 2), (0.5, 4), (0.7, 4), (0.0, 12)])
def test_sparse_cells_of_large_clouds(clustered, min_pts):
    cells, n = check(230, clustered, min_pts)
    assert (cells > 130000 + n // 6) == (clustered < 0.6)


def check(segs, clustered, min_pts):
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    eps, per = 0.05, 960
    rng = np.random.default_rng(segs + min_pts)
    pts, cells = [], 0
    for s in range(segs):
        p = rng.uniform(-4, 4, (per, 3))
        nc = int(per * clustered) // 8
        if nc:
            p[:8 * nc] = (rng.uniform(-4, 4, (nc, 1, 3)) + rng.uniform(-0.03, 0.03, (nc, 8, 3))).reshape(-1, 3)
        if s == 1:  # the last cells of the key range and points far past it
            e = 32767 * eps
            p[-40:] = [(e + 0.01 * k, -e - 0.012 * k, 3 * e) for k in range(40)]
        if s == 2:
            p[-30:] = p[-30]
        cells += len(np.unique(np.floor(p / eps), axis=0))
        pts.append(p[rng.permutation(per)])
    p = np.concatenate(pts).astype(np.float32)
    n = len(p)
    off = np.arange(segs + 1, dtype=np.int32) * per
    dp, do = t.from_numpy(p).cuda(), t.from_numpy(off).cuda()
    assert np.array_equal(disc.dbscan_denoise(dp, do, eps, min_pts).cpu().numpy(), og.dbscan_keep(p, off, eps, min_pts))
    dp[5] = float("nan")  # no neighbour, not even itself
    assert disc.dbscan_denoise(dp, do, eps, min_pts)[5].item() == 0
    return cells, n
