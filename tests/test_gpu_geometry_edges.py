"""The geometry kernels at the edges of their work splits, against the oracle,
exactly: mask words and row blocks of the back-projection, dense cells and
many-cell neighbourhoods of the denoising, sort chunks of the voxel lists,
and overlaps with and without the boxes; also the forms that a graph capture
takes (no workspace)."""
import numpy as np
import pytest

import disc_inputs as di
from disc_inputs.scene import depth_scene
from gpu_common import dev_bits, torch
from oracle import geometry as og

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    disc.load()
    return disc


def _dev(pts, off):
    t = torch()
    return t.from_numpy(np.ascontiguousarray(pts, np.float32)).cuda(), t.from_numpy(off.astype(np.int32)).cuda()


@pytest.mark.parametrize("h,w,stride", [(1, 1, 1), (31, 64, 1), (33, 65, 2), (97, 1283, 1), (300, 520, 5)])
def test_backproject_blocks(gpu, h, w, stride):
    """Full, empty, one-pixel and random masks over readings that include
    every kind of missing one."""
    t = torch()
    rng = np.random.default_rng(h * w)
    depth = rng.uniform(0.05, 12.0, (h, w)).astype(np.float32)
    for v in (np.nan, np.inf, -np.inf, 0.0, -1.0):
        depth[rng.random((h, w)) < 0.03] = v
    u8 = np.zeros((5, h, w), np.uint8)
    u8[0] = 1
    u8[2, h - 1, w - 1] = 1
    u8[3] = rng.random((h, w)) < 0.3
    u8[4, h // 2:, : max(1, w // 3)] = 1
    cam = depth_scene(1, 32, 64, n_obj=2, min_area=1).camera
    bits = di.pack_masks(u8)
    want, woff = og.backproject(depth, bits, w, cam, stride)
    d, b = t.from_numpy(depth).cuda(), dev_bits(bits)
    pts, off = gpu.backproject(d, b, h, w, cam, stride)
    assert np.array_equal(off.cpu().numpy(), woff)
    assert np.array_equal(pts.cpu().numpy().view(np.uint32), want.view(np.uint32))


def test_calls_that_can_be_captured(gpu):
    """disc_backproject and disc_voxel_overlap in a graph, replayed between
    eager calls, give the eager results."""
    t = torch()
    h, w = 97, 130
    sc = depth_scene(di.frame_seed(9, 5), h, w, n_obj=12)
    d, b = t.from_numpy(sc.depth).cuda(), dev_bits(sc.bits)
    pts, off = gpu.backproject(d, b, h, w, sc.camera, 1)
    vox, voff, _ = gpu.voxelize(pts, off, 0.05)
    m = off.shape[0] - 1
    pairs = t.tensor([(i, j) for i in range(m) for j in range(m)], dtype=t.int32, device="cuda")
    cnt = gpu.voxel_overlap(vox, voff, vox, voff, pairs)
    lib = gpu.load()
    import ctypes

    mk, cm = gpu.make_masks(b, h, w), gpu.make_camera(sc.camera)
    pts2, cnt2 = t.zeros_like(pts), t.zeros_like(cnt)
    t.cuda.synchronize()
    g = t.cuda.CUDAGraph()
    with t.cuda.graph(g):
        st = t.cuda.current_stream().cuda_stream
        assert lib.disc_backproject(d.data_ptr(), ctypes.byref(mk), ctypes.byref(cm), 1, off.data_ptr(),
                                    pts2.data_ptr(), st) == 0
        assert lib.disc_voxel_overlap(vox.data_ptr(), voff.data_ptr(), m, vox.data_ptr(), voff.data_ptr(), m,
                                      pairs.data_ptr(), pairs.shape[0], cnt2.data_ptr(), st) == 0
    for _ in range(3):
        pts2.zero_()
        cnt2.zero_()
        g.replay()
        assert t.equal(gpu.voxel_overlap(vox, voff, vox, voff, pairs), cnt)
        assert t.equal(gpu.backproject(d, b, h, w, sc.camera, 1)[0], pts)
        t.cuda.synchronize()
        assert t.equal(pts2.view(t.int32), pts.view(t.int32)) and t.equal(cnt2, cnt)


@pytest.mark.parametrize("eps,min_pts", [(0.05, 1), (0.05, 7), (0.05, 200), (1.0, 64)])
def test_dbscan_cells(gpu, eps, min_pts):
    """Cells of one point, of 64, 65 and 300 points, points on cell corners
    (27 cells in reach), coincident points and a lone NaN."""
    rng = np.random.default_rng(11)
    segs = [0.5 + 0.02 * rng.random((64, 3)), 0.5 + 0.02 * rng.random((65, 3)), 0.5 + 0.02 * rng.random((300, 3)),
            rng.uniform(-0.4, 0.4, (900, 3)),
            np.stack(np.meshgrid(*[np.arange(-3, 4) * 0.05] * 3, indexing="ij"), -1).reshape(-1, 3),
            np.repeat(rng.uniform(0, 1, (5, 3)), 40, axis=0), np.zeros((0, 3)), rng.uniform(-50, 50, (70, 3))]
    pts = np.concatenate(segs).astype(np.float32)
    off = np.cumsum([0] + [len(x) for x in segs])
    keep = gpu.dbscan_denoise(*_dev(pts, off), eps, min_pts).cpu().numpy()
    assert np.array_equal(keep, og.dbscan_keep(pts, off, eps, min_pts))
    lone = pts.copy()
    lone[-1] = np.nan  # no neighbour, not even itself
    keep = gpu.dbscan_denoise(*_dev(lone, off), eps, min_pts).cpu().numpy()
    assert keep[-1] == 0


@pytest.mark.parametrize("counts", [(0, 1, 64, 65, 1023), (1024, 1025, 0, 2048), (9000, 3, 17000), (1,) * 150,
                                    (700,) * 40])
def test_voxel_chunks(gpu, counts):
    """Segments whose distinct voxels fill no, one or many sort chunks (more
    than eight too), and more segments in a workgroup than it counts in LDS;
    every voxel hit twice, points shuffled within their segment."""
    rng = np.random.default_rng(sum(counts))
    v = 0.05
    segs = []
    for c in counts:
        code = rng.choice(60 ** 3, size=c, replace=False)
        cell = np.stack([code // 3600, code // 60 % 60, code % 60], -1) - 30
        p = np.concatenate([(cell + rng.uniform(0.1, 0.9, cell.shape)) * v for _ in range(2)])
        segs.append(p[rng.permutation(len(p))])
    pts = np.concatenate(segs).astype(np.float32)
    off = np.cumsum([0] + [len(x) for x in segs])
    keep = (rng.random(len(pts)) < 0.9).astype(np.int32)
    for k in (None, keep):
        kd = None if k is None else torch().from_numpy(k).cuda()
        vox, voff, status = gpu.voxelize(*_dev(pts, off), v, keep=kd)
        rv, roff = og.voxelize(pts, off, k, v)
        assert not status.cpu().numpy().any()
        assert np.array_equal(voff.cpu().numpy(), roff)
        assert np.array_equal(vox.cpu().numpy(), rv)


@pytest.mark.parametrize("few", [False, True])
def test_overlap_lists(gpu, few):
    """Lists below, at and above the staged chunk, empty ones, far apart and
    nested; every pair once (no boxes are made) and often (they are)."""
    t = torch()
    rng = np.random.default_rng(5)
    sizes = [0, 1, 500, 4096, 4097, 9000, 300]
    lists = []
    for k, c in enumerate(sizes):
        code = rng.choice(24 ** 3, size=c, replace=False)
        cell = np.stack([code // 576, code // 24 % 24, code % 24], -1) + (0 if k < 6 else 1000)
        lists.append(cell[np.lexsort(cell.T[::-1])])
    vox = np.concatenate(lists).astype(np.int32)
    off = np.cumsum([0] + sizes)
    pairs = [(i, j) for i in range(7) for j in range(7)] + [(-1, 0), (0, 7), (7, 7)]
    pairs = pairs if few else 12 * pairs
    dv, do = t.from_numpy(vox).cuda(), t.from_numpy(off.astype(np.int32)).cuda()
    got = gpu.voxel_overlap(dv, do, dv, do, t.tensor(pairs, dtype=t.int32, device="cuda")).cpu().numpy()
    sets = [set(map(tuple, x.tolist())) for x in lists]
    want = [len(sets[i] & sets[j]) if 0 <= i < 7 and 0 <= j < 7 else 0 for i, j in pairs]
    assert got.tolist() == want
