"""Calls whose work items, at one workgroup each, come to 2^32 threads and more,
which one dimension of a launch cannot hold: they run, and give what smaller
calls give."""
import numpy as np
import pytest

import disc_inputs as di
from disc_inputs.scene import depth_scene
from gpu_common import torch
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


def test_backproject_masks(gpu):
    """2^21 masks of two row blocks; a few of them, the last among them, have points."""
    t = torch()
    h, w, m = 33, 64, (1 << 21) + 3
    rng = np.random.default_rng(3)
    depth = rng.uniform(0.5, 4.0, (h, w)).astype(np.float32)
    cam = depth_scene(1, 32, 64, n_obj=2, min_area=1).camera
    some = di.pack_masks((rng.random((5, h, w)) < 0.4).astype(np.uint8))
    at = np.array([0, 1, 70001, m - 2, m - 1])
    bits = t.zeros((m, h, 1), dtype=t.int64, device="cuda")
    bits[t.from_numpy(at).cuda()] = t.from_numpy(some.view(np.int64)).cuda()
    pts, off = gpu.backproject(t.from_numpy(depth).cuda(), bits, h, w, cam, 1)
    want, woff = og.backproject(depth, some, w, cam, 1)
    off = off.cpu().numpy()
    assert np.array_equal(off[at], woff[:-1]) and np.array_equal(off[at + 1], woff[1:])
    assert np.array_equal(pts.cpu().numpy().view(np.uint32), want.view(np.uint32))


def test_overlap_pairs(gpu):
    t = torch()
    rng = np.random.default_rng(4)
    sizes = [0, 1, 40, 300, 77]
    lists = []
    for c in sizes:
        code = rng.choice(8 ** 3, size=c, replace=False)
        cell = np.stack([code // 64, code // 8 % 8, code % 8], -1)
        lists.append(cell[np.lexsort(cell.T[::-1])])
    sets = [set(map(tuple, x.tolist())) for x in lists]
    table = t.tensor([[len(a & b) for b in sets] for a in sets], dtype=t.int32, device="cuda")
    vox = t.from_numpy(np.concatenate(lists).astype(np.int32)).cuda()
    off = t.from_numpy(np.cumsum([0] + sizes).astype(np.int32)).cuda()
    pairs = t.randint(0, 5, ((1 << 23) + 7, 2), device="cuda", dtype=t.int32, generator=t.Generator("cuda").manual_seed(1))
    got = gpu.voxel_overlap(vox, off, vox, off, pairs)
    assert t.equal(got, table[pairs[:, 0].long(), pairs[:, 1].long()])


def test_query_rows(gpu):
    """More query rows than one launch ranks."""
    t = torch()
    q, m, k = (1 << 22) + 3, 5, 2
    g = t.Generator("cuda").manual_seed(2)
    emb = t.randn(m, 16, device="cuda", generator=g)
    text = t.randn(q, 16, device="cuda", generator=g).bfloat16()
    scores, idx, sim = gpu.query_topk(emb, text, k)
    best, at = sim.sort(dim=1, descending=True, stable=True)
    assert t.equal(idx, at[:, :k].int()) and t.equal(scores, best[:, :k])
    for a in range(0, q, 1 << 20):
        x, y = text[a:a + (1 << 20)].double(), emb.double()
        want = (x @ y.T) / x.norm(dim=1)[:, None] / y.norm(dim=1)
        # 16 products and two norms in FP32: below 20 roundings of 2^-24
        assert (sim[a:a + (1 << 20)] - want).abs().max().item() < 1.2e-6


def test_pooling_tiles(gpu):
    """2^15 FP32 frames of one mask, 2048 channels: 2^20 pooling tiles."""
    t = torch()
    n, C, E = 1 << 15, 2048, 128
    g = t.Generator("cuda").manual_seed(3)
    tok = t.randn(2, 2, C, device="cuda", generator=g)
    proj = t.randn(C, E, device="cuda", generator=g) * C ** -0.5
    u8 = t.zeros(1, 16, 16, dtype=t.uint8, device="cuda")
    u8[0, 2:13, 3:11] = 1
    fr = gpu.FrameInput(tok, gpu.pack_masks(u8), 16, 16, 8, None)
    want = gpu.embed_frames([fr], proj)[0].out
    outs = gpu.embed_frames([fr] * n, proj)
    assert t.equal(t.cat([o.out for o in outs]), want.expand(n, E))
