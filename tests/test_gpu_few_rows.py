"""The FP32 pooling and projection of few masks (16 x 16 tiles straight from
memory) at the edges of their tiles: one mask up to one past 64, patch grids of
one to nine K groups with ragged ends, channel counts that end inside a
projection group, FP32 and BF16 projections, several frames.  The sums are
promised bit for bit: pooled features equal those of the tiled pooling
(pool_tile = 1), and a mask's embedding does not depend on how many masks
share the call."""
import numpy as np
import pytest

import disc_inputs as di
from gpu_common import COS_FP32, check_embeddings, dev_proj, frame_input, oracle_frame, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    disc.load()
    return disc


def _part(fr, a, b):
    return di.Frame(fr.tokens, fr.bits[a:b], fr.h, fr.w)


@pytest.mark.parametrize("h,w,P,C,E,pdtype", [
    (200, 240, 16, 128, 128, "f32"),    # 195 patches: one group
    (336, 336, 16, 320, 256, "f32"),    # 441: two groups, K of the projection ends inside its second group
    (480, 640, 16, 256, 384, "bf16"),   # 1200: five groups
    (719, 641, 14, 192, 128, "f32"),    # 2392: ten groups, ragged width
])
def test_few_rows(gpu, h, w, P, C, E, pdtype):
    m = 81
    bits = di.masks_mixed(h + C, m, h, w, 5e-4, 0.4)
    bits[3] = 0
    tok = di.tokens_normal(C + P, -(-h // P), -(-w // P), C, "f32", P)
    fr = di.Frame(tok, bits, h, w)
    Pm = di.projection(9, C, E, pdtype)
    proj = dev_proj(Pm, pdtype)
    f32 = dict(gemm_dtype=0)
    tiled = gpu.embed_frames([frame_input(fr)], proj, pooled=True, options=gpu.make_options(pool_tile=1, **f32))[0]
    want, pooled = tiled.out.cpu().numpy(), tiled.pooled.cpu().numpy()
    check_embeddings(want, tiled.status.cpu().numpy(), oracle_frame(fr, Pm, pdtype), COS_FP32, "tiled")
    # the first call of a shape times every form (each writes the result), the second runs the one chosen
    for a, b in [(0, 1), (0, 15), (0, 16), (1, 18), (0, 64), (5, 70)]:
        part = frame_input(_part(fr, a, b))
        for _ in range(2):
            got = gpu.embed_frames([part], proj, pooled=True, options=gpu.make_options(**f32))[0]
            assert np.array_equal(got.pooled.cpu().numpy(), pooled[a:b]), (a, b)
            assert np.array_equal(got.out.cpu().numpy(), want[a:b]), (a, b)
        if b - a <= 64 and pdtype == "f32":  # untimed: the rule
            out = gpu.embed_masks_noalloc(part, proj, pooled=True, options=gpu.make_options(**f32))
            assert np.array_equal(out.pooled.cpu().numpy(), pooled[a:b]) and np.array_equal(out.out.cpu().numpy(), want[a:b])
    parts = [frame_input(_part(fr, a, b)) for a, b in [(0, 7), (7, 24), (24, 40)]]
    got = gpu.embed_frames(parts, proj, pooled=True, options=gpu.make_options(**f32))
    assert np.array_equal(np.concatenate([o.out.cpu().numpy() for o in got]), want[:40])
    assert np.array_equal(np.concatenate([o.pooled.cpu().numpy() for o in got]), pooled[:40])
