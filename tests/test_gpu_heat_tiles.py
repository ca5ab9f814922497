"""disc_query_heatmap at the edges of its tiles: the BF16 contraction with 64
and 128 token rows (one step of K up to more than its prefetch holds), the FP32
one, up to 16 queries with E in quarters,
query tiles of 32 with the norms taken on the way and 64 with separate norms; every pair of token and projection type.

Against the definition in float64 on the stored values.  The arithmetic is
FP32 over K = C and K = E, each sum's error near sqrt(K) 2^-24 of its terms'
norm, below 2e-6 of |t| |y| here; the bar of 3e-5 max D leaves room for D's
own cancellation."""
import pytest

from gpu_common import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    disc.load()
    return disc


@pytest.mark.parametrize("tok,proj", [("bf16", "bf16"), ("f8", "bf16"), ("f32", "f32"), ("bf16", "f32"), ("f8", "f32"),
                                      ("f32", "bf16")])
@pytest.mark.parametrize("gh,gw,c,e,q", [
    (1, 1, 64, 128, 1),       # one token: D is r / (r + eps) = 0
    (7, 9, 64, 128, 16),      # 63 rows, one step of K
    (5, 13, 192, 128, 17),    # 65 rows, second query tile
    (8, 16, 320, 384, 33),    # five steps: the prefetch wraps
    (43, 47, 256, 1024, 3),   # 2021 rows
    (65, 64, 128, 1024, 5),   # tall BF16 tiles
    (63, 65, 128, 1024, 64),  # the same, last tile one row short; 32 x 32 similarity tiles
    (64, 65, 64, 128, 512),   # separate norms
])
def test_heat_tiles(gpu, tok, proj, gh, gw, c, e, q):
    t = torch()
    g = t.Generator().manual_seed(gh * 1000 + gw + c + q)
    G = gh * gw
    x = t.randn(G, c, generator=g) + 0.5
    scale = None
    if tok == "f8":
        scale = x.abs().amax(1) / 448
        x = (x / scale[:, None]).to(t.float8_e4m3fn)
        f64 = x.double() * scale.double()[:, None]
    else:
        x = x.to(t.bfloat16) if tok == "bf16" else x
        f64 = x.double()
    P = t.randn(c, e, generator=g) / c ** 0.5
    P = P.to(t.bfloat16) if proj == "bf16" else P
    text = t.randn(q, e, generator=g)
    text[q // 2] = 0
    text = text.to(t.bfloat16) if proj == "bf16" else text
    y = f64 @ P.double()
    r = (f64 - f64.mean(0)).norm(dim=1)
    D = r / (r.mean() + 1e-6)
    want = t.nn.functional.normalize(text.double(), dim=1) @ t.nn.functional.normalize(y, dim=1).T * D
    got = gpu.query_heatmap(x.view(gh, gw, c).cuda(), P.cuda(), text.cuda(), 16,
                            None if scale is None else scale.cuda()).cpu().double().view(q, G)
    assert not got[q // 2].any()
    assert (got - want).abs().max() <= 3e-5 * max(float(D.max()), 1.0)
