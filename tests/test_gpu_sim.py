"""The similarity matrix of disc_query_topk at the edges of its tiles (16, 32
and 64 rows, K steps of 32 and 64), against float64, and the same bits from
every tile shape."""
import numpy as np
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


def _inputs(q, m, e, bf16):
    t = torch()
    g = t.Generator(device="cuda").manual_seed(q * 7919 + m * 31 + e)
    emb = t.randn(m, e, generator=g, device="cuda")
    text = t.randn(q, e, generator=g, device="cuda")
    return emb, text.to(t.bfloat16) if bf16 else text


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("q,m", [(1, 1), (16, 65), (17, 31), (33, 64), (65, 257), (600, 3600)])
@pytest.mark.parametrize("e", [16, 32, 80, 1024, 4096])
def test_sim_tiles_vs_float64(gpu, q, m, e, bf16):
    t = torch()
    emb, text = _inputs(q, m, e, bf16)
    _, _, sim = gpu.query_topk(emb, text, 3)
    want = t.nn.functional.normalize(text.double(), dim=1) @ t.nn.functional.normalize(emb.double(), dim=1).T
    # a sum of e products in FP32, each step rounded: (e - 1) u sum |t y| at most, and sum |t y| <= |t| |y|; the
    # norms and their products add a few u more, e u in all for each norm's own sum
    assert (sim.double() - want).abs().max().item() <= (3 * e + 8) * 2.0 ** -24


@pytest.mark.parametrize("bf16", [False, True])
def test_sim_bits_do_not_depend_on_the_tile(gpu, bf16):
    """600 x 3600 runs 64 x 64 tiles, 40 queries of them 32 x 32, 9 of them 16 x 64."""
    t = torch()
    emb, text = _inputs(600, 3600, 208, bf16)
    whole = gpu.query_topk(emb, text, 5)[2]
    for a, n in ((0, 40), (97, 40), (560, 40), (311, 9), (591, 9)):
        assert t.equal(gpu.query_topk(emb, text[a:a + n].contiguous(), 5)[2], whole[a:a + n])
