"""The stored pooling choice of a shape is not taken for a batch of the same
tile count whose tiles hold other numbers of masks: which forms a call launches
does not depend on the calls before it."""
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


def _kernels(call):
    t = torch()
    t.cuda.synchronize()
    with t.profiler.profile(activities=[t.profiler.ProfilerActivity.CUDA]) as p:
        call()
        t.cuda.synchronize()
    names = {e.key for e in p.key_averages()}
    assert any("k_proj" in x for x in names), "the profiler saw no kernels"
    return names


# (C, not met in other tests; batches of (frames, masks each) in call order): 8 tiles of one or of 64 masks, one tile of 1, 17 or 64
@pytest.mark.parametrize("C,order", [(448, [(8, 1), (1, 512)]), (576, [(1, 512), (8, 1)]), (704, [(1, 1), (1, 17), (1, 64)]),
                                     (832, [(1, 64), (1, 1)])])
def test_choice_by_masks(gpu, C, order):
    t = torch()
    g = t.Generator("cuda").manual_seed(C)
    tok = t.randn(20, 20, C, device="cuda", generator=g)
    proj = t.randn(C, 128, device="cuda", generator=g) * C ** -0.5
    u8 = t.zeros(512, 160, 160, dtype=t.uint8, device="cuda")
    for i in range(512):
        u8[i, (7 * i) % 100:(7 * i) % 100 + 40, (11 * i) % 90:(11 * i) % 90 + 50] = 1
    bits = gpu.pack_masks(u8)
    for n, m in order:
        frames = [gpu.FrameInput(tok, bits[i * m:(i + 1) * m].contiguous(), 160, 160, 8, None) for i in range(n)]
        for first in (True, False):
            names = _kernels(lambda: gpu.embed_frames(frames, proj))
            few, tiled = any("k_pool_few" in x for x in names), any("k_pool<" in x for x in names)
            if m > 128:  # never a candidate
                assert tiled and not few, (n, m, names)
            elif first:  # both forms are timed
                assert tiled and few, (n, m, names)
            else:
                assert tiled != few, (n, m, names)


@pytest.mark.parametrize("C,m", [(1280, 8), (1280, 120)])
def test_first_call_work(gpu, C, m):
    """A first call runs at most six forms twice, as many as there are without the one for few masks."""
    t = torch()
    g = t.Generator("cuda").manual_seed(C)
    tok = t.randn(20, 20, C, device="cuda", generator=g)
    proj = t.randn(C, 128, device="cuda", generator=g) * C ** -0.5
    u8 = t.zeros(m, 160, 160, dtype=t.uint8, device="cuda")
    u8[:, 30:110, 20:140] = 1
    fr = gpu.FrameInput(tok, gpu.pack_masks(u8), 160, 160, 8, None)
    t.cuda.synchronize()
    with t.profiler.profile(activities=[t.profiler.ProfilerActivity.CUDA]) as p:
        gpu.embed_frames([fr], proj)
        t.cuda.synchronize()
    n = sum(e.count for e in p.key_averages() if "k_pool<" in e.key or "k_pool_few" in e.key)
    assert 2 <= n <= 12, [(e.key, e.count) for e in p.key_averages()]


def test_wavefronts(gpu):
    """Beyond one workgroup per CU the form for few masks runs with four wavefronts each."""
    t = torch()
    C = 896
    g = t.Generator("cuda").manual_seed(C)
    tok = t.randn(36, 36, C, device="cuda", generator=g)  # six K groups
    proj = t.randn(C, 128, device="cuda", generator=g) * C ** -0.5
    u8 = t.zeros(4, 288, 288, dtype=t.uint8, device="cuda")
    u8[:, 30:210, 20:240] = 1
    fr = gpu.FrameInput(tok, gpu.pack_masks(u8), 288, 288, 8, None)
    for n, form in ((1, "k_pool_few<8>"), (12, "k_pool_few<4>")):
        names = _kernels(lambda: gpu.embed_frames([fr] * n, proj))  # a first call: every form runs
        assert [x for x in ("k_pool_few<4>", "k_pool_few<8>") if any(x in y for y in names)] == [form]


@pytest.mark.parametrize("C,side,m,few", [(960, 360, 8, True), (960, 368, 8, False), (1088, 256, 64, True),
                                          (1088, 264, 64, False), (1088, 560, 1, True)])
def test_untimed(gpu, C, side, m, few):
    """The rule of untimed calls: 8 and 9 groups of 256 patches, 4 and 5 beyond 1024 channels, one mask."""
    t = torch()
    g = t.Generator("cuda").manual_seed(C)
    n = side // 8
    tok = t.randn(n, n, C, device="cuda", generator=g)
    proj = t.randn(C, 128, device="cuda", generator=g) * C ** -0.5
    u8 = t.zeros(m, side, side, dtype=t.uint8, device="cuda")
    u8[:, 30:210, 20:140] = 1
    fr = gpu.FrameInput(tok, gpu.pack_masks(u8), side, side, 8, None)
    names = _kernels(lambda: gpu.embed_masks_noalloc(fr, proj))
    assert any("k_pool_few" in x for x in names) == few and any("k_pool<" in x for x in names) != few
