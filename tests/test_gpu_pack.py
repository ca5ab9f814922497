"""disc_pack_masks over the row widths where its 16-byte chunks are whole, cut
by the row's end or by the buffer's, at every alignment of the source."""
import numpy as np
import pytest

import disc_inputs as di
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


@pytest.mark.parametrize("w", [1, 15, 16, 17, 63, 64, 65, 130, 1280])
@pytest.mark.parametrize("m,h", [(1, 1), (3, 37), (2, 300)])
def test_pack_masks_widths_and_alignments(gpu, w, m, h):
    t = torch()
    rng = np.random.default_rng(w * 1000 + h)
    # any non-zero byte is a set pixel
    u8 = np.where(rng.random((m, h, w)) < 0.4, rng.integers(1, 256, (m, h, w)), 0).astype(np.uint8)
    want = di.pack_masks(u8)
    for shift in (0, 1, 7):
        buf = t.zeros(u8.size + shift, dtype=t.uint8, device="cuda")
        src = buf[shift:].view(m, h, w)
        src.copy_(t.from_numpy(u8))
        assert np.array_equal(gpu.pack_masks(src).cpu().numpy().view(np.uint64), want), shift
        assert np.array_equal(gpu.pack_masks(src != 0).cpu().numpy().view(np.uint64), want), "bool"
    turned = (t.from_numpy(np.ascontiguousarray(u8.transpose(0, 2, 1))).cuda() != 0).transpose(1, 2)
    assert np.array_equal(gpu.pack_masks(turned).cpu().numpy().view(np.uint64), want), "strided bool"
