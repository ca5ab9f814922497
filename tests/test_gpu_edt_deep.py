"""The column search at both ends of its depths: tall masks wide and deep enough that
the exact 32-bit search decodes every squared row distance the table can hold (0
to 576, and all beyond), and thin masks whose rows need only the nearest
distances: equal to the oracle's distances."""
import numpy as np
import pytest

import disc_inputs as di
import oracle
from gpu_common import dev_bits, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,cut", [(1150, 1300, 0), (1149, 1290, 3), (1000, 1153, 1)])
def test_deep_interior(h, w, cut):
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    yy, xx = np.indices((h, w))
    u8 = np.ones((4, h, w), np.uint8)
    u8[0, :cut] = 0
    u8[1, h // 2, w // 2] = 0                       # one hole in the middle
    u8[2, :, :40 + cut] = 0                          # left edge inside a word
    u8[2, 5:, w - 7:] = 0
    u8[3] = ((yy - h / 2) / (h / 2 - cut)) ** 2 + ((xx - w / 2) / (w / 2 - 3)) ** 2 <= 1.0
    bits = di.pack_masks(u8)
    got = disc.edt_sq(dev_bits(bits), h, w)
    t.cuda.synchronize()
    want = oracle.edt_sq(bits, w)
    assert want.max() > 440 ** 2
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("h,w", [(60, 130), (250, 200), (500, 333), (700, 150)])
def test_shallow_interior(h, w):
    """Bands of 1 to 14 pixels along rows, columns and diagonals, and holes 3 to 8 apart: groups whose rows are all
    within five pixels of the outside, just beyond, or both, in every class of heights."""
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    yy, xx = np.indices((h, w))
    masks = []
    for k in range(1, 15):
        masks += [yy % (k + 1) < k, xx % (k + 1) < k, (xx + 2 * yy) % (3 * k) < 2 * k, (xx - 3 < k) & (xx >= 3)]
    for k in range(3, 9):
        masks += [(yy % k > 0) | (xx % k > 0), (yy % (2 * k) > 0) | (xx % k > 0)]
    u8 = np.stack(masks).astype(np.uint8)
    bits = di.pack_masks(u8)
    b = dev_bits(bits)
    got = disc.edt_sq(b, h, w)
    t.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.edt_sq(bits, w))
    band = disc.patch_weights(b, h, w, 16, distinct=0, edt_layout=1)
    assert t.equal(band, disc.patch_weights(b, h, w, 16, distinct=0, edt_layout=2))
