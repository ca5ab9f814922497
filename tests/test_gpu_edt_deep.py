"""Tall masks wide and deep enough that the exact 32-bit search decodes every
squared row distance the table can hold (0 to 576, and all beyond): equal to
the oracle's distances."""
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
