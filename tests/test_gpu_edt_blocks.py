"""The direct column search at the edges of its 8-row blocks and 8-distance
steps: items one row short of, at and past a block, a class and a step, with
interiors deep enough that whole blocks are skipped, narrow waists that only a
far step finds, and rows whose mask columns end on 64-bit words.  Whole-number
results: equal to the oracle's, and the patch weights equal to the band
layout's bit for bit."""
import numpy as np
import pytest

import disc_inputs as di
import oracle
from gpu_common import dev_bits, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    disc.load()
    return disc


# box rows + 2 padding rows: the classes' ends (32, 64, ..., 512), the tall
# class, and one row to either side of a block
@pytest.mark.parametrize("rows", [1, 5, 6, 7, 14, 15, 30, 31, 62, 63, 126, 127, 254, 255, 256, 263, 510, 511, 600])
@pytest.mark.parametrize("w", [64, 191, 640])
def test_block_edges(gpu, rows, w):
    h = rows + 3
    rng = np.random.default_rng(rows * 1000 + w)
    u8 = np.zeros((6, h, w), np.uint8)
    u8[0, 1 : 1 + rows] = 1                      # full box: every edge is the frame's or a padding row's
    u8[1, 2 : 2 + rows, w // 4 : w - 3] = 1
    u8[1, 2 + rows // 2, w // 2] = 0             # one hole in the middle
    u8[2, 1 : 1 + rows] = 1
    u8[2, 1 + rows // 3 : 1 + rows // 3 + 1, : w // 2] = 0   # a cut through one half
    yy, xx = np.indices((h, w))
    u8[3] = ((yy - 1 - rows / 2) / (rows / 2 + 0.6)) ** 2 + ((xx - w / 2) / (w / 2.2)) ** 2 <= 1.0
    u8[4, 1 : 1 + rows] = rng.random((rows, w)) < 0.9        # many runs per row
    u8[5, 1 : 1 + rows, 63 : min(w, 129)] = 1    # columns at the ends of words
    bits = di.pack_masks(u8)
    b = dev_bits(bits)
    got = gpu.edt_sq(b, h, w)
    torch().cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.edt_sq(bits, w))
    band = gpu.patch_weights(b, h, w, 16, distinct=0, edt_layout=1).cpu().numpy()
    direct = gpu.patch_weights(b, h, w, 16, distinct=0, edt_layout=2).cpu().numpy()
    assert np.array_equal(band, direct)
    # AREA counts pixels: whole numbers, without the column search
    for P in (14, 16):
        want = oracle.spatial_weights(bits, w, P, 1)
        area = gpu.patch_weights(b, h, w, P, spatial=1, distinct=0, edt_layout=2).cpu().numpy()
        assert np.array_equal(area.reshape(want.shape), want)
