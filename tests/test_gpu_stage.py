"""The call's descriptors on the device, written by a kernel from its arguments
for up to eight frames and uploaded for more: batches of one, two, eight and
nine frames with no mask, one, 64, 65 and 130 masks a frame in turn give every
frame the bits it has alone."""
import numpy as np
import pytest

import disc_inputs as di
from gpu_common import dev_proj, frame_input, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    disc.load()
    return disc


@pytest.mark.parametrize("n", [1, 2, 8, 9])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_stage(gpu, n, dtype):
    C, E, P = 128, 128, 16
    proj = dev_proj(di.projection(4, C, E, dtype), dtype)
    frames = []
    for i in range(n):
        h, w, m = 120 + 17 * i, 200 - 9 * i, (130, 1, 0, 64, 65)[i % 5]
        bits = di.masks_mixed(50 + i, max(m, 1), h, w, 2e-3, 0.4)[:m]
        frames.append(di.Frame(di.tokens_normal(i, -(-h // P), -(-w // P), C, dtype, P), bits, h, w))
    ins = [frame_input(f) for f in frames]
    for _ in range(2):  # the second call finds the first one's workspace
        batch = gpu.embed_frames(ins, proj)
        for f, one in zip(batch, ins):
            if one.m == 0:
                continue
            alone = gpu.embed_frames([one], proj)[0]
            assert np.array_equal(f.out.cpu().numpy(), alone.out.cpu().numpy())
            assert np.array_equal(f.status.cpu().numpy(), alone.status.cpu().numpy())
