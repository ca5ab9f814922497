"""The ranking of disc_query_topk at the edges of its kernels: rows of one and
of several chunks, k at both ends of its range, equal scores, and rows whose
large scores fall on few threads.  The ranking is compared with a stable sort
of the similarities that the same call returns, exactly."""
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


def _check(gpu, emb, text, k):
    t = torch()
    scores, idx, sim = (x.cpu().numpy() for x in gpu.query_topk(t.from_numpy(emb).cuda(), t.from_numpy(text).cuda(), k))
    n = min(k, emb.shape[0])
    want = np.argsort(-sim, axis=1, kind="stable")[:, :n]
    assert np.array_equal(idx[:, :n], want)
    assert np.array_equal(scores[:, :n], np.take_along_axis(sim, want, axis=1))
    assert (idx[:, n:] == -1).all() and np.isneginf(scores[:, n:]).all()


@pytest.mark.parametrize("m", [1, 63, 1023, 1025, 8192, 8193, 32768, 32769, 100003])
@pytest.mark.parametrize("k", [1, 10, 64, 65, 256])
def test_topk_rows(gpu, m, k):
    rng = np.random.default_rng(m + k)
    emb = rng.standard_normal((m, 16)).astype(np.float32)
    emb[rng.integers(0, m, m // 3)] = emb[0]  # equal scores
    _check(gpu, emb, rng.standard_normal((3, 16)).astype(np.float32), k)


@pytest.mark.parametrize("m,k", [(8000, 10), (8000, 256), (32768, 64), (32768, 256)])
def test_topk_few_threads_hold_the_largest(gpu, m, k):
    """Scores that grow with the index, fall with it, are all equal, and a row
    whose large scores repeat every 1024 elements and sink from group to group
    of four threads: at m = 32768, k = 64 the 64th group maximum lies below
    about 8000 elements, more than the candidate list takes."""
    i = np.arange(m)
    group = i % 1024 // 4
    rows = [i, -i, np.zeros(m), np.where(group < 64, 1e5 - 1000.0 * group + i * 1e-3, -i)]
    for s in rows:
        ang = np.pi * (s - s.min()) / max(1.0, float(np.ptp(s))) if np.ptp(s) else np.full(m, 1.0)
        emb = np.zeros((m, 16), np.float32)
        emb[:, 0], emb[:, 1] = -np.cos(ang), np.sin(ang)
        text = np.zeros((2, 16), np.float32)
        text[:, 0], text[1, 1] = 1.0, 0.5
        _check(gpu, emb, text, k)
