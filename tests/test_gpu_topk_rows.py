"""The ranking of many short rows (256 threads a row) at the ends of its range:
rows of 2047 to 2049 elements, k of 64 and 65, fewer elements than k, equal
scores, and rows whose large scores fall on few threads, more of them than the
candidate list takes.  Compared with a stable sort of the similarities that the
same call returns, exactly."""
import numpy as np
import pytest

from gpu_common import torch

pytestmark = pytest.mark.gpu


def _check(emb, text, k):
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    scores, idx, sim = (x.cpu().numpy() for x in disc.query_topk(t.from_numpy(emb).cuda(), t.from_numpy(text).cuda(), k))
    n = min(k, emb.shape[0])
    want = np.argsort(-sim, axis=1, kind="stable")[:, :n]
    assert np.array_equal(idx[:, :n], want)
    assert np.array_equal(scores[:, :n], np.take_along_axis(sim, want, axis=1))
    assert (idx[:, n:] == -1).all() and np.isneginf(scores[:, n:]).all()


@pytest.mark.parametrize("m", [1, 7, 255, 257, 2047, 2048, 2049])
@pytest.mark.parametrize("k", [1, 2, 63, 64, 65])
def test_rows(m, k):
    rng = np.random.default_rng(m + k)
    emb = rng.standard_normal((m, 16)).astype(np.float32)
    emb[rng.integers(0, m, m // 3)] = emb[0]
    _check(emb, rng.standard_normal((300, 16)).astype(np.float32), k)


@pytest.mark.parametrize("k", [1, 10, 64])
def test_few_threads_hold_the_largest(k):
    """Large scores in the columns of 64 to 90 threads, all eight of each: at k = 64 the 64th thread's maximum lies
    below more than 512 elements; also rows that rise, fall and are all equal."""
    m = 2048
    i = np.arange(m)
    rows = [i, -i, np.zeros(m), np.where(i % 256 < 64, 1e5 - 100.0 * (i % 256) - i * 1e-3, -i),
            np.where(i % 256 < 90, 1e5 - 100.0 * (i % 256) + i * 1e-3, -i)]
    for s in rows:
        ang = np.pi * (s - s.min()) / max(1.0, float(np.ptp(s))) if np.ptp(s) else np.full(m, 1.0)
        emb = np.zeros((m, 16), np.float32)
        emb[:, 0], emb[:, 1] = -np.cos(ang), np.sin(ang)
        text = np.zeros((2, 16), np.float32)
        text[:, 0], text[1, 1] = 1.0, 0.5
        _check(emb, text, k)
