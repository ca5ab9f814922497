"""Voxel overlap of lists whose lengths lie around the counts at which a thread
takes 1, 2, 4 or 8 entries and a list takes several rounds, every length
against every other, with and without boxes."""
import numpy as np
import pytest

from gpu_common import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("repeat", [1, 7])
def test_lengths(repeat):
    check([0, 1, 63, 65, 511, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 4608, 8193], repeat)


def test_lengths_of_many_pairs():
    check([0, 1, 65, 255, 256, 257, 512, 513, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 6145, 10000], 22)


def check(sizes, repeat):
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    rng = np.random.default_rng(8)
    lists = []
    for c in sizes:
        code = rng.choice(22 ** 3, size=c, replace=False)
        cell = np.stack([code // 484, code // 22 % 22, code % 22], -1) - 11
        lists.append(cell[np.lexsort(cell.T[::-1])])
    sets = [set(map(tuple, x.tolist())) for x in lists]
    n = len(sizes)
    pairs = [(i, j) for i in range(n) for j in range(n)] * repeat
    assert (len(pairs) > 512) == (repeat > 1)
    vox = t.from_numpy(np.concatenate(lists).astype(np.int32)).cuda()
    off = t.from_numpy(np.cumsum([0] + sizes).astype(np.int32)).cuda()
    got = disc.voxel_overlap(vox, off, vox, off, t.tensor(pairs, dtype=t.int32, device="cuda")).cpu().numpy()
    assert got.tolist() == [len(sets[i] & sets[j]) for i, j in pairs]
