"""disc_backproject and disc_voxel_overlap beside other streams, threads and
graph captures: threads that each work on their own stream under one handle,
a buffer that grows and is then used by a smaller call, a capture in another
thread, and the forms that a capture takes against the ones that use the
workspace.  Every result exactly as by a call alone."""
import ctypes
import threading

import numpy as np
import pytest

import disc_inputs as di
from disc_inputs.scene import depth_scene
from gpu_common import dev_bits, torch
from oracle import geometry as og

pytestmark = pytest.mark.gpu
PER_THREAD = 2  # hipStreamPerThread


@pytest.fixture(scope="module", autouse=True)
def gpu():
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_03935_amd as disc

    disc.load()
    return disc


class Frame:
    """A depth frame's segments, its points and voxel lists, and the two calls on a stream."""

    def __init__(self, gpu, seed, h, w):
        t = torch()
        self.lib, self.h, self.w = gpu.load(), h, w
        self.sc = depth_scene(di.frame_seed(9, seed), h, w, n_obj=12)
        self.d, self.b = t.from_numpy(self.sc.depth).cuda(), dev_bits(self.sc.bits)
        self.pts, self.off = gpu.backproject(self.d, self.b, h, w, self.sc.camera, 1)
        self.vox, self.voff, _ = gpu.voxelize(self.pts, self.off, 0.05)
        self.m = self.off.shape[0] - 1
        every = [(i, j) for i in range(self.m) for j in range(self.m)]
        # more pairs than run at once and than lists: the calls that make boxes
        self.pairs = t.tensor(every * (1 + 700 // len(every)), dtype=t.int32, device="cuda")
        self.cnt = gpu.voxel_overlap(self.vox, self.voff, self.vox, self.voff, self.pairs)
        self.mk, self.cm = gpu.make_masks(self.b, h, w), gpu.make_camera(self.sc.camera)
        self.pts2, self.cnt2 = t.zeros_like(self.pts), t.zeros_like(self.cnt)

    def write(self, stream):
        assert self.lib.disc_backproject(self.d.data_ptr(), ctypes.byref(self.mk), ctypes.byref(self.cm), 1,
                                         self.off.data_ptr(), self.pts2.data_ptr(), stream) == 0

    def overlap(self, stream):
        p = self.pairs.shape[0]
        assert p > 512 and p > 2 * self.m
        v, o = self.vox.data_ptr(), self.voff.data_ptr()
        assert self.lib.disc_voxel_overlap(v, o, self.m, v, o, self.m, self.pairs.data_ptr(), p, self.cnt2.data_ptr(),
                                           stream) == 0

    def clear(self):
        self.pts2.zero_()
        self.cnt2.zero_()

    def same(self):
        t = torch()
        return t.equal(self.pts2.view(t.int32), self.pts.view(t.int32)) and t.equal(self.cnt2, self.cnt)


def test_threads_with_their_own_default_stream(gpu):
    frames = [Frame(gpu, 20 + i, 97, 130 + 64 * i) for i in range(3)]
    torch().cuda.synchronize()
    for _ in range(3):
        for f in frames:
            f.clear()
        torch().cuda.synchronize()
        errors = []

        def work(f):
            try:
                for _ in range(20):
                    f.write(PER_THREAD)
                    f.overlap(PER_THREAD)
                torch().cuda.synchronize()  # a thread's stream ends with it, perhaps before its work
            except AssertionError as e:
                errors.append(e)

        th = [threading.Thread(target=work, args=(f,)) for f in frames]
        for x in th:
            x.start()
        for x in th:
            x.join()
        torch().cuda.synchronize()
        assert not errors and all(f.same() for f in frames)


def test_growing_buffer(gpu):
    """A small frame, one whose bits need a larger buffer, and the small one again, in a row on one stream."""
    st = torch().cuda.Stream()
    small, large = Frame(gpu, 31, 97, 130), Frame(gpu, 32, 1080, 1920)
    want, woff = og.backproject(large.sc.depth, large.sc.bits, large.w, large.sc.camera, 1)
    assert np.array_equal(large.off.cpu().numpy(), woff)
    for f in (small, large):
        f.clear()
    torch().cuda.synchronize()
    for f in (small, large, small):
        f.write(st.cuda_stream)
        f.overlap(st.cuda_stream)
    torch().cuda.synchronize()
    assert np.array_equal(large.pts2.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert small.same() and large.same()


def test_captured_forms(gpu):
    """The captured calls have no workspace, the eager ones do: the same results, replay after replay."""
    t = torch()
    f = Frame(gpu, 41, 97, 130)
    t.cuda.synchronize()
    g = t.cuda.CUDAGraph()
    with t.cuda.graph(g):
        st = t.cuda.current_stream().cuda_stream
        f.write(st)
        f.overlap(st)
    for _ in range(3):
        f.clear()
        g.replay()
        assert t.equal(gpu.voxel_overlap(f.vox, f.voff, f.vox, f.voff, f.pairs), f.cnt)
        t.cuda.synchronize()
        assert f.same()


def test_capture_in_another_thread(gpu):
    """A graph captured (globally) while another thread's call makes its buffer and grows it."""
    t = torch()
    frames = [Frame(gpu, 51, 97, 130), Frame(gpu, 52, 720, 1280)]
    st, x, y = t.cuda.Stream(), t.arange(1000, device="cuda"), t.zeros(1000, dtype=t.int64, device="cuda")
    for f in frames:
        f.clear()
    t.cuda.synchronize()
    inside, done, errors = threading.Event(), threading.Event(), []

    def work():
        try:
            inside.wait()
            for f in frames:
                f.write(st.cuda_stream)
                f.overlap(st.cuda_stream)
        except AssertionError as e:
            errors.append(e)
        done.set()

    th = threading.Thread(target=work)
    th.start()
    g = t.cuda.CUDAGraph()
    with t.cuda.graph(g):
        y.add_(x)
        inside.set()
        done.wait()
        y.add_(x)
    th.join()
    for _ in range(3):
        g.replay()
    t.cuda.synchronize()
    assert not errors and all(f.same() for f in frames)
    assert t.equal(y, 6 * x)
