"""Batches that a caller captures without having planned them before: on an
empty and on a full cache of plans, many in one graph, and the pinned memory of
destroyed graphs, which a later batch frees.

Sorted segments are unique, so the comparison is element by element with no
tolerance."""
import gc

import numpy as np
import pytest

import mmsgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_07961_amd as m
    m._lib.lib()
    return m


class Batch:
    def __init__(self, mms, sizes, seed):
        self.mms, self.seed = mms, seed
        self.off = np.concatenate(([0], np.cumsum(sizes))).astype(np.uint64)
        self.ws = torch.empty(mms.segmented_workspace_bytes(self.off), dtype=torch.uint8, device="cuda")
        self.keys = torch.empty(int(self.off[-1]), dtype=torch.int32, device="cuda")
        self.out = torch.empty_like(self.keys)
        self.fill(0)

    def fill(self, trial):
        self.x = mmsgen.uniform_u32(mmsgen.seed_for(self.seed, trial), self.keys.numel())
        self.keys.copy_(torch.from_numpy(self.x.view(np.int32)))
        self.out.zero_()

    def sort(self):
        self.mms.segmented_sort(self.keys, self.off, out_keys=self.out, workspace=self.ws, i32=False)

    def check(self):
        assert np.array_equal(self.out.cpu().numpy().view(np.uint32), oracle.sort_segments(self.x, self.off))


@pytest.mark.parametrize("kept", [0, 12])
def test_capture_of_batches_not_planned(mms, kept):
    """kept eager batches before the capture: more than there are plans kept."""
    eager = [Batch(mms, [50 + 9 * i, 4000 + i], 80 + i) for i in range(kept)]
    for b in eager:
        b.sort()
    batches = [Batch(mms, s, 60 + i) for i, s in enumerate([[5, 3000, 40_000 + kept, 3], [7, 9], [20_000] * 3])]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for b in batches:
            b.sort()
    for trial in range(3):
        for b in batches + eager:
            b.fill(trial)
        for b in eager:
            b.sort()
            b.check()
        g.replay()
        torch.cuda.synchronize()
        for b in batches:
            b.check()


def mapped_bytes():
    """The process's address space, in which pinned memory shows."""
    with open("/proc/self/status") as f:
        return next(int(line.split()[1]) * 1024 for line in f if line.startswith("VmSize"))


def test_images_of_destroyed_graphs_are_freed(mms):
    """Another signature every time, with an image of 21.6 MB each."""
    before = mapped_bytes()
    held = torch.empty(64 << 20, dtype=torch.uint8, pin_memory=True)
    if mapped_bytes() - before < held.numel() // 2:
        pytest.skip("pinned memory does not show in the address space")
    plain = Batch(mms, [10, 20], 91)
    most = Batch(mms, [3] * 300_030, 90)    # buffers for all of them

    def once(i):
        off = most.off[:300_000 + i + 1]
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            mms.segmented_sort(most.keys, off, out_keys=most.out, workspace=most.ws, i32=False)
        g.replay()
        torch.cuda.synchronize()
        want = oracle.sort_segments(most.x[: int(off[-1])], off)
        assert np.array_equal(most.out[: int(off[-1])].cpu().numpy().view(np.uint32), want)
        del g
        gc.collect()
        plain.sort()
        torch.cuda.synchronize()

    for i in range(4):
        once(i)
    before = mapped_bytes()
    for i in range(4, 20):
        once(i)
    grown = mapped_bytes() - before
    assert grown < 4 * 21_600_000, grown
