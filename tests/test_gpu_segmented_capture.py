"""A batch whose launches a caller captures into a graph of its own: every
replay sorts what the input buffer holds then, also after more batches than the
library keeps plans for, with eager work between the replays.

Sorted segments are unique, so the comparison is element by element with no
tolerance."""
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


def batch(mms, sizes, seed):
    off = np.concatenate(([0], np.cumsum(sizes))).astype(np.uint64)
    x = mmsgen.uniform_u32(seed, int(off[-1]))
    return off, x, torch.empty(mms.segmented_workspace_bytes(off), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("sizes", [[5, 3000, 40_000, 3], [700, 1, 0, 2000, 64]])
def test_captured_batch_replays(mms, sizes):
    off, x, ws = batch(mms, sizes, mmsgen.seed_for(71, len(sizes)))
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    out = torch.empty_like(xd)
    mms.segmented_sort(xd, off, out_keys=out, workspace=ws, i32=False)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mms.segmented_sort(xd, off, out_keys=out, workspace=ws, i32=False)
    for trial in range(4):
        x = mmsgen.uniform_u32(mmsgen.seed_for(72, trial), x.size)
        xd.copy_(torch.from_numpy(x.view(np.int32)))
        out.zero_()
        for i in range(10):   # other batches, more than there are plans kept
            o2, x2, w2 = batch(mms, [100 + 7 * i, 3000 + i + trial], mmsgen.seed_for(73, i))
            got = mms.segmented_sort(torch.from_numpy(x2.view(np.int32)).cuda(), o2, workspace=w2, i32=False)
            assert np.array_equal(got.cpu().numpy().view(np.uint32), oracle.sort_segments(x2, o2))
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), oracle.sort_segments(x, off)), trial
