"""Base case of the 16-per-lane shapes at its edges, against the oracle: sizes
around a lane's words (16), a wave's (1024) and each power of two up to the
tile, where whole waves and merge steps are left out, and tiles in a row with a
ragged last one.

Sorted keys and stable pairs are unique, so the comparison is element by
element with no tolerance."""
import numpy as np
import pytest

import mmsgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [1, 2, 3, 5, 15, 16, 17, 63, 64, 65, 1023, 1024, 1025, 1027, 2047, 2048, 2049, 3000, 4095, 4096, 4097, 5001,
         8191, 8192, 8193, 9217, 33000]


@pytest.fixture(scope="module")
def mms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_07961_amd as m
    m._lib.lib()
    yield m
    m.set_tuning([])
    m._lib.load_tuning(m._lib.lib())


def families(n, i):
    x = mmsgen.uniform_u32(mmsgen.seed_for(61, i), n)
    yield x
    u = mmsgen.uniform_u32(mmsgen.seed_for(62, i), n) % np.uint32(3)
    yield np.where(u == 0, np.uint32(0xFFFFFFFF), np.where(u == 1, x % np.uint32(5), x)).astype(np.uint32)
    yield np.arange(n, dtype=np.uint32)
    yield np.arange(n, dtype=np.uint32)[::-1].copy()


@pytest.mark.parametrize("base", [2, 5, 6])
def test_tile_net_keys(mms, base):
    mms.set_tuning([(64, 16, 2048, 3, base)])
    for i, n in enumerate(SIZES):
        for x in families(n, i):
            xd = torch.from_numpy(x.view(np.int32)).cuda()
            for i32 in (False, True):
                assert np.array_equal(mms.sort(xd, i32=i32).cpu().numpy().view(np.uint32), oracle.sort(x, i32=i32)), n


def test_tile_net_pairs(mms):
    mms.set_tuning([(64, 16, 3840, 0, 5, mms.MMS_PAIRS)])
    assert mms.plan(10**6, pairs=True).tile == 4096
    for i, n in enumerate(SIZES):
        v = np.arange(n, dtype=np.uint32) * np.uint32(0x9E3779B1)
        vd = torch.from_numpy(v.view(np.int32)).cuda()
        for x in families(n, i):
            xd = torch.from_numpy(x.view(np.int32)).cuda()
            for i32 in (False, True):
                gk, gv = mms.sort_pairs(xd, vd, i32=i32)
                ok, ov = oracle.sort(x, v, i32=i32)
                assert np.array_equal(gk.cpu().numpy().view(np.uint32), ok), n
                assert np.array_equal(gv.cpu().numpy().view(np.uint32), ov), n


def test_tile_net_unaligned_segments(mms):
    """A batch's segments start anywhere: no 16-byte alignment of the input or
    the output."""
    mms.set_tuning([(64, 16, 2048, 3, 6), (64, 16, 3840, 0, 5, mms.MMS_PAIRS)])
    sizes = [1, 8191, 3, 8192, 4097, 2, 20001, 1025]
    off = np.concatenate(([0], np.cumsum(sizes))).astype(np.uint64)
    x = mmsgen.uniform_u32(mmsgen.seed_for(63, 0), int(off[-1])) % np.uint32(5000)
    v = np.arange(x.size, dtype=np.uint32)
    xd, vd = (torch.from_numpy(a.view(np.int32)).cuda() for a in (x, v))
    k = mms.segmented_sort(xd, off, i32=False).cpu().numpy().view(np.uint32)
    pk, pv = (t.cpu().numpy().view(np.uint32) for t in mms.segmented_sort(xd, off, values=vd, i32=False))
    for a, b in zip(off[:-1], off[1:]):
        a, b = int(a), int(b)
        ok, ov = oracle.sort(x[a:b], v[a:b])
        assert np.array_equal(k[a:b], ok) and np.array_equal(pk[a:b], ok) and np.array_equal(pv[a:b], ov)
