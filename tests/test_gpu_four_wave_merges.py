"""The word merges' four-wave kernels (256-word blocks, items of up to 252
words, 16 rows), which launches of more than 1024 tiles take: stable pairs with
short last runs of every length around a chunk (2 words), an item and a block,
with pairs of runs of uneven sizes (levels with more items than rows, several
passes), with ties and the key that the sentinel holds; then 64-bit pairs and
keys that share words, merged a second time.

A stable order is unique, so the comparison is element by element with no
tolerance."""
import numpy as np
import pytest

import mmsgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T = 2048   # base shape 0
EDGES = [1, 2, 3, 4, 5, 7, 125, 127, 128, 129, 249, 251, 252, 253, 255, 256, 257, 505, 1500]


@pytest.fixture(scope="module")
def mms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_07961_amd as m
    m._lib.lib()
    yield m
    m.set_tuning([])
    m._lib.load_tuning(m._lib.lib())


def check_batch(mms, x, sizes):
    """One batch: the tiles of all segments are one launch's."""
    off = np.concatenate(([0], np.cumsum(sizes))).astype(np.uint64)
    assert int(off[-1]) == x.size and sum(-(-n // 3840) for n in sizes if n > T) > 1024
    v = np.arange(x.size, dtype=np.uint32) * np.uint32(0x9E3779B1)
    xd, vd = (torch.from_numpy(a.view(np.int32)).cuda() for a in (x, v))
    gk, gv = mms.segmented_sort(xd, off, values=vd, i32=False)
    ok, ov = oracle.sort_segments(x, off, v)
    assert np.array_equal(gk.cpu().numpy().view(np.uint32), ok)
    assert np.array_equal(gv.cpu().numpy().view(np.uint32), ov)


@pytest.mark.parametrize("K", [2, 16])
@pytest.mark.parametrize("ties", [False, True])
def test_short_last_runs(mms, K, ties):
    mms.set_tuning([(64, K, 3840, 0, 0, mms.MMS_PAIRS)])
    sizes = [runs * T + r for r in EDGES for runs in (1, 3, 16)] * 10
    x = mmsgen.uniform_u32(mmsgen.seed_for(65, K), sum(sizes))
    if ties:   # a third of the keys are the largest one, a third few values
        u = mmsgen.uniform_u32(mmsgen.seed_for(66, K), x.size) % np.uint32(3)
        x = np.where(u == 0, np.uint32(0xFFFFFFFF), np.where(u == 1, x % np.uint32(5), x)).astype(np.uint32)
    check_batch(mms, x, sizes)


@pytest.mark.parametrize("weights", [(30, 1, 1, 1, 1, 1, 1, 1), (1, 1, 1, 1, 1, 1, 1, 30), (9, 1, 9, 1, 9, 1, 9, 1),
                                     (17, 16, 17, 16, 17, 16, 17, 16)])
def test_uneven_pairs_of_runs(mms, weights):
    """Groups of 16 runs whose shares of the keys' lower half follow the weights
    of their pairs."""
    mms.set_tuning([(64, 16, 3840, 0, 0, mms.MMS_PAIRS)])
    groups = 120
    x = mmsgen.uniform_u32(mmsgen.seed_for(67, weights[0]), groups * 16 * T).reshape(groups, 16, T)
    for k in range(16):
        low = T * weights[k // 2] // (2 * max(weights))
        x[:, k, :low] >>= np.uint32(1)
        x[:, k, low:] |= np.uint32(0x80000000)
    check_batch(mms, np.ascontiguousarray(x).reshape(-1), [16 * T] * groups)


@pytest.mark.parametrize("kind", ["short", "long", "one_low"])
def test_words_shared_in_large_sorts(mms, kind):
    n = 1090 * 3456 + 77
    low = mmsgen.splitmix64(mmsgen.seed_for(68, 1), n)
    far = mmsgen.splitmix64(mmsgen.seed_for(68, 2), n)
    if kind == "short":       # a few keys to an id, differing in every low bit but one
        x = (far % np.uint64(n // 3) * np.uint64((1 << 64) // n)) & np.uint64(0xFFFFFFFFFFFF0000) | (low & np.uint64(0x7FFF))
    elif kind == "long":      # every base tile spans the range, nearly all keys within 2^20
        x = np.where(far % np.uint64(64) == 0, far, low & np.uint64(0xFFFFF)).astype(np.uint64)
    else:                     # one small key against all others at the top
        x = low | np.uint64(0xFFFFFFFFFFF00000)
        x[n // 2] = 0
    v = np.arange(n, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    xd, vd = (torch.from_numpy(a.view(np.int64)).cuda() for a in (x, v))
    ok, ov = oracle.sort_u64(x, v, i64=False)
    assert np.array_equal(mms.sort64(xd, i64=False).cpu().numpy().view(np.uint64), ok)
    gk, gv = mms.sort_pairs64(xd, vd, i64=False)
    assert np.array_equal(gk.cpu().numpy().view(np.uint64), ok)
    assert np.array_equal(gv.cpu().numpy().view(np.uint64), ov)
