"""Word merge of stable pairs at its edges, against the oracle: short last runs
of every length around a chunk (2 words), an item (252) and a block (256),
levels whose pairs need more items than a workgroup has rows (16, several
passes), lone pieces, and keys equal to the one the sentinel holds.  Then
64-bit keys that agree in the leading 40 bits of their tile's range and differ
below, in short runs (finished by exchanges of neighbours) and in long ones
(by ranking).

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


def check(mms, x):
    v = np.arange(x.size, dtype=np.uint32) * np.uint32(0x9E3779B1)
    xd, vd = (torch.from_numpy(a.view(np.int32)).cuda() for a in (x, v))
    for i32 in (False, True):
        gk, gv = mms.sort_pairs(xd, vd, i32=i32)
        ok, ov = oracle.sort(x, v, i32=i32)
        assert np.array_equal(gk.cpu().numpy().view(np.uint32), ok)
        assert np.array_equal(gv.cpu().numpy().view(np.uint32), ov)


@pytest.mark.parametrize("K", [2, 4, 8, 16])
def test_word_merge_edges(mms, K):
    mms.set_tuning([(64, K, 3840, 0, 0, mms.MMS_PAIRS)])
    for i, r in enumerate(EDGES):
        for runs in (1, 3, 16):
            n = runs * T + r
            x = mmsgen.uniform_u32(mmsgen.seed_for(53, i), n)
            check(mms, x)
            # a third of the keys are the largest one, a third few values
            u = mmsgen.uniform_u32(mmsgen.seed_for(54, i), n) % np.uint32(3)
            check(mms, np.where(u == 0, np.uint32(0xFFFFFFFF), np.where(u == 1, x % np.uint32(5), x)).astype(np.uint32))
    check(mms, np.full(5 * T + 77, 0xFFFFFFFF, dtype=np.uint32))
    # every run its own range: tiles of one long piece, both ways round
    z = np.arange(20 * T + 31, dtype=np.uint32)
    check(mms, z)
    check(mms, z[::-1].copy())


@pytest.mark.parametrize("weights", [(1, 1, 1, 1, 1, 1, 1, 1), (30, 1, 1, 1, 1, 1, 1, 1), (1, 1, 1, 1, 1, 1, 1, 30),
                                     (9, 1, 9, 1, 9, 1, 9, 1), (17, 16, 17, 16, 17, 16, 17, 16)])
def test_word_merge_uneven_pairs(mms, weights):
    """16 runs whose shares of the keys' lower half follow the weights of
    their pairs: the tiles there have uneven pieces, many of a size just past
    a whole number of items."""
    mms.set_tuning([(64, 16, 3840, 0, 0, mms.MMS_PAIRS)])
    x = mmsgen.uniform_u32(mmsgen.seed_for(55, 0), 16 * T).reshape(16, T)
    for k in range(16):
        low = T * weights[k // 2] // (2 * max(weights))
        x[k, :low] >>= np.uint32(1)
        x[k, low:] |= np.uint32(0x80000000)
    check(mms, np.ascontiguousarray(x).reshape(-1))


def check64(mms, x):
    v = np.arange(x.size, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    xd, vd = (torch.from_numpy(a.view(np.int64)).cuda() for a in (x, v))
    for i64 in (False, True):
        got = mms.sort64(xd, i64=i64)
        assert np.array_equal(got.cpu().numpy().view(np.uint64), oracle.sort_u64(x, i64=i64))
        gk, gv = mms.sort_pairs64(xd, vd, i64=i64)
        ok, ov = oracle.sort_u64(x, v, i64=i64)
        assert np.array_equal(gk.cpu().numpy().view(np.uint64), ok)
        assert np.array_equal(gv.cpu().numpy().view(np.uint64), ov)


@pytest.mark.parametrize("n", [4097, 16 * 4096 + 1, 20 * 4096 + 2047])
@pytest.mark.parametrize("kind", ["short", "equal_and_short", "long", "long_few", "one_low"])
def test_keys_that_share_a_word(mms, n, kind):
    low = mmsgen.splitmix64(mmsgen.seed_for(56, 1), n)
    far = mmsgen.splitmix64(mmsgen.seed_for(56, 2), n)
    if kind == "short":               # runs of about four keys per tile share their leading bits
        x = (far % np.uint64(1000) * np.uint64(0x0041000000000000)) | (low & np.uint64(0xFFFF))
    elif kind == "equal_and_short":   # with equal keys among them
        x = (far % np.uint64(700) * np.uint64(0x005D000000000000)) | (low & np.uint64(0x3))
    elif kind == "long":              # every tile spans the range, nearly all keys within 2^20
        x = np.where(far % np.uint64(64) == 0, far, low & np.uint64(0xFFFFF)).astype(np.uint64)
    elif kind == "long_few":          # the same with ties
        x = np.where(far % np.uint64(64) == 0, far, low & np.uint64(0x3F)).astype(np.uint64)
    else:                             # one small key against all others at the top
        x = low | np.uint64(0xFFFFFFFFFFF00000)
        x[n // 2] = 0
    check64(mms, x)
