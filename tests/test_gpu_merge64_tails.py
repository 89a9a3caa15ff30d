"""64-bit merges whose last tile holds fewer elements than its workgroup's
waves have load steps for, with keys that do not fit the tile's words: every
wave has to take the same branches (the tile's range, the check of the words'
order, the second sort), those without a load step too.  Both kernels: eight
waves up to 1024 tiles of a round, four above.

Orders are unique (a stable sort), so the comparison is element by element with
no tolerance."""
import numpy as np
import pytest

import mmsgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILE = 3456   # outputs of a merge tile


@pytest.fixture(scope="module")
def mms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_07961_amd as m
    m._lib.lib()
    return m


def shared(n, seed, top):
    """n keys, about three to each of n / 3 ids spread over the high bits, with a
    small counter in the low ones; the last `top` of them in order are spread
    over the upper half, the others over the lower."""
    a = mmsgen.splitmix64(mmsgen.seed_for(61, seed), n)
    b = mmsgen.splitmix64(mmsgen.seed_for(62, seed), n)

    def keys(lo, hi):
        m = hi - lo
        ids = b[lo:lo + max(m // 3, 1)] >> np.uint64(33)
        return (ids[(a[lo:hi] >> np.uint64(20)) % np.uint64(ids.size)] << np.uint64(32)) | (a[lo:hi] & np.uint64(7))

    x = keys(0, n)
    x[n - top:] = keys(n - top, n) | np.uint64(1 << 63)
    return x[np.argsort(b, kind="stable")]


def reaches(x, r):
    """Whether the last tile's r keys span 2^50 or more and their words (the
    leading 50 bits of the span) leave some of them out of order."""
    s = np.sort(x)[-r:]
    span = int(s[-1] - s[0])
    if span < 1 << 50:
        return False
    p = (s - s[0]) >> np.uint64(span.bit_length() - 50)
    return bool(((p[1:] == p[:-1]) & (s[1:] != s[:-1])).any())


def check(mms, x):
    v = np.arange(x.size, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    xd, vd = (torch.from_numpy(a.view(np.int64)).cuda() for a in (x, v))
    ok, ov = oracle.sort_u64(x, v, i64=False)
    assert np.array_equal(mms.sort64(xd, i64=False).cpu().numpy().view(np.uint64), ok)
    gk, gv = mms.sort_pairs64(xd, vd, i64=False)
    assert np.array_equal(gk.cpu().numpy().view(np.uint64), ok)
    assert np.array_equal(gv.cpu().numpy().view(np.uint64), ov)


@pytest.mark.parametrize("r", [1, 2, 64, 127, 128, 129, 255, 257, 383, 500, 640, 767, 900])
def test_short_last_tile_of_eight_waves(mms, r):
    for tiles in (2, 17):
        n = tiles * TILE + r
        x = shared(n, r, n // 2)
        assert r < 64 or reaches(x, r)
        check(mms, x)


@pytest.mark.parametrize("r", [1, 130, 300, 510])
def test_short_last_tile_of_four_waves(mms, r):
    n = 1100 * TILE + r
    x = shared(n, r, 1500)
    assert r < 64 or reaches(x, r)
    check(mms, x)
