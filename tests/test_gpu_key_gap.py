"""64-bit base tiles whose keys leave a run of bits at zero, so that the rest
may fit the tile's words though the range does not: runs just too short, just
long enough and longer, at the bottom, in the middle and below the top bits,
two of them, and a run of ones, for which there is no such form.

Keys have one right order and pairs one stable order, so the comparison is
element by element with no tolerance."""
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


def mask(lo, hi):
    return ((1 << hi) - 1) ^ ((1 << lo) - 1)


def keys(n, varying, ties, constant=0):
    """n keys of which the bits of `varying` vary; with ties few values of the
    top half of them."""
    x = mmsgen.splitmix64(mmsgen.seed_for(64, n), n)
    if ties:
        few = x[: max(n // 30, 1)] & np.uint64(0xFFFFFFFF00000000)
        x = few[(x % np.uint64(few.size)).astype(np.int64)] | (x & np.uint64(0xFFFFFFFF))
    return (x & np.uint64(varying)) | np.uint64(constant)


# (first bit of the run, its length) for keys of 64 varying bits
RUNS = [(0, 13), (0, 14), (0, 40), (1, 13), (1, 14), (10, 13), (10, 14), (10, 22), (18, 14), (36, 14), (37, 14), (37, 26),
        (49, 14), (50, 13), (2, 61)]


@pytest.mark.parametrize("run", RUNS)
@pytest.mark.parametrize("ones", [False, True])
def test_runs_of_bits(mms, run, ones):
    gap = mask(run[0], run[0] + run[1])
    for top in (64, 57):     # the bits above `top` are zero too
        varying = mask(0, top) & ~gap
        for n in (2, 65, 1500, 4096, 2 * 4096 + 7):
            for ties in (False, True):
                check(mms, keys(n, varying, ties, gap & mask(0, top) if ones else 0))


def test_two_runs(mms):
    for gaps in ((3, 8, 20, 34), (3, 17, 30, 36), (0, 7, 20, 27)):
        varying = mask(0, 64) & ~mask(gaps[0], gaps[1]) & ~mask(gaps[2], gaps[3])
        check(mms, keys(4000, varying, True))


def check(mms, x):
    v = np.arange(x.size, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    xd, vd = (torch.from_numpy(a.view(np.int64)).cuda() for a in (x, v))
    for i64 in (False, True):
        ok, ov = oracle.sort_u64(x, v, i64=i64)
        assert np.array_equal(mms.sort64(xd, i64=i64).cpu().numpy().view(np.uint64), ok)
        gk, gv = mms.sort_pairs64(xd, vd, i64=i64)
        assert np.array_equal(gk.cpu().numpy().view(np.uint64), ok)
        assert np.array_equal(gv.cpu().numpy().view(np.uint64), ov)
