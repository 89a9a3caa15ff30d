"""64-bit keys whose merge tiles span just below, at and above 2^62, where the
words stop being the whole keys, with ties, with the key that the sentinel
equals, and with keys that differ in their low bits only.  Both merge kernels:
eight waves up to 1024 tiles of a round, four above.  Element by element
against the oracle (keys) and NumPy's sort where the oracle would take long."""
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


def check(mms, x, want):
    got = mms.sort64(torch.from_numpy(x.view(np.int64)).cuda(), i64=False)
    assert np.array_equal(got.cpu().numpy().view(np.uint64), want)


def two_ends(n, seed, base, span, low):
    """Half the keys within `low` of base, half within `low` of base + span, and
    both ends themselves: a tile of every merge group holds some of both."""
    u = mmsgen.splitmix64(mmsgen.seed_for(63, seed), n)
    d = (u >> np.uint64(8)) % np.uint64(low)
    x = np.where(u & np.uint64(1), np.uint64(base + span) - d, np.uint64(base) + d).astype(np.uint64)
    x[: n // 50] = np.uint64(base)
    x[n // 50: n // 25] = np.uint64(base + span)
    return x[np.argsort(u >> np.uint64(1), kind="stable")]


SPANS = [(1 << 62) - 2, (1 << 62) - 1, 1 << 62, (1 << 62) + 1, (1 << 64) - 1]


@pytest.mark.parametrize("span", SPANS)
@pytest.mark.parametrize("low", [3, 1 << 13, 1 << 40])
def test_spans_of_eight_waves(mms, span, low):
    base = min(12345, (1 << 64) - 1 - span)
    for n in (4097, 5 * 4096 + 77, 3 * 16 * 4096 + 1999):
        x = two_ends(n, n, base, span, low)
        check(mms, x, oracle.sort_u64(x, i64=False))


@pytest.mark.parametrize("span", SPANS)
def test_spans_of_four_waves(mms, span):
    base = min(12345, (1 << 64) - 1 - span)
    for low in (5, 1 << 14):
        x = two_ends(1030 * 3456 + 321, 7, base, span, low)
        check(mms, x, np.sort(x))
