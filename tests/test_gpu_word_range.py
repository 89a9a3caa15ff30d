"""64-bit sorts at the range of keys that a word holds in full (2^50): tiles
whose keys span just less, as much, and more than that, ties among them, at
both ends of the 64-bit range and across the sign bit, against the oracle.

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


def keys(span, low, ties, n):
    """n keys in [low, low + span], both ends taken, half of them from few values."""
    r = mmsgen.splitmix64(mmsgen.seed_for(62, 1), n)
    x = r % np.uint64(span) if span < 2**64 - 1 else r
    if ties:
        few = x[:37].copy()
        x = np.where(r >> np.uint64(63) == 0, x, few[(r % np.uint64(37)).astype(np.int64)])
    x[n // 3], x[n // 2], x[-1], x[0] = 0, span, span, 0
    return x + np.uint64(low)


@pytest.mark.parametrize("span", [2**50 - 2, 2**50 - 1, 2**50, 2**50 + 1, 2**51, 2**40, 1])
@pytest.mark.parametrize("low", [0, 2**63 - 2**49, 2**64 - 2**51 - 1])
def test_keys_of_a_span(mms, span, low):
    for n in (4096, 4099, 5 * 4096 + 1, 20 * 4096 + 2047):
        for ties in (False, True):
            x = keys(span, low, ties, n)
            v = np.arange(n, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
            xd, vd = (torch.from_numpy(a.view(np.int64)).cuda() for a in (x, v))
            for i64 in (False, True):
                ok, ov = oracle.sort_u64(x, v, i64=i64)
                assert np.array_equal(mms.sort64(xd, i64=i64).cpu().numpy().view(np.uint64), ok), (n, ties, i64)
                gk, gv = mms.sort_pairs64(xd, vd, i64=i64)
                assert np.array_equal(gk.cpu().numpy().view(np.uint64), ok), (n, ties, i64)
                assert np.array_equal(gv.cpu().numpy().view(np.uint64), ov), (n, ties, i64)
