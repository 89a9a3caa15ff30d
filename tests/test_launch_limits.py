"""Calls whose launches come near 2^32 threads, the most that one may have."""
import numpy as np
import pytest

import paper_1702_07961_amd as mms

torch = pytest.importorskip("torch")

MANY = 1 << 23    # segments: with 512 threads each 2^32


def offsets(ns, long):
    """ns segments of one key, one of them of `long` keys."""
    n = np.ones(ns, dtype=np.uint64)
    n[ns // 3] = long
    return np.concatenate((np.zeros(1, dtype=np.uint64), np.cumsum(n, dtype=np.uint64)))


def align(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("ns,one_pass", [(MANY - 1, True), (MANY, False)])
def test_base_tile_of_many_segments(ns, one_pass):
    """8192-key tiles (512 threads) sort every segment in one pass, if the launch
    holds them; else the batch has a merge round and its table."""
    off = offsets(ns, 5000)
    single = align(int(off[-1]) * 4) + align(align(ns * 64) + ns * 8)
    assert (mms.segmented_workspace_bytes(off) == single) == one_pass


def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.gpu
def test_many_segments_and_one_long():
    gpu()
    off = offsets(MANY, 5000)
    x = torch.empty(int(off[-1]), dtype=torch.int32, device="cuda").random_(-(1 << 31), 1 << 31)
    a = MANY // 3
    want = x.clone()
    want[a:a + 5000] = torch.sort(x[a:a + 5000])[0]
    assert torch.equal(mms.segmented_sort(x, off), want)


@pytest.mark.gpu
def test_most_keys_in_the_smallest_merge_tiles():
    """2^32 - 1 keys in merge tiles of 1024 with the sixteen-wave shape: in order,
    and the same sum of keys and of their squares (mod 2^64)."""
    gpu()
    n = (1 << 32) - 1
    x = torch.empty(n, dtype=torch.int32, device="cuda").random_(-(1 << 31), 1 << 31)

    def sums(t):
        s = [0, 0]
        for c in t.split(1 << 28):
            c = c.to(torch.int64)
            s[0] += int(c.sum())
            s[1] += int((c * c).sum())
        return [v % (1 << 64) for v in s]

    before = sums(x)
    mms.set_tuning([(64, 16, 1024, 1, 6)])
    try:
        mms.sort(x, out=x, i32=True)
        torch.cuda.synchronize()
    finally:
        mms._lib.load_tuning(mms._lib.lib())
    assert sums(x) == before
    last = None
    for c in x.split(1 << 28):
        assert bool((c[1:] >= c[:-1]).all())
        assert last is None or int(c[0]) >= last
        last = int(c[-1])
