"""Row-block keys merge at its edges, against the oracle: short last runs of
every length around a chunk (4 keys) and an item (62 chunks of a 256-key
block, 30 of a 128-key one), level totals around a whole number of rows, and
keys equal to the one that fills the slots past a piece (0xFFFFFFFF).

Keys have one right order, so the comparison is element by element with no
tolerance."""
import numpy as np
import pytest

import mmsgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T = 2048   # base shape 0
EDGES = [1, 2, 3, 4, 5, 7, 119, 120, 121, 123, 124, 127, 129, 247, 248, 249, 251, 253, 256, 257, 1500]


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
    xd = torch.from_numpy(x.view(np.int32)).cuda()
    assert np.array_equal(mms.sort(xd, i32=False).cpu().numpy().view(np.uint32), oracle.sort(x))
    assert np.array_equal(mms.sort(xd, i32=True).cpu().numpy().view(np.uint32), oracle.sort(x, i32=True))


@pytest.mark.parametrize("variant,K,tout", [(3, 16, 7424), (0, 16, 8192), (1, 8, 6144), (2, 16, 2048), (2, 4, 4096),
                                            (3, 2, 1024)])
def test_row_merge_edges(mms, variant, K, tout):
    mms.set_tuning([(64, K, tout, variant, 0)])
    for i, r in enumerate(EDGES):
        for runs in (1, 3, 16):
            n = runs * T + r
            x = mmsgen.uniform_u32(mmsgen.seed_for(51, i), n)
            check(mms, x)
            # a third of the keys are the largest one, a third of the rest few
            u = mmsgen.uniform_u32(mmsgen.seed_for(52, i), n) % np.uint32(3)
            y = np.where(u == 0, np.uint32(0xFFFFFFFF), np.where(u == 1, x % np.uint32(5), x)).astype(np.uint32)
            check(mms, y)
    check(mms, np.full(5 * T + 77, 0xFFFFFFFF, dtype=np.uint32))
    # every run its own range (levels of one long and many empty pieces), both ways round
    z = np.arange(40 * T + 31, dtype=np.uint32)
    check(mms, z)
    check(mms, z[::-1].copy())
