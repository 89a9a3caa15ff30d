"""Merge levels of keys that need several passes: 16 runs whose shares of the
keys' lower half follow the weights of their pairs, so the tiles there have
uneven pieces, many of a size just past a whole number of items (248 keys, or
120 in the smaller blocks), and more items than a workgroup has rows.  Every
block shape at its smallest and largest merge tile.

Sorted keys are unique, so the comparison is element by element with no
tolerance."""
import numpy as np
import pytest

import mmsgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T = 8192   # base shape 6
WEIGHTS = [(1, 1, 1, 1, 1, 1, 1, 1), (30, 1, 1, 1, 1, 1, 1, 1), (1, 1, 1, 1, 1, 1, 1, 30), (9, 1, 9, 1, 9, 1, 9, 1),
           (17, 16, 17, 16, 17, 16, 17, 16)]


@pytest.fixture(scope="module")
def mms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_07961_amd as m
    m._lib.lib()
    yield m
    m.set_tuning([])
    m._lib.load_tuning(m._lib.lib())


@pytest.mark.parametrize("variant,tout", [(3, 1024), (3, 7424), (3, 7680), (3, 7936), (0, 8192), (1, 1024), (1, 7424),
                                          (1, 7680), (2, 1024), (2, 3584), (2, 3840)])
def test_uneven_pairs(mms, variant, tout):
    mms.set_tuning([(64, 16, tout, variant, 6)])
    for j, weights in enumerate(WEIGHTS):
        x = mmsgen.uniform_u32(mmsgen.seed_for(57, j), 16 * T).reshape(16, T)
        for k in range(16):
            low = T * weights[k // 2] // (2 * max(weights))
            x[k, :low] >>= np.uint32(1)
            x[k, low:] |= np.uint32(0x80000000)
        x = np.ascontiguousarray(x).reshape(-1)
        xd = torch.from_numpy(x.view(np.int32)).cuda()
        for i32 in (False, True):
            assert np.array_equal(mms.sort(xd, i32=i32).cpu().numpy().view(np.uint32), oracle.sort(x, i32=i32)), weights
