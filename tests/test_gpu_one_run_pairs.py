"""Keys merge tiles in which some pairs of runs have one empty run, which the
256-key blocks leave where they are: runs of disjoint ranges (in any order of
the runs), half of the runs interleaved, and a few keys out of place, with odd
counts of runs and a short last one.

Keys have one right order, so the comparison is element by element with no
tolerance."""
import numpy as np
import pytest

import mmsgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T = 2048   # base shape 0


@pytest.fixture(scope="module")
def mms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_07961_amd as m
    m._lib.lib()
    yield m
    m.set_tuning([])
    m._lib.load_tuning(m._lib.lib())


def inputs(runs, tail, seed):
    """Keys in runs of T, the last one of `tail`."""
    n = (runs - 1) * T + tail
    rng = np.random.default_rng(seed)
    ranks = np.arange(n, dtype=np.uint32)
    by_run = [ranks[r * T:min(n, (r + 1) * T)] for r in range(runs)]
    full = rng.permutation(runs - 1)
    shuffled = np.concatenate([by_run[r] for r in full] + [by_run[-1]])      # disjoint ranges
    half = shuffled.copy()
    m = (runs - 1) // 2 * T
    half[:m] = rng.permutation(half[:m])                                     # half of the runs interleave
    swapped = ranks.copy()
    i, j = rng.integers(0, n, 7), rng.integers(0, n, 7)
    for a, b in zip(i, j):
        swapped[a], swapped[b] = swapped[b], swapped[a]
    return {"sorted": ranks, "shuffled": shuffled, "half": half, "swapped": swapped}


@pytest.mark.parametrize("K", [2, 4, 16])
@pytest.mark.parametrize("tout", [1024, 7424, 8192])
def test_one_run_pairs(mms, K, tout):
    mms.set_tuning([(64, K, tout, 3, 0)])
    for runs in (2, 3, 16, 21):
        for tail in (1, 1023, T):
            for name, x in inputs(runs, tail, mmsgen.seed_for(61, runs) & 0xFFFF).items():
                xd = torch.from_numpy(x.view(np.int32)).cuda()
                got = mms.sort(xd, i32=False).cpu().numpy().view(np.uint32)
                assert np.array_equal(got, oracle.sort(x)), (runs, tail, name)
