"""Launch parameters and workspace of sorts that one base tile holds (CPU only)."""
import pytest

import paper_1702_07961_amd as mms

TILE = {0: 2048, 1: 2048, 2: 2048, 3: 4096, 5: 4096, 4: 8192, 6: 8192}   # base shape: keys


@pytest.fixture()
def table():
    lib = mms._lib.lib()
    mms._lib.load_tuning(lib)
    yield mms
    mms._lib.load_tuning(lib)


def base(n, pairs=False):
    return mms.get_tuning(n, pairs)[4]


@pytest.mark.parametrize("n", [1, 256, 257, 1000, 1024, 1025, 2048, 2049, 4096])
def test_the_smallest_tile_that_holds_the_keys(table, n):
    """One workgroup sorts them: a larger tile only adds waves that hold nothing."""
    assert TILE[base(n)] == (2048 if n <= 2048 else 4096)


def test_no_workspace_up_to_the_smallest_tile(table):
    """The binding does not ask for these."""
    for pairs in (False, True):
        for shape in TILE:
            table.set_tuning([(64, 16, 8192, 0, shape), (64, 16, 3840, 0, shape, mms.MMS_PAIRS)])
            assert all(table.workspace_bytes(n, pairs) == 0 for n in (1, 1000, mms._ONE_TILE))
        assert table.workspace_bytes(mms._ONE_TILE, pairs, keys64=True) == 0
