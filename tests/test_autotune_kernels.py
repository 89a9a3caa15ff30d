"""The autotuner's candidates name every merge kernel once (CPU only)."""
import json

import pytest

from paper_1702_07961_amd import autotune


@pytest.mark.parametrize("tile,kernels", [(2048, [0, 1, 2, 4]), (4096, [0, 1, 4]), (7424, [0, 1, 4]), (8192, [0, 4])])
def test_one_name_for_a_kernel(tile, kernels):
    """launch_merge_keys: sixteen waves (1) up to 7424, eight waves of 128-key blocks
    (2) up to 3584, the heap (4), and one kernel for all else."""
    assert [v for v in autotune.VARIANTS if autotune.kernel_of(tile, v) == v] == kernels


def test_the_table_names_kernels_that_run():
    with open(autotune.DEFAULT_TABLE) as f:
        table = json.load(f)
    for e in table["entries"]:
        assert e["variant"] == autotune.kernel_of(e["merge_tile"], e["variant"])
