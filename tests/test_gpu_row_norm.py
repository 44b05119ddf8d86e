"""Norm launches of 2049 .. 4096 columns and few planes, whose threads have all of a row's loads under way together: one block
at the narrowest such row (most threads without a second chunk), with and without planes, and a bound above the row count."""
import pytest

from paper_2602_06412_amd import workloads as wl
from tests.layer_check import check_layers
from tests.test_gpu_loose_bounds import check_bound

pytestmark = pytest.mark.gpu

SHAPE = wl.Shape("row-norm", 1, 2176, 2, 128, 1024, 1056, "bf16")


@pytest.mark.parametrize("rows", [[1], [40], [300], [576], [577], [831]])
def test_block(rows):
    check_layers(SHAPE, 1, 840 if rows[0] > 300 else 310, rows)


@pytest.mark.parametrize("m", [0, 37])
def test_rows_past_the_count_stay(m):
    """And the rows below it are those of the tight bound; the cache holds their K and V and nothing else."""
    check_bound(SHAPE, 100, m, 100)
