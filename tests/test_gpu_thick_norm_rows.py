"""The wave-per-row norm kernel (800 rows and more of d = 4096) leaves four rows at a time through LDS and takes its rows in
an order of its own: row counts that end inside a group of four, of 32 and of 256 rows, against the oracle."""
import pytest

from paper_2602_06412_amd import workloads as wl
from tests.test_gpu_thin_attention_split import check_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,N,rows", [(1, 2110, [2051]), (1, 810, [801]), (2, 1200, [1190, 1098])])
def test_row_groups(batch, N, rows):
    check_block(wl.Shape("thick-norm", 1, 4096, 2, 128, 128, 1056, "bf16"), batch, N, rows)
