"""Thin attention of 64 queries per workgroup (more than one round of workgroups of 32): one block whose output is dominated by
its attention, against the oracle, with waves that have no tile, one, an odd number and the most, a workgroup whose second half
of queries holds one row or none, and several sequences."""
import pytest

from paper_2602_06412_amd import workloads as wl
from tests.test_gpu_thin_attention_split import check_block

pytestmark = pytest.mark.gpu

SHAPE = wl.Shape("thin-pairs", 1, 512, 32, 128, 512, 1056, "bf16")


@pytest.mark.parametrize("batch,N,rows", [
    (5, 60, [33, 60, 1, 32, 60]),       # one key tile: two of the four waves have none
    (1, 300, [257]),                    # five tiles, the last one ragged; the last workgroup holds one row
    (2, 1020, [288, 33]),
    (1, 2040, [289]),                   # 32 tiles
])
def test_pairs(batch, N, rows):
    check_block(SHAPE, batch, N, rows)
