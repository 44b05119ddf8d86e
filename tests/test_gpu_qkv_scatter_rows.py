"""The Q|K|V projection that rotates and scatters its rows itself: active rows anywhere in their sequences (neighbouring rows
in one block of cache slots, in different blocks, whole aligned blocks of sixteen, a ragged last tile), against the
oracle: the block attends to the cache rows it has just written."""
import pytest

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.test_gpu_thin_attention_split import check_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,batch,N,rows", [
    (256, 4, 1, 300, [40]),
    (256, 4, 2, 600, [600, 333]),
    (256, 2, 3, 210, [209, 3, 100]),
    (512, 8, 2, 1200, [1100, 1081]),        # taller tiles
])
def test_rows_anywhere(d, heads, batch, N, rows):
    kernel, splits, _, _, _ = B.sl_linear_plan(sum(rows), 3 * heads * 128, d)
    assert kernel == 1 and splits == 1
    check_block(wl.Shape("scatter", 1, d, heads, 128, 128, 1056, "bf16"), batch, N, rows)
