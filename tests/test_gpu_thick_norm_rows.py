"""The wave-per-row norm kernel (many rows of d = 4096) leaves four rows at a time through LDS and takes its rows in an order
of its own: row counts that end inside a group of four, of 32 and of 256 rows, against the oracle, row by row.  Both of
its forms feed what is compared: the norm alone (after a projection that added to the residual itself) and add + norm
(after one that left partial sums: too short for the ring kernel, or split), behind the attention as well as between
two blocks."""
import pytest

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.layer_check import check_layers

pytestmark = pytest.mark.gpu


def _adds(m, n, k):
    """The projection leaves fp32 sums: the norm behind it is the form that adds."""
    kernel, splits, _, _, _ = B.sl_linear_plan(m, n, k)
    return kernel != 1 or splits > 1


@pytest.mark.parametrize("batch,N,rows", [(1, 850, [835]), (1, 2110, [2051]), (2, 1200, [1190, 1098])])
@pytest.mark.parametrize("heads,d_ff,out_adds,down_adds", [
    (1, 128, True, True),
    (2, 1024, False, False),
    (2, 128, False, True),
])
def test_row_groups(batch, N, rows, heads, d_ff, out_adds, down_adds):
    M = sum(rows)
    assert _adds(M, 4096, heads * 128) == out_adds and _adds(M, 4096, d_ff) == down_adds
    check_layers(wl.Shape("thick-norm", 2, 4096, heads, 128, d_ff, 1056, "bf16"), batch, N, rows)


def test_split_projections_add_their_planes():
    """down with several planes: k long enough that the plan splits it"""
    M, d_ff = 857, 4096
    assert B.sl_linear_plan(M, 4096, d_ff)[1] > 1
    check_layers(wl.Shape("thick-norm-split", 2, 4096, 2, 128, d_ff, 1056, "bf16"), 1, 900, [M])
