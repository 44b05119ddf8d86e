"""Norm launches of 2049 .. 4096 columns and few planes, which load a row before they look at the row count: one block at the
narrowest such row (most threads without a second chunk), with and without planes, and a bound above the row count."""
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, weights_to_device
from tests.layer_check import check_layers

pytestmark = pytest.mark.gpu

SHAPE = wl.Shape("row-norm", 1, 2176, 2, 128, 1024, 1056, "bf16")


@pytest.mark.parametrize("rows", [[1], [40], [300], [576], [577], [831]])
def test_block(rows):
    check_layers(SHAPE, 1, 840 if rows[0] > 300 else 310, rows)


def test_rows_past_the_count_stay():
    sess = B.Session(SHAPE, weights_to_device(wl.make_weights(SHAPE, seed=1)), 1, 100)
    x = wl.gaussian_rows(1, 100, SHAPE.d_model, "bf16").to(DEV)
    idx = torch.arange(100, dtype=torch.int32, device=DEV)
    for m in (0, 37):
        out = torch.full_like(x, -7.0)
        B.sl_forward_layers(sess.ctx, x, out, idx, torch.tensor([m], dtype=torch.int32, device=DEV), 100, 0, 1, sess.workspace)
        torch.cuda.synchronize()
        assert bool((out[m:] == -7.0).all()) and bool(torch.isfinite(out[:m].float()).all())
    sess.close()
