"""Layers of few rows whose shape the few-row kernels do not take (too few column slices, or more than one round of them): gate|up
with SwiGLU on ring tiles of every height from 64 to 256 rows, and Q|K|V split over the reduction with RoPE and the cache
write behind it, against the oracle."""
import pytest

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.layer_check import check_layers
from tests.test_wavek_forms_cpu import GATE_UP, PLANES, QKV, form

pytestmark = pytest.mark.gpu

SHAPE = wl.Shape("ring-layers", 1, 1024, 8, 128, 12416, 1056, "bf16")


@pytest.mark.parametrize("rows,gate_up_height,qkv_splits", [(100, 64, 4), (213, 128, 4), (300, 160, 2), (380, 192, 2),
                                                            (420, 224, 2), (500, 256, 2)])
def test_block(rows, gate_up_height, qkv_splits):
    d, H, dff = SHAPE.d_model, SHAPE.n_heads, SHAPE.d_ff
    assert not any(form(*f)[0] for f in ((QKV, rows, H, d), (GATE_UP, rows, dff, d), (PLANES, rows, d, H * 128), (PLANES, rows, d, dff)))
    assert B.sl_linear_plan(rows, 2 * dff, d)[:3] == (1, 1, gate_up_height)
    assert B.sl_linear_plan(rows, 3 * H * 128, d)[:2] == (1, qkv_splits)
    check_layers(SHAPE, 1, rows + 20, [rows], evaluations=2)
