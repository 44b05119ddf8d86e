"""The ring kernel of the projections loads its weights with or without the non-temporal hint, by a rule on its row tiles and
workgroups: every epilogue in the form without it, against fp64 and the oracle, at ragged row counts."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, bf16_ulp
from tests.layer_check import check_layers
from tests.test_gpu_linear import _bound, _inputs

pytestmark = pytest.mark.gpu


def _cached(m_upper, n, k):
    """The rule, restated: more than one row tile and round, and short tiles or more than 3072 rows."""
    kernel, splits, height, cols, _ = B.sl_linear_plan(m_upper, n, k)
    tiles = -(-m_upper // height)
    slots = 8 * tiles * -(-(-(-n // cols)) // 8) * splits
    return kernel == 1 and tiles > 1 and slots > 256 and (height <= 160 or tiles * height > 3072)


@pytest.mark.parametrize("n,k,m_upper,m", [(256 * 129 + 96, 256, 300, 281), (8192, 512, 3300, 3290)])
def test_plain_rows(n, k, m_upper, m):
    assert _cached(m_upper, n, k) and B.sl_linear_splits(m_upper, n, k) == 1
    w, x = _inputs(k + m, n, k, m_upper)
    wd, xd = w.to(DEV), x.to(DEV)
    packed = torch.empty_like(wd)
    B.sl_linear_pack(wd, packed)
    m_dev = torch.tensor([m], dtype=torch.int32, device=DEV)
    y32 = torch.full((1, m_upper, n), float("nan"), device=DEV)
    y16 = torch.full((m_upper, n), -7.0, device=DEV, dtype=torch.bfloat16)
    B.sl_linear_forward(xd, packed, m_dev, m_upper, n, k, 1, y_f32=y32)
    B.sl_linear_forward(B.tile_activations(xd), packed, m_dev, m_upper, n, k, 1, y_bf16=y16, x_tiled=1)
    torch.cuda.synchronize()
    x64, w64 = x[:m].double().numpy(), w.double().numpy()
    ref = x64 @ w64.T
    bound = _bound(x64, w64, k)
    assert np.all(np.abs(y32[0, :m].double().cpu().numpy() - ref) <= bound)
    got = y16.double().cpu().numpy()
    assert np.all(np.abs(got[:m] - ref) <= bound + 0.5 * bf16_ulp(ref) * (1 + 1e-9)) and np.all(got[m:] == -7.0)


@pytest.mark.parametrize("d,heads,d_ff,batch,N,rows,launches", [
    (256, 16, 4096, 3, 1200, [1150, 1100, 1050], ["qkv", "gate_up"]),        # 160- and 224-row tiles
    (4096, 2, 1024, 4, 1200, [1200, 1151, 1130, 1119], ["out", "down"]),     # the residual epilogue
])
def test_fused_epilogues(d, heads, d_ff, batch, N, rows, launches):
    hd, M = heads * 128, sum(rows)
    shapes = {"qkv": (3 * hd, d), "out": (d, hd), "gate_up": (2 * d_ff, d), "down": (d, d_ff)}
    for name in launches:
        assert _cached(M, *shapes[name]) and B.sl_linear_splits(M, *shapes[name]) == 1
    check_layers(wl.Shape("weight-hint", 1, d, heads, 128, d_ff, 1056, "bf16"), batch, N, rows)
