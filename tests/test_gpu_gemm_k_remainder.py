"""The ring kernel of the projections (launches bounded by more than 32 rows) unrolls its k loop over eight k-tiles of
32 and leaves it early: reductions that are not whole trips, every tile height, ragged rows and columns, against the fp64
product with the bound of tests/test_gpu_linear.py (any summation order of fp32)."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from tests.gpu_util import DEV, bf16_ulp
from tests.test_gpu_linear import _bound, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [256, 384, 640])                           # 8, 12, 20 k-tiles
@pytest.mark.parametrize("rows", [(33, 33), (96, 81), (128, 1), (160, 131), (192, 177), (224, 208), (256, 241)])
@pytest.mark.parametrize("x_tiled", [0, 1])
def test_k_remainders_and_tile_heights(k, rows, x_tiled):
    m_upper, m = rows
    n = 256 * 129 + 96                                                    # enough column tiles for the fitted height, one ragged
    kernel, splits, height, _, _ = B.sl_linear_plan(m_upper, n, k)
    assert (kernel, splits, height) == (1, 1, max(64, (m_upper + 31) // 32 * 32))
    w, x = _inputs(k + m_upper, n, k, m_upper)
    wd, xd = w.to(DEV), x.to(DEV)
    packed = torch.empty_like(wd)
    B.sl_linear_pack(wd, packed)
    xin = B.tile_activations(xd) if x_tiled else xd
    m_dev = torch.tensor([m], dtype=torch.int32, device=DEV)
    y32 = torch.full((1, m_upper, n), float("nan"), device=DEV)
    y16 = torch.full((m_upper, n), -7.0, device=DEV, dtype=torch.bfloat16)
    B.sl_linear_forward(xin, packed, m_dev, m_upper, n, k, 1, y_f32=y32, x_tiled=x_tiled)
    B.sl_linear_forward(xin, packed, m_dev, m_upper, n, k, 1, y_bf16=y16, x_tiled=x_tiled)
    torch.cuda.synchronize()
    x64, w64 = x[:m].double().numpy(), w.double().numpy()
    ref = x64 @ w64.T
    bound = _bound(x64, w64, k)
    assert np.all(np.abs(y32[0, :m].double().cpu().numpy() - ref) <= bound)
    got = y16.double().cpu().numpy()
    assert np.all(np.abs(got[:m] - ref) <= bound + 0.5 * bf16_ulp(ref) * (1 + 1e-9))
    assert np.all(got[m:] == -7.0), "rows beyond the device-side count must not be written"


@pytest.mark.parametrize("k", [320, 448])                                  # 10 and 14 k-tiles: only the cycle probe takes them
def test_probe_k_remainders(k):
    m, n = 70, 256 + 32
    w, x = _inputs(k, n, k, m)
    wd = w.to(DEV)
    packed = torch.empty_like(wd)
    B.sl_linear_pack(wd, packed)
    m_dev = torch.tensor([m], dtype=torch.int32, device=DEV)
    y = torch.zeros(m, n, device=DEV, dtype=torch.bfloat16)
    B.sl_linear_clock_probe(x.to(DEV), packed, m_dev, m, n, k, y, torch.zeros(8, dtype=torch.int64, device=DEV))
    torch.cuda.synchronize()
    x64, w64 = x.double().numpy(), w.double().numpy()
    ref = x64 @ w64.T
    assert np.all(np.abs(y.double().cpu().numpy() - ref) <= _bound(x64, w64, k) + 0.5 * bf16_ulp(ref) * (1 + 1e-9))
