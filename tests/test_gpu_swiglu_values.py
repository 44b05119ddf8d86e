"""silu(gate) * up of the three bf16 kernels that apply it (ring and weight-stream epilogues, the kernel behind a k-split
projection) on chosen values.  One block with Out = 0 and down = identity; every row is a single non-zero entry, whose
norm is exactly sqrt(d) at that place, so gate and up of a row are one column of their weights times a power of two and
the block returns silu(gate) * up rounded to bf16 once.

The formula is evaluated in fp32 as g / (1 + exp(-g)) * u: one ulp for the exponential, half a one each for the sum, the
quotient and the product, 2.5 * 2^-23 of the value in all.  Below g = -88.73 the exponential is infinite and the result
a zero, whatever finite u is; g = +inf gives inf * u, g = -inf and NaN give NaN."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, bf16_ulp, weights_to_device

pytestmark = pytest.mark.gpu


def _values(d, rng):
    """gate and up [row, column], bf16 values times sqrt(d)"""
    shape = (d, d)
    g = rng.normal(0.0, 2.0, shape)
    pick = rng.random(shape)
    g = np.where(pick < 0.25, rng.uniform(-88.5, 30.0, shape), g)
    g = np.where(pick < 0.10, rng.uniform(-120.0, -87.0, shape), g)
    g = np.where(pick < 0.02, rng.choice([0.0, 1e-30, -1e-30, 1e4, -1e4], shape), g)
    u = rng.normal(0.0, 1.0, shape) * 10.0 ** rng.uniform(-2, 2, shape)
    u = np.where((g < -90.0) & (rng.random(shape) < 0.5), 1e30, u)
    return tuple((torch.as_tensor(v) / d ** 0.5).bfloat16() for v in (g, u))


@pytest.mark.parametrize("d,rows,swiglu_launches", [(256, 256, 0), (256, 32, 0), (1024, 64, 1)],
                         ids=["ring", "weight-stream", "k-split"])
def test_values(d, rows, swiglu_launches):
    s = wl.Shape("swiglu", 1, d, 2, 128, d, 1056, "bf16")
    w = wl.make_weights(s, seed=1)
    lay = w["layers"][0]
    g, u = _values(d, np.random.default_rng(d + rows))
    g[7, 5], g[9, 5], u[7, 5] = 3e38, -3e38, 1.0                           # overflow: +inf and -inf in those rows
    lay["w_gate"], lay["w_up"] = g.T.contiguous(), u.T.contiguous()        # row r of the batch has its entry at place r
    lay["w_down"], lay["wo"] = torch.eye(d, dtype=torch.bfloat16), torch.zeros_like(lay["wo"])
    lay["ffn_norm"] = torch.ones_like(lay["ffn_norm"])
    x = torch.zeros(rows, d, dtype=torch.bfloat16)
    x[torch.arange(rows), torch.arange(rows)] = 16.0
    last = rows - 1                                                         # a row of NaN, alone in its sequence
    x[last] = float("nan")
    idx = torch.arange(rows, dtype=torch.int32, device=DEV)
    sess = B.Session(s, weights_to_device(w), 2, last)
    m = torch.tensor([rows], dtype=torch.int32, device=DEV)
    B.sl_profile_begin(sess.ctx, 64)
    out = sess.forward_layers(x.to(DEV), idx, m, rows)
    assert B.sl_profile_end(sess.ctx)["swiglu"][1] == swiglu_launches
    got = out.double().cpu().numpy()
    sess.close()
    g64, u64 = (v[:rows].double().numpy() * d ** 0.5 for v in (g, u))
    assert got[7, 5] == np.inf and np.isnan(got[9, 5]) and np.isnan(got[last]).all()
    ok = np.ones((rows, d), dtype=bool)
    ok[[7, 9, last]] = False                                                # 0 * inf in the identity product
    ok[np.arange(rows), np.arange(rows)] = False                            # the residual's own entry
    zero = ok & (g64 < -88.73)
    assert zero.sum() > 100 and np.all(got[zero] == 0.0)
    ok &= g64 > -88.72
    with np.errstate(over="ignore"):
        ref = g64 / (1.0 + np.exp(-g64)) * u64
    err = np.abs(got - ref)
    assert np.all(err[ok] <= (0.5 * bf16_ulp(ref) + 2.5 * 2.0 ** -23 * np.abs(ref))[ok])
