"""silu(gate) * up of the bf16 kernels that apply it (ring, weight-stream, waves-along-k and 2 x 2 wave epilogues, the kernel behind a
k-split projection) on chosen values.  One block with Out = 0 and down = identity (of d_ff columns those from `first` on); every row is
a single non-zero entry, whose norm is exactly sqrt(d) at that place (d a power of four), so gate and up of a row are one column of their
weights times a power of two and the block returns silu(gate) * up rounded to bf16 once.

The formula is evaluated in fp32 as g / (1 + exp(-g)) * u.  Below |g| = 87 the exponential is the hardware's 2^x (one ulp) of an argument
reduced to at most a half in two parts, whose last addition rounds by 2^-26 at most (a tenth of an ulp of the result); half an ulp each for
the sum, the quotient (a product with the reciprocal, corrected once) and the product: below 2.75 * 2^-23 of the value in all.  Other
values take the library's exponential and quotient, 2.5 * 2^-23.  Rounded to bf16 such errors show next to a rounding boundary only: what
is tested is that no value takes a formula that fails for it, and both to 2^-9.  Below g = -88.73 the exponential is infinite and the result
a zero, whatever finite u is; g = +inf gives inf * u, g = -inf and NaN give NaN."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, bf16_ulp, weights_to_device
from tests.test_wavek_forms_cpu import GATE_UP, form

pytestmark = pytest.mark.gpu


def _values(d, d_ff, rng):
    """gate and up [row, column], bf16 values times sqrt(d)"""
    shape = (d, d_ff)
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
    check_values(d, d, rows, 0, swiglu_launches)


# 163 workgroups of 48 + 48 columns, or two row tiles of 82 of 96 + 96, the last ones ragged; 1, 3, 9 and 16 blocks of 16 rows
@pytest.mark.parametrize("rows,first,kernel", [(16, 0, 1), (40, 6784, 1), (130, 3000, 1), (256, 6784, 1), (300, 0, 2), (512, 3000, 2),
                                               (512, 6784, 2)])
def test_values_of_few_rows(rows, first, kernel):
    assert form(GATE_UP, rows, 7808, 1024)[0] == kernel
    check_values(1024, 7808, rows, first, 0)


def check_values(d, d_ff, rows, first, swiglu_launches):
    s = wl.Shape("swiglu", 1, d, 2, 128, d_ff, 1056, "bf16")
    w = wl.make_weights(s, seed=1)
    lay = w["layers"][0]
    g, u = _values(d, d_ff, np.random.default_rng(d + rows))
    g[7, first + 5], g[9, first + 5], u[7, first + 5] = 3e38, -3e38, 1.0   # overflow: +inf and -inf in those rows
    lay["w_gate"], lay["w_up"] = g.T.contiguous(), u.T.contiguous()        # row r of the batch has its entry at place r
    lay["w_down"] = torch.eye(d, d_ff, dtype=torch.bfloat16).roll(first, 1)
    lay["wo"] = torch.zeros_like(lay["wo"])
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
    g64, u64 = (v[:rows, first:first + d].double().numpy() * d ** 0.5 for v in (g, u))
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
    assert np.all(err[ok] <= (0.5 * bf16_ulp(ref) + 2.75 * 2.0 ** -23 * np.abs(ref))[ok])
