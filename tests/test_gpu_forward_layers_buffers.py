"""sl_forward_layers runs on the output buffer itself when it can: separate buffers, the same buffer in and out, overlapping
ones and ones the 16-byte row kernels cannot take must all give the same rows bit for bit, leave the input alone (unless
it is the output) and write no row beyond the device-side count."""
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, weights_to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [wl.S_BF16, wl.C1], ids=lambda s: s.name)
@pytest.mark.parametrize("rows", [5, 130])
def test_input_and_output_buffers(shape, rows):
    N, upper, d = 192, rows + 3, shape.d_model
    w = weights_to_device(wl.make_weights(shape, seed=2, norm_gain_jitter=0.05))
    sess = B.Session(shape, w, 1, N)
    x = wl.gaussian_rows(7, upper, d, shape.storage).to(DEV)
    idx = torch.arange(0, upper, dtype=torch.int32, device=DEV)
    m = torch.tensor([rows], dtype=torch.int32, device=DEV)

    def run(src, dst):
        B.sl_forward_layers(sess.ctx, src, dst, idx, m, upper, 0, shape.n_layers, sess.workspace)
        torch.cuda.synchronize()

    out = torch.full_like(x, -7.0)
    before = x.clone()
    run(x, out)
    assert torch.equal(x, before) and bool((out[rows:] == -7.0).all()) and bool(torch.isfinite(out[:rows]).all())
    ref = out[:rows].clone()
    same = x.clone()
    run(same, same)
    assert torch.equal(same[:rows], ref) and torch.equal(same[rows:], x[rows:])
    big = torch.empty(upper * d + d, dtype=x.dtype, device=DEV)             # output one row behind the input: overlapping
    src, dst = big[d:].view(upper, d), big[:upper * d].view(upper, d)
    src.copy_(x)
    run(src, dst)
    assert torch.equal(dst[:rows], ref)
    odd_in, odd_out = (torch.empty(upper * d + 1, dtype=x.dtype, device=DEV)[1:].view(upper, d) for _ in range(2))
    for a, b in ((odd_in, odd_out), (odd_in, torch.empty_like(x)), (x, odd_out)):
        a.copy_(x)
        b.fill_(-7.0)
        run(a, b)
        assert torch.equal(b[:rows], ref) and bool((b[rows:] == -7.0).all())
    sess.close()
