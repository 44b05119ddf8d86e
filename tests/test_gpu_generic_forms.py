"""The shape-generic projection kernels have two tile forms and an element-wise path for weights that are not 16-byte
aligned: one whole step (every row active) of models whose dimensions leave ragged tiles in each of them, against the
oracle's forward."""
import numpy as np
import pytest
import torch

from oracle import model as om
from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import check_logits, dev, oracle_cfg

pytestmark = pytest.mark.gpu

ODD = dict(n_layers=1, d_model=264, n_heads=3, d_head=32, d_ff=344, vocab=520)          # ragged in every dimension
CASES = [("fp32", ODD, 70), ("bf16", ODD, 70), ("fp32", dict(ODD, vocab=1032), 1050),    # 64 x 64 tiles in the head
         ("bf16", dict(ODD, vocab=1032), 1050)]


def _shifted(t, by):
    """The same values at an address `by` elements past an aligned one."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda:0")
    out = buf[by:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("storage,dims,N", CASES)
@pytest.mark.parametrize("shift", [0, 1])
def test_generic_tile_forms(storage, dims, N, shift):
    shape = wl.Shape("odd-" + storage, storage=storage, **dims)
    w = wl.make_weights(shape, seed=3, norm_gain_jitter=0.05)
    wd = {k: _shifted(v, shift) for k, v in w.items() if k != "layers"}
    wd["layers"] = [{k: _shifted(v, shift) for k, v in l.items()} for l in w["layers"]]
    tokens = wl.prompt_uniform(5, N, shape.vocab, shape.mask_id)
    ref, _, _ = om.forward_full(oracle_cfg(shape), wl.weights_to_numpy64(w), tokens)
    sess = B.Session(shape, wd, 1, N)
    zero = torch.zeros(N, dtype=torch.uint8, device="cuda:0")
    sess.step(dev(tokens, torch.int32), zero.clone(), zero, torch.full((1,), 1e-3, device="cuda:0"), 1, 0, N, 0,
              new_lock=torch.empty_like(zero))
    torch.cuda.synchronize()
    z = sess.logits_view(1).double().cpu().numpy()
    sess.close()
    check_logits(z, np.asarray(ref), storage, f"generic {storage} N={N} shift={shift}")
