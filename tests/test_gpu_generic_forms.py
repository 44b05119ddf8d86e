"""The shape-generic projection kernels have two tile forms (16 x 16 and 64 x 64) and an element-wise path for weights that
are not 16-byte aligned: one whole step (every row active) of models whose dimensions leave ragged tiles, against the
oracle's forward.  Q|K|V (three matrices in a launch), gate|up (with SwiGLU) and the head each run in both forms."""
import numpy as np
import pytest
import torch

from oracle import model as om
from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import check_logits, dev, oracle_cfg

pytestmark = pytest.mark.gpu

ODD = dict(n_layers=1, d_model=264, n_heads=3, d_head=32, d_ff=344, vocab=520)          # ragged in every dimension
WIDE = dict(ODD, n_heads=9, d_ff=680, vocab=1032)
# model, rows, launches in the 64 x 64 form; Out and down (264 columns) stay in the 16 x 16 one
CASES = [(storage, dims, N, wide) for dims, N, wide in [(ODD, 70, ()), (dict(ODD, vocab=1032), 1050, ("head",)),
                                                        (WIDE, 1500, ("qkv", "gate_up", "head"))] for storage in ("fp32", "bf16")]


def _wide(n, rows, matrices):
    """The launcher's rule: 16 x 16 tiles up to 1024 workgroups, or while 64 x 64 ones would not fill the chip."""
    tiles = lambda edge: -(-n // edge) * -(-rows // edge) * matrices  # noqa: E731
    return tiles(16) > 1024 and tiles(64) >= 192


def _shifted(t, by):
    """The same values at an address `by` elements past an aligned one."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda:0")
    out = buf[by:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("storage,dims,N,wide", CASES)
@pytest.mark.parametrize("shift", [0, 1])
def test_generic_tile_forms(storage, dims, N, wide, shift):
    shape = wl.Shape("odd-" + storage, storage=storage, **dims)
    hd = shape.n_heads * shape.d_head
    launches = {"qkv": (hd, 3), "out": (shape.d_model, 1), "gate_up": (shape.d_ff, 1), "down": (shape.d_model, 1),
                "head": (shape.vocab, 1)}
    assert tuple(name for name, (n, z) in launches.items() if _wide(n, N, z)) == wide
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
