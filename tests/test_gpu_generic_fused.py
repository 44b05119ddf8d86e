"""fp32 layers of few tiles carry RMSNorm, RoPE with the cache scatter and the residual adds in their projections; a layer whose
weights are not 16-byte aligned has launches of its own for them.  Whole steps against the oracle's forward: every head size, reductions
of one, several and more load trips, ragged dimensions, and models whose layers and head differ in that."""
import numpy as np
import pytest
import torch

from oracle import model as om
from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import check_logits, dev, oracle_cfg
from tests.test_gpu_generic_forms import _shifted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shifts", [(0, 0, 0), (0, 1, 0), (1, 0, 1)])          # elements off alignment: layer 0, layer 1, head
@pytest.mark.parametrize("d,heads,dh,d_ff,rows", [(248, 3, 32, 264, 70), (264, 2, 64, 768, 17), (256, 1, 128, 688, 16), (40, 1, 256, 776, 1)])
def test_fused_layers(d, heads, dh, d_ff, rows, shifts):
    shape = wl.Shape("fused", 2, d, heads, dh, d_ff, 136, "fp32")
    w = wl.make_weights(shape, seed=6, norm_gain_jitter=0.05)
    wd = {k: _shifted(v, shifts[2]) for k, v in w.items() if k != "layers"}
    wd["layers"] = [{k: _shifted(v, shifts[i]) for k, v in l.items()} for i, l in enumerate(w["layers"])]
    tokens = wl.prompt_uniform(5, rows, shape.vocab, shape.mask_id)
    ref, _, _ = om.forward_full(oracle_cfg(shape), wl.weights_to_numpy64(w), tokens)
    sess = B.Session(shape, wd, 1, rows)
    zero = torch.zeros(rows, dtype=torch.uint8, device="cuda:0")
    sess.step(dev(tokens, torch.int32), zero.clone(), zero, torch.full((1,), 1e-3, device="cuda:0"), 1, 0, rows, 0,
              new_lock=torch.empty_like(zero))
    torch.cuda.synchronize()
    z = sess.logits_view(1).double().cpu().numpy()
    sess.close()
    check_logits(z, np.asarray(ref), "fp32", f"fused d={d} dh={dh} rows={rows} shifts={shifts}")
