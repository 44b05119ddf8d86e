"""Thin attention launches of long sequences (more than 16 key tiles): one workgroup per 32 queries and head, its keys
split over further workgroups.  One block whose output is dominated by its attention, against the oracle, at the edges of
query tiles, of key splits (a last one that is shorter, a wave without a tile) and of the batch."""
import numpy as np
import pytest
import torch

from oracle import model as om
from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, oracle_cfg, weights_to_device

pytestmark = pytest.mark.gpu

CASES = [  # sequences, slots, active rows of each sequence
    (1, 1030, [1]),
    (1, 1100, [33]),            # 18 tiles: five splits, the last of two tiles
    (1, 1100, [1100]),          # unsplit: more than 128 workgroups
    (1, 2048, [64]),
    (3, 1090, [31, 1, 70]),     # 18 tiles over six query tiles' worth of workgroups
    (1, 2300, [2300]),          # beyond one workgroup per CU: the pipelined kernel
]


def check_block(shape, batch, N, rows):
    """One block over `rows` active rows of each sequence, wherever they lie, with every slot's K and V cached before."""
    w = wl.make_weights(shape, seed=4, norm_gain_jitter=0.05)
    lay = w["layers"][0]
    lay["wq"], lay["wo"], lay["w_down"] = lay["wq"] * 4, lay["wo"] * 64, lay["w_down"] * 0
    w64 = wl.weights_to_numpy64(w)["layers"][0]
    sess = B.Session(shape, weights_to_device(w), batch, N)
    x0 = wl.gaussian_rows(1, batch * N, shape.d_model, "bf16")
    x1 = wl.gaussian_rows(2, batch * N, shape.d_model, "bf16")
    rng = np.random.default_rng(3)
    slots = [np.sort(rng.permutation(N)[:r]) for r in rows]

    def run(x, idx):
        out = torch.empty_like(x)
        m = torch.tensor([len(idx)], dtype=torch.int32, device=DEV)
        B.sl_forward_layers(sess.ctx, x, out, torch.as_tensor(idx, dtype=torch.int32, device=DEV), m, len(idx), 0, 1, sess.workspace)
        torch.cuda.synchronize()
        return out

    run(x0.to(DEV), np.arange(batch * N))                       # fills the caches
    idx = np.concatenate([b * N + s for b, s in enumerate(slots)])
    xin = x1[torch.as_tensor(idx)]
    got = run(xin.to(DEV), idx).double().cpu().numpy()
    sess.close()
    cfg, at = oracle_cfg(shape), 0
    for b, s in enumerate(slots):
        Kc, Vc = (np.zeros((N, shape.n_heads, 128)) for _ in range(2))
        om.layer_active(cfg, w64, x0[b * N:(b + 1) * N].double().numpy(), np.arange(N), Kc, Vc)
        xb = xin[at:at + len(s)].double().numpy()
        ref = om.layer_active(cfg, w64, xb, s, Kc, Vc)
        # q, k, v, o and the result are rounded to bf16 on both sides; where the unrounded values straddle a rounding
        # boundary they land one spacing (2^-8 of the value) apart, in the 2-norm at most that for all five together
        # as each flips for a few elements only; twice that is allowed
        rel = np.linalg.norm(got[at:at + len(s)] - ref) / np.linalg.norm(ref - xb)
        print(f"{shape.name} batch {batch} N {N} rows {rows} heads {shape.n_heads} sequence {b}: {rel:.2e}", flush=True)
        assert rel <= 2.0 ** -7
        at += len(s)


@pytest.mark.parametrize("heads", [4, 9])
@pytest.mark.parametrize("batch,N,rows", CASES)
def test_thin_attention_with_split_keys(batch, N, rows, heads):
    check_block(wl.Shape("thin-attention", 1, 512, heads, 128, 128, 1056, "bf16"), batch, N, rows)
