"""Blocks of a bf16 model against the oracle, row by row (not collected by pytest)."""
import numpy as np
import torch

from oracle import model as om
from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, oracle_cfg, second_evaluation_cfg, weights_to_device


def check_layers(shape, batch, N, rows, evaluations=1):
    """sl_forward_layers on `rows` active rows of each sequence, wherever they lie, after a pass that caches every slot; both
    branches of a block well above the residual's spacing (32 wo, 32 w_down).

    Both sides round the same tensors to bf16; a value near a rounding boundary lands on either neighbour, and the next
    operator carries that on.  How far two correct evaluations of a row then lie apart is measured in the same run, as the
    oracle against itself with sums perturbed by 1e-7 (tests/gpu_util.py): the GPU's rows may be 1.25 times as far from
    the oracle in the median and twice in the worst row.  One wrong 16-byte piece of a normalised row is 4 % of it
    at d = 4096, 18 % at d = 256; two correct evaluations differ by 1 %.

    The rows of a short sequence share their keys and values, so the median over them is nearly one draw: for 64 slots of
    d = 512 eight perturbed evaluations lie at 0 to 3.9e-3.  `evaluations` of them are made and the farthest is the measure."""
    w = wl.make_weights(shape, seed=4, norm_gain_jitter=0.05)
    for lay in w["layers"]:
        lay["wo"], lay["w_down"] = lay["wo"] * 32, lay["w_down"] * 32
    layers64 = wl.weights_to_numpy64(w)["layers"]
    sess = B.Session(shape, weights_to_device(w), batch, N)
    x0 = wl.gaussian_rows(1, batch * N, shape.d_model, "bf16")
    x1 = wl.gaussian_rows(2, batch * N, shape.d_model, "bf16")
    rng = np.random.default_rng(3)
    slots = [np.sort(rng.permutation(N)[:r]) for r in rows]

    def run(x, idx):
        m = torch.tensor([len(idx)], dtype=torch.int32, device=DEV)
        out = sess.forward_layers(x, torch.as_tensor(idx, dtype=torch.int32, device=DEV), m, len(idx))
        torch.cuda.synchronize()
        return out

    assert evaluations >= 1
    run(x0.to(DEV), np.arange(batch * N))                       # fills the caches
    idx = np.concatenate([b * N + s for b, s in enumerate(slots)])
    xin = x1[torch.as_tensor(idx)]
    got = run(xin.to(DEV), idx).double().cpu().numpy()
    sess.close()
    cfg, at = oracle_cfg(shape), 0
    for b, s in enumerate(slots):
        xb, refs = xin[at:at + len(s)].double().numpy(), []
        for c in [cfg] + [second_evaluation_cfg(cfg, seed) for seed in range(evaluations)]:
            full, ref = x0[b * N:(b + 1) * N].double().numpy(), xb
            for lw in layers64:
                Kc, Vc = (np.zeros((N, shape.n_heads, 128)) for _ in range(2))
                full = om.layer_active(c, lw, full, np.arange(N), Kc, Vc)
                ref = om.layer_active(c, lw, ref, s, Kc, Vc)
            refs.append(ref)
        scale = np.linalg.norm(refs[0] - xb, axis=1)
        e, *ys = (np.linalg.norm(z - refs[0], axis=1) / scale for z in [got[at:at + len(s)]] + refs[1:])
        median, largest = max(np.median(y) for y in ys), max(y.max() for y in ys)
        print(f"{shape.name} batch {batch} N {N} rows {rows} heads {shape.n_heads} d_ff {shape.d_ff} sequence {b}: row errors "
              f"median {np.median(e):.2e} largest {e.max():.2e} (row {int(e.argmax())} of {len(s)}), second evaluation "
              f"{median:.2e} {largest:.2e}", flush=True)
        assert np.median(e) <= 1.25 * median and e.max() <= 2.0 * largest
        at += len(s)
