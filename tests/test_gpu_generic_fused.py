"""fp32 layers of few tiles carry RMSNorm, RoPE with the cache scatter and the residual adds in their projections; a layer whose
weights are not 16-byte aligned has launches of its own for them.  Whole steps against the oracle's forward: every head size, reductions
of one, several and more load trips, ragged dimensions, and models whose layers and head differ in that; the launches are counted.
Layers alone: several sequences, rows anywhere, slots cached before, bounds above the row count."""
import numpy as np
import pytest
import torch

from oracle import model as om
from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, check_logits, dev, oracle_cfg, weights_to_device
from tests.test_gpu_generic_forms import _shifted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shifts", [(0, 0, 0), (0, 1, 0), (1, 0, 1)])          # elements off alignment: layer 0, layer 1, head
@pytest.mark.parametrize("d,heads,dh,d_ff,rows", [(248, 3, 32, 264, 70), (264, 2, 64, 768, 17), (256, 1, 128, 688, 16), (40, 1, 256, 776, 1),
                                              (520, 2, 256, 768, 33), (768, 17, 32, 1000, 16)])    # nine to twelve chunks a wave at once
def test_fused_layers(d, heads, dh, d_ff, rows, shifts):
    shape = wl.Shape("fused", 2, d, heads, dh, d_ff, 136, "fp32")
    w = wl.make_weights(shape, seed=6, norm_gain_jitter=0.05)
    wd = {k: _shifted(v, shifts[2]) for k, v in w.items() if k != "layers"}
    wd["layers"] = [{k: _shifted(v, shifts[i]) for k, v in l.items()} for i, l in enumerate(w["layers"])]
    tokens = wl.prompt_uniform(5, rows, shape.vocab, shape.mask_id)
    ref, _, _ = om.forward_full(oracle_cfg(shape), wl.weights_to_numpy64(w), tokens)
    sess = B.Session(shape, wd, 1, rows)
    zero = torch.zeros(rows, dtype=torch.uint8, device="cuda:0")
    B.sl_profile_begin(sess.ctx, 64)
    sess.step(dev(tokens, torch.int32), zero.clone(), zero, torch.full((1,), 1e-3, device="cuda:0"), 1, 0, rows, 0,
              new_lock=torch.empty_like(zero))
    launches = {name: n for name, (_, n) in B.sl_profile_end(sess.ctx).items()}
    # a layer of its own launches has one of RoPE and two of add + norm; a fused one has a norm where an unfused layer or head reads
    # its rows
    fused = [s == 0 for s in shifts[:2]] + [shifts[2] == 0 == shifts[1]]
    assert launches["rope_kv"] == sum(not f for f in fused[:2])
    assert launches["add_norm"] == sum((0 if fused[i + 1] else 1) if fused[i] else 2 for i in range(2))
    z = sess.logits_view(1).double().cpu().numpy()
    sess.close()
    check_logits(z, np.asarray(ref), "fp32", f"fused d={d} dh={dh} rows={rows} shifts={shifts}")


@pytest.mark.parametrize("shifts", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("heads,dh,batch,N,rows,bound", [
    (3, 32, 3, 37, [5, 0, 30], 35),             # no row in a sequence; no room to spare
    (2, 64, 2, 130, [17, 70], 200),
    (1, 128, 4, 66, [1, 66, 16, 40], 250),
    (1, 256, 2, 90, [33, 12], 46),
])
def test_layers_of_scattered_rows(heads, dh, batch, N, rows, bound, shifts):
    """Sums of at most 312 fp32 terms, relative error 2^-24 sqrt(312) at most a few times; five in a chain, twice: below 2e-5 of the
    branches' own size.  A row of another sequence or slot is above 0.1."""
    shape = wl.Shape("fused-layers", 2, 264, heads, dh, 312, 136, "fp32")
    w = wl.make_weights(shape, seed=6, norm_gain_jitter=0.05)
    for lay in w["layers"]:                               # both branches of the residual's own size
        lay["wo"], lay["w_down"] = lay["wo"] * 8, lay["w_down"] * 32
    w64, wd = wl.weights_to_numpy64(w)["layers"], weights_to_device(w)
    wd["layers"] = [{k: _shifted(v, shifts[i]) for k, v in l.items()} for i, l in enumerate(w["layers"])]
    sess, cfg, rng = B.Session(shape, wd, batch, N), oracle_cfg(shape), np.random.default_rng(N)
    slots = [np.sort(rng.permutation(N)[:r]) for r in rows]
    M, x0 = sum(rows), wl.gaussian_rows(1, batch * N, shape.d_model, "fp32")
    every = torch.arange(batch * N, dtype=torch.int32, device=DEV)
    sess.forward_layers(x0.to(DEV), every, torch.tensor([batch * N], dtype=torch.int32, device=DEV), batch * N)
    x = wl.gaussian_rows(2, bound, shape.d_model, "fp32")
    out, ids = torch.full((bound, shape.d_model), -7.0, device=DEV), torch.zeros(bound, dtype=torch.int32, device=DEV)
    ids[:M] = torch.as_tensor(np.concatenate([b * N + s for b, s in enumerate(slots)]), dtype=torch.int32, device=DEV)
    B.sl_profile_begin(sess.ctx, 64)
    B.sl_forward_layers(sess.ctx, x.to(DEV), out, ids, torch.tensor([M], dtype=torch.int32, device=DEV), bound, 0, 2, sess.workspace)
    assert B.sl_profile_end(sess.ctx)["rope_kv"][1] == sum(s != 0 for s in shifts)
    assert bool((out[M:] == -7.0).all())
    kv, at = [[t.double().cpu().numpy() for t in sess.kv_read(l)] for l in range(2)], 0
    got, x64 = out[:M].double().cpu().numpy(), x.double().numpy()
    sess.close()
    rel = lambda a, b: np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)  # noqa: E731
    for b, s in enumerate(slots):
        full, ref = x0[b * N:(b + 1) * N].double().numpy(), x64[at:at + len(s)]
        for l in range(2):
            Kc, Vc = np.zeros((N, heads, dh)), np.zeros((N, heads, dh))
            full = om.layer_active(cfg, w64[l], full, np.arange(N), Kc, Vc)
            if len(s):
                ref = om.layer_active(cfg, w64[l], ref, s, Kc, Vc)
            errors = rel(kv[l][0][b], Kc), rel(kv[l][1][b], Vc)
            print(f"layers dh={dh} shifts={shifts} sequence {b} layer {l}: K {errors[0]:.1e} V {errors[1]:.1e}", flush=True)
            assert max(errors) < 2e-5
        if len(s):
            e = rel(got[at:at + len(s)] - x64[at:at + len(s)], ref - x64[at:at + len(s)])
            print(f"layers dh={dh} shifts={shifts} sequence {b}: rows {e:.1e}", flush=True)
            assert e < 2e-5
        at += len(s)
