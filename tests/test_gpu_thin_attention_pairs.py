"""Thin attention of 64 queries per workgroup (more than one round of workgroups of 32): one block whose output is dominated by
its attention, against the oracle, with waves that have no tile, one, an odd number and the most, a workgroup whose second half
of queries holds one row or none, and several sequences."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, weights_to_device
from tests.test_gpu_thin_attention_split import check_block
from tests.test_thin_attention_grid_cpu import form, queries

pytestmark = pytest.mark.gpu

SHAPE = wl.Shape("thin-pairs", 1, 512, 32, 128, 512, 1056, "bf16")


def taken(shape, batch, N, rows):
    """queries per workgroup of a launch whose bound is the row count"""
    splits, grid, may = form(sum(rows), batch, shape.n_heads, -(-N // 64) * 64)
    assert splits == 1 and may
    return queries(rows, shape.n_heads, grid)[1]


@pytest.mark.parametrize("batch,N,rows,width", [
    (5, 60, [33, 60, 1, 32, 60], 32),   # one round of 32 queries, under a bound of more; one key tile: three of the four waves have none
    (5, 60, [33, 60, 33, 32, 60], 64),  # one key tile: two of the four waves have none, and none has a second state
    (8, 150, [33, 60, 32, 1, 33, 33, 33, 33], 64),        # three tiles: one of the pairs' second states has none
    (1, 300, [257], 64),                # five tiles, the last one ragged; the last workgroup holds one row
    (2, 1020, [288, 33], 64),
    (1, 2040, [289], 64),               # 32 tiles
])
def test_pairs(batch, N, rows, width):
    assert taken(SHAPE, batch, N, rows) == width
    check_block(SHAPE, batch, N, rows)


# four heads, so that the workgroups' tiles are searched for among more than 64 tiles or sequences
FEW_HEADS = wl.Shape("thin-pairs-4", 1, 256, 4, 128, 256, 1056, "bf16")


@pytest.mark.parametrize("batch,N,rows,width", [
    (3, 1000, [1000, 980, 80], 64),     # 66 tiles of 32, 34 of 64
    (70, 60, [1] * 70, 32),             # two rounds of either
    (70, 100, [33] * 40 + [1] * 30, 64),                  # 110 tiles of 32 in a grid of 91
    (66, 130, [1] * 60 + [130, 2, 40, 1, 33, 64], 64),    # rows behind the first 64 sequences; 74 tiles of 32 in a grid of 71
])
def test_pairs_among_many_sequences(batch, N, rows, width):
    assert taken(FEW_HEADS, batch, N, rows) == width
    check_block(FEW_HEADS, batch, N, rows)


@pytest.mark.parametrize("N,rows", [(300, [65, 190]), (1020, [1, 255]), (230, [33, 33, 33, 97])])
def test_results_do_not_depend_on_the_form(N, rows):
    """Probes of the same rows over the same keys, alone (one round of workgroups of 32 queries) and beside the other sequences' (64
    queries each, a row bound of more than one round): a row's partial sums are the same four and are added in the same order, so
    the logits are the same bit by bit.  The projections' launches follow the bound, which is equal."""
    batch, total = len(rows), sum(rows)
    assert not form(total, 1, SHAPE.n_heads, -(-N // 64) * 64)[2] and taken(SHAPE, batch, N, rows) == 64
    w = wl.make_weights(SHAPE, seed=4, norm_gain_jitter=0.05)
    lay = w["layers"][0]
    lay["wq"], lay["wo"], lay["w_down"] = lay["wq"] * 4, lay["wo"] * 64, lay["w_down"] * 0
    w = weights_to_device(w)
    one, many = B.Session(SHAPE, w, 1, N).unlock_state(), B.Session(SHAPE, w, batch, N).unlock_state()
    x0 = wl.gaussian_rows(1, N, SHAPE.d_model, "bf16").to(DEV)
    one.forward_layers(x0, torch.arange(N, dtype=torch.int32, device=DEV), torch.tensor([N], dtype=torch.int32, device=DEV), N)
    torch.cuda.synchronize()
    half = SHAPE.n_heads * -(-N // 64) * 64 * 128 * 2                    # K, then V, of a sequence, behind the cos/sin table
    table = one.kv.numel() - 2 * half
    for part in range(2):
        at = table + part * batch * half
        many.kv[at:at + batch * half] = one.kv[table + part * half:table + (part + 1) * half].repeat(batch)
    rng = np.random.default_rng(N)
    tokens = torch.as_tensor(rng.integers(0, SHAPE.vocab, (batch, N)).astype(np.int32), device=DEV)
    picked = torch.zeros(batch, N, dtype=torch.uint8, device=DEV)
    for b, r in enumerate(rows):
        picked[b, torch.as_tensor(rng.permutation(N)[:r], device=DEV)] = 1

    def probe(sess, tok, which):
        sess.probe_logits.fill_(-7.0 if sess is many else -9.0)
        B.sl_unlock_probe(sess.ctx, tok, which, sess.t_lock, total, sess.probe_idx, sess.cu_probe, sess.probe_logits, sess.probe_kl,
                          sess.probe_conf, sess.probe_argmax, sess.workspace)
        torch.cuda.synchronize()
        return sess.probe_logits

    got, at = probe(many, tokens.reshape(-1), picked.reshape(-1)), 0
    for b, r in enumerate(rows):
        alone = probe(one, tokens[b].contiguous(), picked[b].contiguous())
        assert torch.equal(got[at:at + r], alone[:r]), f"sequence {b}: {int((got[at:at + r] != alone[:r]).sum())} logits differ"
        at += r
    one.close(), many.close()
