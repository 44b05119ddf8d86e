"""The projections of at most 512 rows whose waves split the reduction (shapes that give 160 to 256 workgroups): every
epilogue against the oracle at the edges of the row blocks, of the passes of 64 rows and of the two-row-tile form (81 rows on),
with rows anywhere, whole aligned blocks of sixteen slots, a ragged last column slice and an odd number of heads."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, weights_to_device
from tests.layer_check import check_layers
from tests.test_gpu_loose_bounds import check_bound
from tests.test_wavek_forms_cpu import GATE_UP, PLANES, form

pytestmark = pytest.mark.gpu

# Q|K|V 162 slices of 64 columns (216 of 96), gate|up 163 of 48 + 48 (the last with 32 of 48)
QKV_GATE_UP = wl.Shape("few-rows", 1, 512, 27, 128, 7808, 1056, "bf16")
# Out and down 42 slices of 64 columns x 4 splits, down with the shortest reduction (four steps)
OUT_DOWN = wl.Shape("few-rows-planes", 1, 2688, 16, 128, 2048, 1056, "bf16")


@pytest.mark.parametrize("batch,N,rows", [
    (1, 300, [1]),
    (1, 300, [17]),
    (2, 130, [31, 18]),
    (1, 300, [80]),
    (1, 300, [81]),
    (1, 300, [97]),
    (2, 128, [128, 128]),       # every slot: V leaves in whole blocks
    (3, 120, [103, 1, 120]),
    (1, 300, [256]),
    (1, 300, [257]),            # gate|up: two row tiles and 2 x 2 waves
    (2, 200, [200, 184]),
    (1, 520, [385]),            # Q|K|V: the ring kernel again
    (1, 520, [512]),
])
def test_qkv_and_gate_up(batch, N, rows):
    check_layers(QKV_GATE_UP, batch, N, rows)


def test_whole_blocks_of_short_sequences():
    """64 slots each: one oracle evaluation is too few to tell how far two correct ones lie apart (tests/layer_check.py)."""
    check_layers(QKV_GATE_UP, 2, 64, [64, 64], evaluations=8)


# 5 trips of the deepest operand ring and 10 of the shorter one in Q|K|V, gate|up and down, 2 and 4 in Out; a reduction that is
# not a power of two; column slices that leave CUs idle.  One row count for each height of each form.
LONG = wl.Shape("few-rows-long", 1, 2560, 32, 128, 10240, 1056, "bf16")
LONG_ROWS = [9, 31, 48, 62, 80, 95, 112, 127, 153, 192, 221, 256, 300, 381, 440, 512]


@pytest.mark.parametrize("rows", LONG_ROWS)
def test_every_height_over_several_trips(rows):
    check_layers(LONG, 1, rows + 9, [rows], evaluations=2)


@pytest.mark.parametrize("d,heads,d_ff", [
    (128, 2, 7808),             # gate|up in two steps of 64 (the other projections need k in whole 128s)
    (384, 2, 7808),             # six
    (2560, 2, 512),             # Out in one step, down in two
    (2560, 6, 1280),            # three, the ring's depth, and five
])
def test_two_by_two_waves_in_few_steps(d, heads, d_ff):
    takes = [form(GATE_UP, 300, d_ff, d), form(PLANES, 300, d, heads * 128), form(PLANES, 300, d, d_ff)]
    assert [f[0] for f in takes] == ([2, 0, 0] if d < 2560 else [0, 2, 2])
    check_layers(wl.Shape("few-steps", 1, d, heads, 128, d_ff, 1056, "bf16"), 1, 300, [300], evaluations=2)


@pytest.mark.parametrize("rows", [[961], [1024]])
def test_gate_up_in_two_full_rounds(rows):
    check_layers(wl.Shape("few-rows-wide", 1, 256, 2, 128, 11008, 1056, "bf16"), 1, 1024, rows)


@pytest.mark.parametrize("rows", [[5], [64], [65], [129], [225], [256], [257], [321], [390], [449], [512]])
def test_out_and_down(rows):
    check_layers(OUT_DOWN, 1, 260 if rows[0] <= 256 else 520, rows)


@pytest.mark.parametrize("m,m_upper", [(0, 200), (40, 200), (199, 200), (260, 300), (299, 300)])
def test_device_side_row_count_below_the_bound(m, m_upper):
    """The rows below it and their K and V as with the tight bound, the rest of the output and of the cache untouched; in
    forms of two row tiles the second lies wholly or partly beyond the count."""
    check_bound(QKV_GATE_UP, 300, m, m_upper)


@pytest.mark.parametrize("locked", [60, 150])
def test_queries_only(locked):
    """The read-only probe of the locked rows against a step that computes the same rows: one layer, the same tokens, so the
    step writes the K and V that are cached already, bit for bit: a row's sums do not depend on its place in the launch or on
    the number of row tiles."""
    s, N = QKV_GATE_UP, 160
    sess = B.Session(s, weights_to_device(wl.make_weights(s, seed=2)), 1, N)
    tokens = torch.as_tensor(wl.prompt_uniform(3, N, s.vocab, s.mask_id), dtype=torch.int32, device=DEV)
    masked, lock = (torch.zeros(N, dtype=torch.uint8, device=DEV) for _ in range(2))
    eps = torch.full((1,), -1.0, device=DEV)
    sess.step(tokens, masked, lock, eps, 1, 0, N, 0, m_upper=N, new_lock=torch.empty_like(lock))
    lock[torch.as_tensor(np.random.default_rng(0).permutation(N)[:locked])] = 1
    torch.cuda.synchronize()
    kv = sess.kv.clone()
    i32 = lambda n: torch.zeros(n, dtype=torch.int32, device=DEV)  # noqa: E731
    idx, cu, logits = i32(N), i32(2), torch.zeros(locked, s.vocab, dtype=torch.bfloat16, device=DEV)
    kl, conf = torch.zeros(N, device=DEV), torch.zeros(N, device=DEV)
    B.sl_unlock_probe(sess.ctx, tokens, lock, i32(N), locked, idx, cu, logits, kl, conf, i32(N), sess.workspace)
    torch.cuda.synchronize()
    assert torch.equal(sess.kv, kv)
    sess.step(tokens, masked, 1 - lock, eps, 2, 0, N, 0, m_upper=locked, new_lock=torch.empty_like(lock))
    torch.cuda.synchronize()
    assert torch.equal(sess.kv, kv)
    assert torch.equal(logits, sess.logits_view(2)[idx[:locked].long()])
    sess.close()


@pytest.mark.parametrize("m,m_upper", [(1, 16), (40, 80), (40, 200), (100, 200), (200, 300)])
def test_row_ids_end_at_the_count(m, m_upper):
    """active_idx of exactly m entries under a larger bound: the same result as with an array of m_upper entries (what lies
    behind the m-th is not the library's to read; that no lane does is shown by the code, which asks for the ids of rows
    below the count only)."""
    sess = B.Session(QKV_GATE_UP, weights_to_device(wl.make_weights(QKV_GATE_UP, seed=1)), 1, 300)
    x = wl.gaussian_rows(1, m_upper, QKV_GATE_UP.d_model, "bf16").to(DEV)
    ids = torch.as_tensor(np.sort(np.random.default_rng(m).permutation(300)[:m_upper]).astype(np.int32), device=DEV)
    got = []
    for idx in (ids, ids[:m].clone()):
        out = torch.zeros_like(x)
        B.sl_forward_layers(sess.ctx, x, out, idx, torch.tensor([m], dtype=torch.int32, device=DEV), m_upper, 0, 1, sess.workspace)
        torch.cuda.synchronize()
        got.append((out, sess.kv.clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    sess.close()
