"""A row bound above the row count: the rows below the count come out as under the tight bound (other launch plans sum in
another order: rounding), the new K and V of these rows land in the cache, and nothing else is written, neither the rows of the
output past the count nor the cache slots of ids past it."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from paper_2602_06412_amd import workloads as wl
from tests.gpu_util import DEV, weights_to_device

pytestmark = pytest.mark.gpu

_SESSIONS = {}


def _session(shape, N):
    key = (shape, N)
    if key not in _SESSIONS:
        for s in _SESSIONS.values():
            s.close()
        _SESSIONS.clear()
        w = wl.make_weights(shape, seed=1)
        for lay in w["layers"]:                       # both branches well above the residual's spacing
            lay["wo"], lay["w_down"] = lay["wo"] * 32, lay["w_down"] * 32
        sess = _SESSIONS[key] = B.Session(shape, weights_to_device(w), 1, N)
        x0 = wl.gaussian_rows(1, N, shape.d_model, "bf16").to(DEV)
        sess.forward_layers(x0, torch.arange(N, dtype=torch.int32, device=DEV), torch.tensor([N], dtype=torch.int32, device=DEV), N)
        torch.cuda.synchronize()
        sess.kv0 = sess.kv.clone()
    return _SESSIONS[key]


def _run(sess, x, ids, m, m_upper):
    sess.kv.copy_(sess.kv0)
    out = torch.full((m_upper, x.shape[1]), -7.0, dtype=x.dtype, device=DEV)
    xin = torch.full((m_upper, x.shape[1]), 3.0, dtype=x.dtype, device=DEV)
    xin[:m] = x[:m]
    B.sl_forward_layers(sess.ctx, xin, out, ids[:m_upper].clone(), torch.tensor([m], dtype=torch.int32, device=DEV), m_upper, 0, 1,
                        sess.workspace)
    torch.cuda.synchronize()
    return out, [t[0].clone() for t in sess.kv_read(0)]


def check_bound(shape, N, m, m_upper):
    sess = _session(shape, N)
    ids = torch.as_tensor(np.random.default_rng(m_upper).permutation(N).astype(np.int32), device=DEV)
    ids[:m] = ids[:m].sort().values
    x = wl.gaussian_rows(2, N, shape.d_model, "bf16").to(DEV)
    loose, kv = _run(sess, x, ids, m, m_upper)
    again, _ = _run(sess, x, ids, m, m_upper)
    assert torch.equal(loose, again) and bool((loose[m:] == -7.0).all())
    sess.kv.copy_(sess.kv0)
    before = [t[0].clone() for t in sess.kv_read(0)]
    rest = torch.ones(N, dtype=torch.bool, device=DEV)
    rest[ids[:m].long()] = False
    for a, b in zip(kv, before):                      # K, V
        assert torch.equal(a[rest], b[rest])
        assert m == 0 or not torch.equal(a[~rest], b[~rest])
    if m == 0:
        return
    tight, kv_tight = _run(sess, x, ids, m, m)
    # one layer: K and V are roundings of one projection's sums.  Where the two bounds sum in another order (fp32, k terms of
    # about the same size: relative 2^-24 sqrt(k) at most a few times) a value next to a rounding boundary moves by one bf16
    # spacing, 2^-8 relative: less than 1 % of them
    for a, b in zip(kv, kv_tight):
        a, b = a[~rest].double(), b[~rest].double()
        moved = (a - b).abs()
        assert bool((moved <= 2.0 ** -7 * b.abs() + 1e-4).all()) and float((moved > 0).double().mean()) < 0.01
    # rows: every stored value of the block (bf16) may move by a spacing, 2^-9 relative rms; through five roundings in a chain
    # below 1e-2 of the branches' own size, a 16-row block or a k-slice left out is above 0.1
    e = (loose[:m].double() - tight.double()).norm(dim=1) / (tight.double() - x[:m].double()).norm(dim=1)
    print(f"{shape.name} N {N} rows {m} of {m_upper}: row difference median {float(e.median()):.2e} largest {float(e.max()):.2e}", flush=True)
    assert float(e.max()) < 0.03


# one sequence, up to 512 rows and slots: the thin attention kernel, unsplit and (2048 slots) with the keys split
THIN = wl.Shape("loose-thin", 1, 512, 4, 128, 1024, 1056, "bf16")


@pytest.mark.parametrize("N,m,m_upper", [(300, 0, 300), (300, 1, 300), (300, 33, 300), (300, 32, 64), (512, 200, 512), (2048, 40, 256)])
def test_thin_attention(N, m, m_upper):
    check_bound(THIN, N, m, m_upper)


# gate|up by 2 x 2 waves in four row tiles (230 column slices a round), and in two
WIDE = wl.Shape("loose-wide", 1, 256, 2, 128, 11008, 1056, "bf16")


@pytest.mark.parametrize("m,m_upper", [(0, 1024), (16, 1024), (256, 1024), (257, 1000), (600, 1024), (769, 1024), (0, 500), (40, 500),
                                       (250, 500), (260, 500), (499, 500)])
def test_two_by_two_waves(m, m_upper):
    check_bound(WIDE, 1024, m, m_upper)


# every projection of at most 512 rows by the few-row kernels, with two and more trips of their rings: 16-row blocks past the
# count are read from the first block's place, and no row at all ends the launch after its first loads
FEW = wl.Shape("loose-few", 1, 2560, 32, 128, 10240, 1056, "bf16")


@pytest.mark.parametrize("m,m_upper", [(0, 16), (0, 80), (1, 80), (16, 80), (17, 80), (63, 80), (0, 128), (1, 128), (33, 112), (0, 200),
                                       (16, 160), (40, 192), (112, 224), (0, 256), (1, 256), (130, 256), (255, 256), (100, 320), (1, 384),
                                       (193, 384)])
def test_few_row_projections(m, m_upper):
    check_bound(FEW, 400, m, m_upper)
