"""The ring kernel's row tiles touch shared weight lines ahead of their loads, by a rule on tile height and row tiles: sums
against fp64 where chunks, column blocks and sharers do not come out even, and no dependence on the row tiles that are there."""
import numpy as np
import pytest
import torch

from paper_2602_06412_amd import binding as B
from tests.gpu_util import DEV
from tests.test_gpu_linear import _bound, _inputs

pytestmark = pytest.mark.gpu


def _touches(m_upper, n, k):
    """The rule, restated."""
    kernel, splits, height, cols, _ = B.sl_linear_plan(m_upper, n, k)
    tiles = -(-m_upper // height)
    columns = -(-n // cols)
    one_round = 8 * tiles * -(-columns // 8) * splits <= 256
    short = height == 128 and splits > 1 and k // splits <= 1024 and tiles * columns * splits >= 192
    if height == 160:
        return kernel == 1 and one_round and tiles >= 6 and k // splits >= 2048
    return kernel == 1 and one_round and not short and height < 160 and (tiles >= 6 or (height == 128 and tiles == 4))


@pytest.mark.parametrize("n,k,m_upper,ms", [
    (12288, 4096, 512, [512, 130, 1]),          # 128 x 4; with few rows one sharer is left, or none but the tile itself
    (4096, 4096, 1024, [1023, 257]),            # 128 x 8, two splits; three sharers, the fewest that touch
    (4096, 8192, 1280, [1279, 500]),            # 160 x 8, two splits: the tallest tiles that touch
    (8192 - 160, 384, 600, [600, 255]),         # a ragged last column tile
    (8192 - 32, 256, 640, [640]),               # the shortest ring, one chunk to touch
    (1024, 512, 2048, [2040]),                  # more row tiles than column blocks
])
def test_sums(n, k, m_upper, ms):
    assert _touches(m_upper, n, k), B.sl_linear_plan(m_upper, n, k)
    w, x = _inputs(n + k, n, k, m_upper)
    wd = w.to(DEV)
    packed = torch.empty_like(wd)
    B.sl_linear_pack(wd, packed)
    xin = B.tile_activations(x.to(DEV))
    S = B.sl_linear_splits(m_upper, n, k)
    x64, w64 = x.double().numpy(), w.double().numpy()
    first = None
    for m in ms:
        y = torch.full((S, m_upper, n), float("nan"), device=DEV)
        B.sl_linear_forward(xin, packed, torch.tensor([m], dtype=torch.int32, device=DEV), m_upper, n, k, S, y_f32=y, x_tiled=1)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(y[:, :m]).all()) and bool(torch.isnan(y[:, m:]).all())
        assert np.all(np.abs(y[:, :m].double().sum(0).cpu().numpy() - x64[:m] @ w64.T) <= _bound(x64[:m], w64, k))
        first = y if first is None else first
        assert torch.equal(y[:, :m], first[:, :m])
