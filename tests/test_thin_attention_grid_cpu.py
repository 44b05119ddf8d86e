"""The thin attention kernel's launches (no GPU; not part of the C ABI, called by their C++ names): however the rows within a bound lie
in the sequences, the grid has a workgroup for every query tile; and 32 queries are taken per workgroup wherever the tiles that hold
rows make one round of 256 workgroups, whatever the bound says."""
import ctypes as C
import random

import pytest

from paper_2602_06412_amd import binding as B


def form(m_upper, batch, heads, n_pad):
    """(key splits, 0: another kernel; workgroups per head; whether they may take 64 queries)"""
    out = (C.c_int * 3)()
    B.lib()._Z23slk_attention_thin_formiiiiPi(m_upper, batch, heads, n_pad, out)
    return tuple(out)


def queries(rows, heads, grid):
    """(tiles, queries per tile) of a launch that may take 64"""
    t32, t64 = (sum(-(-r // q) for r in rows) for q in (32, 64))
    pairs = B.lib()._Z24slk_attention_thin_pairsiiii(t32, t64, heads, grid)
    return (t64, 64) if pairs else (t32, 32)


def _rows(rng, batch, N, most):
    """row counts of the sequences, `most` in all at most: even, ragged, or nearly all in one sequence"""
    kind, left, rows = rng.randrange(4), most, []
    for b in range(batch):
        want = [most // batch, rng.randint(0, N), rng.randint(0, 70), N if b == batch // 2 else 1][kind]
        rows.append(min(want, N, left))
        left -= rows[-1]
    return rows


@pytest.mark.parametrize("heads", [1, 4, 9, 20, 32, 40, 64, 300])
def test_every_row_has_a_workgroup(heads):
    rng, launches, wide = random.Random(heads), 0, 0
    for _ in range(4000):
        batch, N = rng.choice([1, 1, 2, 3, 4, 8, 12, 16, 70, 255]), rng.choice([40, 64, 300, 512, 1000, 1024, 1100, 2048])
        m_upper = rng.randint(1, min(batch * N, rng.choice([64, 600, 4000, 16000])))
        splits, grid, may = form(m_upper, batch, heads, -(-N // 64) * 64)
        if splits != 1 or not may:
            continue
        rows = _rows(rng, batch, N, rng.choice([m_upper, m_upper, rng.randint(0, m_upper)]))
        tiles, width = queries(rows, heads, grid)
        assert tiles <= grid, (m_upper, batch, N, rows, tiles, width, grid)
        t32 = sum(-(-r // 32) for r in rows)
        assert width == 32 or t32 * heads > 256, (m_upper, batch, N, rows)
        launches, wide = launches + 1, wide + (width == 64)
    assert launches > 20 and (wide > 5) == (heads < 256), (launches, wide)      # (300 heads: one tile by the bound)


def test_known_launches():
    """32 heads: 457 rows of one sequence are one round of 64 queries; eight sequences of 20 rows, or 16 rows under a bound of 512,
    one of 32, in the same launch as their bounds' worst case."""
    for m_upper, batch, rows, width in [(457, 1, [457], 64), (512, 1, [257], 64), (512, 1, [256], 32), (512, 1, [16], 32),
                                        (160, 8, [20] * 8, 32), (256, 2, [96, 160], 32), (200, 4, [50] * 4, 32), (288, 8, [36] * 8, 64),
                                        (300, 4, [75] * 4, 64), (120, 12, [10] * 12, 32)]:
        splits, grid, may = form(m_upper, batch, 32, 1024)
        assert (splits, may) == (1, 1) and queries(rows, 32, grid) == (sum(-(-r // width) for r in rows), width)
    assert form(256, 1, 32, 1024) == (1, 8, 0) and form(513, 1, 32, 1024)[0] == 0
