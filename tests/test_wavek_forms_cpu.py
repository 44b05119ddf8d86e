"""Which form a layer's projection of few rows is launched in (no GPU; not part of the C ABI, called by its C++ name): every form
covers its rows, is one that is compiled, and, at the LLaDA-8B shapes, is one that tests/test_gpu_few_row_projections.py launches
with several trips of its operand rings (each form is a kernel of its own, with its own hand-counted waits)."""
import ctypes as C

import pytest

from paper_2602_06412_amd import binding as B

QKV, GATE_UP, PLANES = 0, 1, 2
D, H, DFF = 4096, 32, 12288
LLADA = {"q|k|v": (QKV, H, D), "gate|up": (GATE_UP, DFF, D), "out": (PLANES, D, H * 128), "down": (PLANES, D, DFF)}
COMPILED = {(QKV, 1, 4): range(1, 6), (QKV, 1, 6): [4, 5, 6, 7, 8, 10, 12], (GATE_UP, 1, 6): [1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16],
            (PLANES, 1, 4): [1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16], (GATE_UP, 2, 6): [10, 12, 14, 16], (PLANES, 2, 4): [10, 12, 14, 16]}


def form(projection, m_upper, width, k):
    """(kernel: 0 another file's, 1 waves along k, 2 2 x 2 waves; 16-row blocks and 16-column blocks per workgroup; row tiles)"""
    out = (C.c_int * 4)()
    B.lib()._Z14slk_wavek_formiiiiPi(projection, m_upper, width, k, out)
    return tuple(out)


@pytest.mark.parametrize("shape", [LLADA, {"q|k|v": (QKV, 27, 512), "gate|up": (GATE_UP, 7808, 512), "out": (PLANES, 2688, 2048)}],
                         ids=["llada", "narrow"])
def test_forms_cover_their_rows_and_are_compiled(shape):
    seen = {}
    for projection, width, k in shape.values():
        for mu in range(1, 1100):
            kernel, blocks, cols, tiles = form(projection, mu, width, k)
            if kernel == 0:
                continue
            assert blocks * 16 * tiles >= mu and blocks * 16 * (tiles - 1) < mu
            seen.setdefault((projection, kernel, cols), set()).add(blocks)
            assert blocks in COMPILED[projection, kernel, cols], (projection, mu, kernel, blocks, cols)
    if shape is LLADA:                                # and nothing is compiled that no row count takes
        assert {f: sorted(b) for f, b in seen.items()} == {f: sorted(b) for f, b in COMPILED.items()}


def test_limits():
    for projection, width, k in LLADA.values():
        assert form(projection, 1, width, k)[0] == 1 and form(projection, 1025, width, k)[0] == 0
        assert form(projection, 0, width, k)[0] == 0
    assert form(QKV, 384, H, D)[0] == 1 and form(QKV, 385, H, D)[0] == 0
    assert [form(GATE_UP, mu, DFF, D)[0] for mu in (256, 257, 512, 513, 960, 961, 1024)] == [1, 2, 2, 0, 0, 2, 2]
    assert [form(PLANES, mu, D, DFF)[0] for mu in (256, 257, 512, 513)] == [1, 2, 2, 0]


def test_every_reachable_form_runs_its_steady_loop_in_the_gpu_tests():
    from tests.test_gpu_few_row_projections import LONG, LONG_ROWS
    d, hd, dff = LONG.d_model, LONG.n_heads * 128, LONG.d_ff
    tested = {}
    for name, (projection, width, k) in {"q|k|v": (QKV, LONG.n_heads, d), "gate|up": (GATE_UP, dff, d), "out": (PLANES, d, hd),
                                         "down": (PLANES, d, dff)}.items():
        for mu in LONG_ROWS:
            kernel, blocks, cols, _ = form(projection, mu, width, k)
            if kernel:
                step, depth = (128, 4 if blocks <= 8 else 2) if kernel == 1 else (64, 3)
                trips = k // (4 if projection == PLANES else 1) // step / depth
                key = (projection, kernel, blocks, cols)
                tested[key] = max(trips, tested.get(key, 0))
    for name, (projection, width, k) in LLADA.items():
        for mu in range(1, 1100):
            kernel, blocks, cols, _ = form(projection, mu, width, k)
            assert kernel == 0 or tested.get((projection, kernel, blocks, cols), 0) >= 3, (name, mu, kernel, blocks, cols)
