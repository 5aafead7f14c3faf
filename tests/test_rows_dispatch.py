"""The many-row path's choices of a kernel by sizes, as the launchers make them (host functions of the library, no GPU)."""
import ctypes as C

import pytest

import paper_2510_25739_amd as H
import synth
from paper_2510_25739_amd import build
from test_gpu_rows import KERNEL_SHAPES, SHAPES
from test_gpu_wide import N_COND, WIDE_SHAPES


@pytest.fixture(scope="module")
def lib():
    import os
    if not os.path.exists(H.lib_path()):
        build.build()
    return C.CDLL(H.lib_path())


@pytest.mark.parametrize("sequences,heads,rows,waves", [
    (3, 20, 6, 8), (12, 20, 16, 8), (12, 20, 17, 4),     # a second row tile: 480 workgroups
    (8, 16, 32, 4), (8, 16, 16, 8), (4, 20, 48, 8), (4, 20, 49, 4), (13, 20, 1, 4), (1, 20, 64, 8)])
def test_step_attention_counts_row_tiles(lib, sequences, heads, rows, waves):
    # a workgroup of eight waves fills a compute unit: they are for launches of fewer workgroups - (sequence, head, 16
    # rows) each - than the chip has units
    assert lib.hawk_rows_attn_waves(sequences, heads, rows) == waves


def products(d, mlp, rows):
    """(what follows the product, N, K) of a layer's four products over tile-major weights."""
    m = (mlp + 31) // 32 * 32
    return [("plain", 3 * d, d), ("residual", d, d), ("swiglu", 2 * m, d), ("residual", d, m)]


def test_every_kernel_a_model_takes_is_compared_with_float64(lib):
    # The shapes of the many-row passes that are compared with a float64 forward reach each product kernel with each epilogue that the
    # model widths take it with, prompt rows of a full batch included.  Costs that change move the choices: then this fails.
    took = lambda d, mlp, rows: {(lib.hawk_rows_kernel(rows, n, k), what) for what, n, k in products(d, mlp, rows)}
    compared = set()
    for d, heads, mlp, batch, scale, n_cond, chunk in SHAPES + KERNEL_SHAPES:
        sequences = batch * (2 if scale != 1.0 else 1)
        compared |= took(d, mlp, sequences * n_cond) | took(d, mlp, sequences * chunk)
    for d, _, mlp, batch in WIDE_SHAPES:
        compared |= took(d, mlp, batch * N_COND)
    models = {}
    for i in (1, 2, 4):
        s = synth.CONFIGS[i]
        for rows in range(1, 4100):
            for kernel in took(s.d_model, s.d_mlp, rows):
                models.setdefault(kernel, []).append((s.d_model, rows))
    left = {k: v[0] for k, v in models.items() if k not in compared}
    assert not left, left
    assert len({k for k, _ in models}) == 19      # no entry of the table without a use
