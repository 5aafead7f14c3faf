"""The contraction kernel with weights in registers (rows.hip: rows_gemm_wide_kernel): every tile with every epilogue, against
a float64 forward.  The shapes reach them by the library's own choice, which test_shapes_reach_every_tile asserts on the CPU."""
import ctypes as C
import os

import pytest

import paper_2510_25739_amd as H_
from paper_2510_25739_amd import build
from test_gpu_rows import BASE, hidden_pair, relative

TILES = (1608, 2012, 1612, 1812, 1616, 812)   # strips * 100 + row tiles of a workgroup
N_COND = 129
WIDE_SHAPES = [   # d_model, heads, d_mlp, prompts of 129 rows (most of them ragged against the tiles' rows)
    (256, 4, 2048, 9), (256, 4, 2048, 12), (256, 4, 704, 56), (256, 4, 352, 128), (256, 4, 96, 63), (256, 4, 2048, 26), (256, 4, 96, 102),
    (512, 8, 704, 56), (512, 8, 96, 128), (512, 8, 96, 96), (768, 12, 96, 127), (1280, 20, 96, 76)]


def test_shapes_reach_every_tile():
    if not os.path.exists(H_.lib_path()):
        build.build()
    lib = C.CDLL(H_.lib_path())
    reached = set()
    for d, _, mlp, batch in WIDE_SHAPES:
        rows, m = batch * N_COND, (mlp + 31) // 32 * 32
        reached |= {(lib.hawk_rows_tile(rows, n, k), what)
                    for what, n, k in (("plain", 3 * d, d), ("residual", d, d), ("swiglu", 2 * m, d), ("residual", d, m))}
    assert {(t, what) for t in TILES for what in ("plain", "residual", "swiglu")} <= reached


@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,mlp,batch", WIDE_SHAPES)
def test_every_tile_and_epilogue(d, heads, mlp, batch):
    # weights and bound as in test_gpu_rows.py: test_every_product_kernel_and_epilogue
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    s = BASE.replace(d_model=d, n_heads=heads, d_mlp=mlp, batch=batch, n_cond=N_COND, n_layers=1)
    got, ref = hidden_pair(H_, s, 1, std=0.8 / d ** 0.5)
    prompt, step = relative(got[:, :N_COND], ref[:, :N_COND]), relative(got[:, N_COND:], ref[:, N_COND:])
    print(f"rows {batch * N_COND}: relative error prompt {prompt:.2e}, step {step:.2e}")
    assert prompt < 1e-3 and step < 1e-3
