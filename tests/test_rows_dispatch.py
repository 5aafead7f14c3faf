"""The many-row path's choices of a kernel by sizes, as the launchers make them (host functions of the library, no GPU)."""
import ctypes as C

import pytest

import paper_2510_25739_amd as H
from paper_2510_25739_amd import build


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
