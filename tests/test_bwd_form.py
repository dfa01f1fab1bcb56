"""The backward's choice of launch form, without a GPU: the measured sizes the rule is stated with, the edges of the
argument checks, and what a wrong chain length would turn over (a chain of zero steps sends every call to separate
launches)."""
import ctypes

import pytest

from paper_2506_01380_amd import binding as nb

S, M, MS, TILES, ROWS = nb.NFD_BWD_SEPARATE, nb.NFD_BWD_MERGED, nb.NFD_BWD_MERGED_SMALL, nb.NFD_BWD_TILES, nb.NFD_BWD_ROWS


@pytest.mark.parametrize("heads,T,frames,form", [
    (12, 336, 16, M), (24, 336, 16, M), (48, 336, 16, M), (64, 336, 16, S),  # us: 280/175/188, 340/302/341, 590/574/705, 763/777/943
    (12, 247, 11, MS),      # 156 / 85 / 66
    (192, 40, 20, MS),      # 116 / 100 / 94
    (32, 576, 64, S),       # 16180 / 17040 / 22900
    (1, 1, 1, MS),
])
def test_matrix_core_form(heads, T, frames, form):
    assert nb.nfd_attn_bwd_form(nb.NFD_BF16, 1, heads, frames, T, 64, frames, frames) == form
    assert nb.nfd_attn_bwd_form(nb.NFD_BF16, 1, heads, frames + 3, T, 64, frames, frames, num_cus=256) == form


@pytest.mark.parametrize("dtype,heads,T,D,kv,q,form", [
    (nb.NFD_FP32, 12, 336, 64, 4, 4, TILES),
    (nb.NFD_FP32, 4096, 1, 64, 1, 1, ROWS),
    (nb.NFD_FP32, 4096, 16, 64, 1, 1, TILES),
    (nb.NFD_BF16, 24, 16, 62, 1, 1, ROWS),
    (nb.NFD_BF16, 24, 336, 62, 2, 2, TILES),
])
def test_general_form(dtype, heads, T, D, kv, q, form):
    assert nb.nfd_attn_bwd_form(dtype, 1, heads, kv, T, D, kv, q) == form


def test_errors():
    L, f = nb.lib(), ctypes.c_int(-7)
    assert L.nfd_attn_bwd_form(nb.NFD_BF16, 1, 1, 1, 1, 64, 1, 1, 0, None) == nb.NFD_ERR_NULL
    assert L.nfd_attn_bwd_form(nb.NFD_BF16, 1, 1, 1, 0, 64, 1, 1, 0, ctypes.byref(f)) == nb.NFD_ERR_SHAPE
    assert L.nfd_attn_bwd_form(nb.NFD_BF16, 1, 1, 1, 1, 64, 2, 1, 0, ctypes.byref(f)) == nb.NFD_ERR_CAPACITY
    assert L.nfd_attn_bwd_form(nb.NFD_BF16, 1, 1, 1, 1, 257, 1, 1, 0, ctypes.byref(f)) == nb.NFD_ERR_UNSUPPORTED
    assert f.value == -7
