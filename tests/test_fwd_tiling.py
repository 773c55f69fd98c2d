"""Which of the two D = 128 query tilings the dispatcher takes (host-only entry of the debug build; 256 compute units where
there is no GPU): the one that was the faster of the two, over launches with at most one 128-row tile per compute unit, and
on both sides of the lines for fuller ones."""
import ctypes

import pytest

import debug_lib

# causal, heads, rows, tile rows
MEASURED = [(1, h, s, 128) for h, s in ((1, 200), (64, 200), (16, 256), (64, 256), (1, 300), (16, 500), (64, 512), (1, 777),
                                        (16, 777), (32, 900), (16, 1024), (32, 1024), (12, 1500), (2, 2048), (16, 2048),
                                        (6, 2500), (1, 3000), (8, 3000))]
MEASURED += [(1, h, s, 256) for h, s in ((1, 6000), (4, 6000), (1, 8192), (4, 8192), (1, 16384), (2, 16384), (32, 4096))]
MEASURED += [(1, 128, 520, 128), (1, 100, 777, 128), (1, 128, 1100, 128), (0, 100, 600, 128), (0, 512, 300, 128),
             (0, 32, 4096, 256), (1, 16, 128, 256), (1, 256, 128, 256), (0, 16, 2048, 256), (0, 8, 4096, 256), (0, 3, 7744, 256),
             (0, 96, 300, 256), (1, 400, 300, 128)]


@pytest.mark.parametrize("causal,heads,rows,want", MEASURED)
def test_the_faster_tiling_is_taken(causal, heads, rows, want):
    choice = ctypes.CDLL(debug_lib.PATH).attn_fwd_d128_tile_rows
    choice.restype, choice.argtypes = ctypes.c_int, [ctypes.c_int] * 4
    assert choice(heads, rows, rows, causal) == want
