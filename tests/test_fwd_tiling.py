"""Which of the two query tilings of D = 64 and 128 the dispatcher takes (host-only entry of the debug build; 256 compute units where
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


MEASURED_64 = [(1, h, s, 128) for h, s in ((1, 64), (400, 300), (256, 567), (600, 300), (96, 1579), (128, 1100), (64, 2549),
                                           (96, 1920), (256, 1605), (48, 2806), (48, 4096))]
MEASURED_64 += [(0, h, s, 256) for h, s in ((96, 320), (128, 320), (64, 520), (96, 384), (256, 138), (64, 777), (32, 2048))]
MEASURED_64 += [(0, h, s, 128) for h, s in ((1, 8192), (16, 2048), (64, 384), (32, 1024), (96, 520), (600, 100))]


def check(D, causal, heads, rows, want):
    choice = ctypes.CDLL(debug_lib.PATH).attn_fwd_tile_rows
    choice.restype, choice.argtypes = ctypes.c_int, [ctypes.c_int] * 5
    assert choice(D, heads, rows, rows, causal) == want


@pytest.mark.parametrize("causal,heads,rows,want", MEASURED)
def test_the_faster_tiling_is_taken(causal, heads, rows, want):
    check(128, causal, heads, rows, want)


@pytest.mark.parametrize("causal,heads,rows,want", MEASURED_64)
def test_the_faster_tiling_is_taken_at_d64(causal, heads, rows, want):
    check(64, causal, heads, rows, want)
