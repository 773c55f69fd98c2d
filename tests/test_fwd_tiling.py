"""Which tiling the dispatcher takes for a D = 64 or 128 launch of at least 64 queries (host-only entry of the debug build; 256
compute units where there is no GPU): the one that was measured to be the fastest, on both sides of the lines."""
import ctypes

import pytest

import debug_lib

# D = 128: causal, heads, queries, keys, tiling (1: 256 rows, 3: 128 rows in 64-row waves, 4: in pairs of 32-row waves).  Up to
# one 128-row tile per compute unit the waves work in pairs
MEASURED = [(1, h, s, s, 4) for h, s in ((1, 200), (64, 200), (16, 256), (64, 256), (1, 300), (16, 500), (64, 512), (1, 777),
                                         (16, 777), (32, 900), (16, 1024), (32, 1024), (12, 1500), (2, 2048), (16, 2048),
                                         (6, 2500), (1, 3000), (8, 3000), (1, 6000), (4, 6000), (1, 8192), (4, 8192),
                                         (1, 16384), (2, 16384), (16, 128), (256, 128))]
MEASURED += [(0, h, s, s, 4) for h, s in ((16, 2048), (8, 4096), (3, 7744))]
# ... and beyond
MEASURED += [(1, h, s, s, 4) for h, s in ((128, 520), (100, 777), (400, 300), (157, 400), (583, 64))]
MEASURED += [(1, h, s, s, 3) for h, s in ((202, 1871), (244, 1088), (241, 1400), (353, 1113))]
MEASURED += [(1, h, s, s, 1) for h, s in ((32, 4096), (96, 1195), (60, 2496), (35, 3299), (48, 2112), (72, 3776))]
MEASURED += [(1, 116, 13065, 333, 1), (1, 48, 13184, 1511, 1), (1, 152, 1640, 2304, 3), (1, 160, 448, 1757, 4)]
MEASURED += [(0, 512, 300, 300, 4), (0, 258, 320, 230, 4), (0, 24, 3072, 3072, 4), (0, 596, 64, 155, 4), (0, 112, 1618, 115, 4),
             (0, 96, 640, 2578, 3), (0, 160, 320, 7680, 3), (0, 12, 10821, 7414, 3),
             (0, 32, 4096, 4096, 1), (0, 96, 300, 300, 1), (0, 304, 704, 704, 1), (0, 96, 320, 4494, 1), (0, 6, 7055, 7055, 1)]

# D = 64: causal, heads, rows, tiling (0: 256 rows, 1: 128)
MEASURED_64 = [(1, h, s, 1) for h, s in ((1, 64), (400, 300), (256, 567), (600, 300), (96, 1579), (128, 1100), (64, 2549),
                                         (96, 1920), (256, 1605), (48, 2806), (48, 4096))]
MEASURED_64 += [(0, h, s, 0) for h, s in ((96, 320), (128, 320), (64, 520), (96, 384), (256, 138), (64, 777), (32, 2048))]
MEASURED_64 += [(0, h, s, 1) for h, s in ((1, 8192), (16, 2048), (64, 384), (32, 1024), (96, 520), (600, 100))]


def check(D, causal, heads, s_q, s_kv, want):
    choice = ctypes.CDLL(debug_lib.PATH).attn_fwd_tiling
    choice.restype, choice.argtypes = ctypes.c_int, [ctypes.c_int] * 5
    assert choice(D, heads, s_q, s_kv, causal) == want


@pytest.mark.parametrize("causal,heads,s_q,s_kv,want", MEASURED)
def test_the_fastest_tiling_is_taken(causal, heads, s_q, s_kv, want):
    check(128, causal, heads, s_q, s_kv, want)


@pytest.mark.parametrize("causal,heads,rows,want", MEASURED_64)
def test_the_faster_tiling_is_taken_at_d64(causal, heads, rows, want):
    check(64, causal, heads, rows, rows, want)
