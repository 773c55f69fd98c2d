"""The plan of a backward launch's walks (plan_walks in csrc/attn_bwd.hip), through a host-only entry of the debug build: every entry
of an XCD's queue belongs to exactly one workgroup, a workgroup's entries rise (it never returns to the first sweep), and the
longest walk is not longer than the most loaded workgroup of any order could do without."""
import ctypes
import random

import debug_lib


def plan(heads, s_q, s_kv, d, causal, tiling, cus=256):
    call = ctypes.CDLL(debug_lib.PATH).attn_bwd_plan
    call.restype, call.argtypes = ctypes.c_float, [ctypes.c_int] * 7 + [ctypes.POINTER(ctypes.c_uint32)] * 2
    first, idx = (ctypes.c_uint32 * 64)(), (ctypes.c_uint32 * 512)()
    ratio = call(heads, s_q, s_kv, d, causal, tiling, cus, first, idx)
    half = lambda words, i: words[i // 2] >> i % 2 * 16 & 0xffff
    return ratio, lambda i: half(first, i), lambda i: half(idx, i)


def test_every_entry_once_and_in_rising_order():
    rng = random.Random(11)
    shapes = [(40, 1500, 1500, 128, 1, 2), (123, 72, 5938, 128, 0, 1), (12, 6000, 6000, 128, 1, 3), (9, 5000, 5000, 128, 1, 2),
              (16, 1000, 8000, 64, 0, 1), (50, 3000, 3000, 64, 1, 1)]
    for _ in range(300):
        shapes.append((rng.randint(1, 200), rng.randint(1, 6000), rng.randint(1, 6000), rng.choice([64, 128]), rng.randint(0, 1),
                       rng.randint(1, 3)))
    planned = 0
    for heads, s_q, s_kv, d, causal, tiling in shapes:
        rows = 256 if d == 128 and tiling == 2 else 128
        slots = 64 if d == 64 or tiling == 3 else 32
        n_kv, n_q = heads * -(-s_kv // rows), heads * -(-s_q // rows)
        n = -(-(-(-n_kv // 8) * 8 + n_q) // 8)      # XCD 0's entries
        ratio, first, idx = plan(heads, s_q, s_kv, d, causal, tiling)
        if n <= slots or n > 768:
            assert ratio == 1 or n > slots       # (a single pass, or too many: no plan)
            continue
        planned += 1
        assert 0 < ratio <= 1.5
        seen = []
        for m in range(slots):
            mine = [idx(i) for i in range(first(m), first(m + 1))]
            assert mine == sorted(mine), (heads, s_q, s_kv, d, causal, tiling, m)
            seen += mine
        assert sorted(seen) == list(range(n)), (heads, s_q, s_kv, d, causal, tiling)
    assert planned > 100
    # where the passes fall badly the plan is far ahead, and it is never taken where it is not
    assert plan(123, 72, 5938, 128, 0, 1)[0] < 0.8 and plan(16, 1000, 8000, 128, 1, 2)[0] < 0.7
    assert plan(128, 4096, 4096, 128, 0, 2)[0] == 1.0
