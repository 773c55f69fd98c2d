"""The tile queue of the backward launch (BwdQueue in csrc/attn_bwd_asm.h), through a host-only entry of the debug build:
whatever the tile counts, workgroups and compute units, every tile of either sweep is taken up exactly once, a
workgroup's entries rise from pass to pass (it never returns to the first sweep), and every entry stays on its XCD."""
import ctypes
import random

import debug_lib


def test_every_tile_once():
    lib = ctypes.CDLL(debug_lib.PATH)
    entry = lib.attn_bwd_queue_entry
    entry.restype, entry.argtypes = ctypes.c_int, [ctypes.c_int] * 6 + [ctypes.POINTER(ctypes.c_int)]
    rng = random.Random(5)
    sizes = [(0, 1), (0, 600), (1, 1), (8, 8), (7, 9), (128, 128), (255, 257), (256, 256), (1, 600), (600, 1)]
    sizes += [(rng.randint(1, 900), rng.randint(1, 900)) for _ in range(60)]
    first_q = ctypes.c_int()
    for n_kv, n_q in sizes:
        slots, cus = rng.choice([(256, 32), (512, 32), (512, 31), (64, 32), (8, 1)])
        seen = []
        entry(n_kv, n_q, 0, slots, cus, 0, first_q)
        total = first_q.value + n_q
        assert first_q.value % 8 == 0 and n_kv <= first_q.value < n_kv + 8
        for wg in range(min(slots, total)):
            last, k = -1, 0
            while True:
                e = entry(n_kv, n_q, wg, slots, cus, k, first_q)
                if e < 0:
                    break
                assert e > last and e % 8 == wg % 8
                last, k = e, k + 1
                seen.append(e)
        assert sorted(seen) == list(range(total)), (n_kv, n_q, slots, cus)


def test_launches_of_one_sweep():
    """Key owners alone: nothing follows them.  Query owners alone: their entries start at 0."""
    lib = ctypes.CDLL(debug_lib.PATH)
    entry = lib.attn_bwd_queue_entry
    entry.restype, entry.argtypes = ctypes.c_int, [ctypes.c_int] * 6 + [ctypes.POINTER(ctypes.c_int)]
    first_q = ctypes.c_int()
    for n_kv in (1, 5, 300, 2053):
        seen = [entry(n_kv, 0, wg, 256, 32, k, first_q) for wg in range(min(n_kv, 256)) for k in range(n_kv // 256 + 2)]
        assert sorted(e for e in seen if e >= 0) == list(range(n_kv))
    entry(0, 7, 0, 256, 32, 0, first_q)
    assert first_q.value == 0


def test_sweeps_run_apart_where_long_query_tiles_would_share_workgroups():
    lib = ctypes.CDLL(debug_lib.PATH)
    apart = lib.attn_bwd_sweeps_apart
    apart.restype, apart.argtypes = ctypes.c_int, [ctypes.c_int] * 5
    for heads, s_q, s_kv, causal, slots, want in [
            (123, 72, 5938, 0, 256, 1), (123, 72, 1500, 0, 256, 1), (123, 72, 1500, 0, 512, 1), (16, 1000, 8000, 0, 256, 1),
            (16, 1000, 8000, 1, 512, 1), (56, 100, 1100, 0, 256, 1), (56, 100, 1100, 0, 512, 1),
            (48, 72, 1500, 0, 256, 0), (123, 64, 512, 1, 256, 0), (400, 72, 5938, 0, 256, 0), (16, 2000, 3000, 1, 512, 0), (48, 1000, 8000, 1, 512, 0),
            (16, 4096, 4096, 0, 256, 0), (8, 72, 5938, 0, 0x7fffffff, 0)]:
        assert apart(heads, s_q, s_kv, causal, slots) == want, (heads, s_q, s_kv, causal, slots)
