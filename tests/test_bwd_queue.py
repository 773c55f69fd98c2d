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
    sizes = [(1, 1), (8, 8), (7, 9), (128, 128), (255, 257), (256, 256), (1, 600), (600, 1)]
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
