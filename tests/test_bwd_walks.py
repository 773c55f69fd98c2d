"""The walks behind a backward launch's plan (BwdWalks, plan_walks in csrc/attn_bwd.hip), through host-only entries of the debug build: every
entry of an XCD's queue belongs to exactly one workgroup, a workgroup's entries rise (it never returns to the first sweep), the longest
walk is what the entries add up to and within the bound of list scheduling, and no plan beats the bound that refuses plans unmade
(without a mask: every plan meets it)."""
import ctypes
import random

import debug_lib

MAX_ENTRIES = 768   # of an XCD (BwdPlan)


def plan(heads, s_q, s_kv, d, causal, tiling, cus=256):
    """(walk by plan over walk by passes, or 1; first(m), idx(i), (by plan, by passes, least), XCD 0's entries in us)"""
    call = ctypes.CDLL(debug_lib.PATH).attn_bwd_plan_walks
    call.restype = ctypes.c_float
    call.argtypes = [ctypes.c_int] * 7 + [ctypes.POINTER(ctypes.c_uint32)] * 2 + [ctypes.POINTER(ctypes.c_float)]
    first, idx, walks = (ctypes.c_uint32 * 64)(), (ctypes.c_uint32 * 512)(), (ctypes.c_float * (3 + MAX_ENTRIES))()
    ratio = call(heads, s_q, s_kv, d, causal, tiling, cus, first, idx, walks)
    half = lambda words, i: words[i // 2] >> i % 2 * 16 & 0xffff
    return ratio, lambda i: half(first, i), lambda i: half(idx, i), walks[:3], walks[3:]


def sizes(heads, s_q, s_kv, d, tiling):
    """rows of a tile, workgroups of an XCD, entries of XCD 0"""
    rows, slots = 256 if d == 128 and tiling == 2 else 128, 64 if d == 64 or tiling == 3 else 32
    n_kv, n_q = heads * -(-s_kv // rows), heads * -(-s_q // rows)
    return rows, slots, -(-n_kv // 8) + -(-n_q // 8)


def test_loads_limits_and_the_bound_of_a_plan():
    rng = random.Random(11)
    shapes = [(40, 1500, 1500, 128, 1, 2), (123, 72, 5938, 128, 0, 1), (12, 6000, 6000, 128, 1, 3), (9, 5000, 5000, 128, 1, 2),
              (16, 1000, 8000, 64, 0, 1), (50, 3000, 3000, 64, 1, 1), (512, 768, 768, 64, 0, 1), (513, 768, 768, 64, 0, 1),
              (512, 768, 768, 128, 1, 1), (513, 768, 768, 128, 1, 1), (64, 512, 512, 64, 0, 1), (65, 512, 512, 64, 0, 1)]
    for _ in range(300):
        shapes.append((rng.randint(1, 200), rng.randint(1, 6000), rng.randint(1, 6000), rng.choice([64, 128]), rng.randint(0, 1),
                       rng.randint(1, 3)))
    planned, single, many = 0, 0, 0
    for shape in shapes:
        heads, s_q, s_kv, d, causal, tiling = shape
        rows, slots, n = sizes(heads, s_q, s_kv, d, tiling)
        entries = -(-heads * -(-s_kv // rows) // 8) * 8 + heads * -(-s_q // rows)
        ratio, first, idx, (by_plan, by_passes, least), cost = plan(*shape)
        if entries <= 8 * slots or entries > 8 * MAX_ENTRIES:      # a single pass, or too many: no plan
            assert ratio == 1
            single, many = single + (n <= slots), many + (n > MAX_ENTRIES)
            continue
        planned += 1
        seen, loads = [], []
        for m in range(slots):
            mine = [idx(i) for i in range(first(m), first(m + 1))]
            assert mine == sorted(mine), (shape, m)
            seen += mine
            loads.append(sum(cost[i] for i in mine))
        assert sorted(seen) == list(range(n)), shape
        cost = cost[:n]
        assert min(cost) > 0 and abs(ratio - by_plan / by_passes) < 1e-5
        passes = [0.0] * slots
        for i, l in enumerate(cost):
            k, m = divmod(i, slots)
            passes[slots - 1 - m if k % 2 else m] += l
        close = lambda x: 1e-4 * x + 1e-3
        if causal and heads % 8:       # (the other XCDs' walks count as well)
            assert max(loads) <= by_plan + close(by_plan) and max(passes) <= by_passes + close(by_passes)
        else:
            assert abs(max(loads) - by_plan) < close(by_plan) and abs(max(passes) - by_passes) < close(by_passes)
            assert by_plan <= sum(cost) / slots + max(cost) + close(by_plan)       # (list scheduling)
        assert least <= by_plan + close(by_plan) and (causal or least >= by_plan - close(by_plan)), shape
    assert planned > 100 and single > 10 and many > 10
    # where the passes fall badly the plan is far ahead, and it is never taken where it is not
    assert plan(123, 72, 5938, 128, 0, 1)[0] < 0.8 and plan(16, 1000, 8000, 128, 1, 2)[0] < 0.7
    assert plan(128, 4096, 4096, 128, 0, 2)[0] == 1.0


def test_hopeless_plans_are_refused_before_they_are_made():
    """No order of these launches' entries is 5 % (D = 64: 7 %) shorter than the passes, which the bound alone says."""
    for shape in [(451, 576, 576, 128, 0, 3), (128, 4096, 4096, 128, 0, 2), (65, 484, 484, 128, 0, 2), (140, 194, 194, 128, 0, 2),
                  (159, 1185, 1185, 128, 0, 2), (213, 1352, 1352, 128, 0, 3), (199, 338, 338, 64, 0, 1)]:
        _, _, _, (by_plan, by_passes, least), _ = plan(*shape)
        assert least >= (0.93 if shape[3] == 64 else 0.95) * by_passes, (shape, by_plan, by_passes, least)


def test_the_tiling_is_chosen_by_the_walk_that_it_gets():
    """A D = 128 launch's estimate rests on its plan's longest walk where the plan is taken, and on the passes' where it is not."""
    call = ctypes.CDLL(debug_lib.PATH).attn_bwd_picked_walk
    call.restype, call.argtypes = ctypes.c_int, [ctypes.c_int] * 5 + [ctypes.POINTER(ctypes.c_float)] * 2
    est, walk = (ctypes.c_float * 3)(), (ctypes.c_float * 2)()
    rng = random.Random(4)
    shapes = [(65, 484, 484, 0), (140, 194, 194, 0), (40, 1500, 1500, 1), (123, 72, 5938, 0), (159, 1185, 1185, 0)]
    for _ in range(400):
        s = rng.randint(64, 5000)
        shapes.append((rng.randint(8, 200), s, s if rng.random() < 0.6 else rng.randint(64, 5000), rng.randint(0, 1)))
    taken = {}
    for heads, s_q, s_kv, causal in shapes:
        t = call(heads, s_q, s_kv, causal, 256, est, walk)
        ratio, _, _, (by_plan, by_passes, _), _ = plan(heads, s_q, s_kv, 128, causal, t)
        planned = ratio < 0.95
        taken[t, planned] = taken.get((t, planned), 0) + 1
        if ratio == 1 and by_passes == 0:       # (a single pass, or too many entries)
            assert not walk[1]
            continue
        assert walk[1] == planned and abs(walk[0] - (by_plan if planned else by_passes)) < 1e-3 * by_passes, (heads, s_q, s_kv, causal, t)
    assert all(taken.get((t, planned), 0) >= 5 for t in (1, 2, 3) for planned in (False, True)), taken
