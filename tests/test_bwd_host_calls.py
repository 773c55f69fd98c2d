"""What a backward call asks of the HIP runtime and launches, on a stand-in for it (fake_hip.py)."""
import random

import fake_hip
from test_bwd_walks import plan, sizes

# heads, S_q, S_kv, D, causal, f16, tiling (0: as dispatched)
CALLS = [(16, 515, 515, 64, 0, 1, 0), (16, 1024, 1024, 128, 0, 0, 0), (128, 4096, 4096, 128, 0, 0, 0), (40, 1500, 1500, 128, 1, 0, 0),
         (123, 72, 5938, 64, 0, 0, 0), (12, 6000, 6000, 128, 1, 1, 2), (300, 300, 300, 128, 0, 0, 3)]


def test_a_kernel_may_use_its_lds_before_it_is_asked_about_or_launched(tmp_path):
    for call, (rc, lines) in zip(CALLS, fake_hip.backward_calls(tmp_path, CALLS)):
        assert rc == 0 and lines[-1]["what"] == "launch", call
        for line in lines:
            assert line["allowed"], (call, line)


def test_a_plan_holds_nothing_but_itself(tmp_path):
    """Its words behind the last entry are zero, whatever stood on the stack."""
    calls = [(123, 72, 5938, 64, 0, 0, 0), (40, 1500, 1500, 128, 1, 0, 0)] * 2 + [(16, 1000, 8000, 64, 1, 0, 0)]
    plans = [line["plan"] for _, lines in fake_hip.backward_calls(tmp_path, calls) for line in lines if "plan" in line]
    assert len(plans) >= 4
    for words in plans:
        first = [w >> s & 0xffff for w in words[:33] for s in (0, 16)]
        slots = first.index(max(first))
        entries = [w >> s & 0xffff for w in words[33:] for s in (0, 16)]
        assert sorted(entries[:first[slots]]) == list(range(first[slots])) and slots in (32, 64)
        assert not any(first[slots + 1:]) and not any(entries[first[slots]:])


def test_a_planned_launch_has_the_workgroups_that_its_kernel_fits(tmp_path):
    """A plan is made for so many workgroups; all of them have to run at once."""
    calls = [(123, 72, 5938, 64, 0, 0, 0), (40, 1500, 1500, 128, 1, 0, 0), (12, 6000, 6000, 128, 1, 1, 2), (40, 1500, 1500, 128, 1, 0, 1)]
    fits, planned = {}, 0
    for call, (rc, lines) in zip(calls, fake_hip.backward_calls(tmp_path, calls)):
        for line in lines:
            if line["what"] == "occupancy":
                fits[line["kernel"]] = line["fits"]
            elif "plan" in line:
                planned += 1
                assert line["grid"] == 256 * fits.get(line["kernel"], 0), (call, line["kernel"], line["grid"])
    assert planned == len(calls)


def test_which_launches_run_one_sweep_after_the_other(tmp_path):
    """Without a plan: few queries against many keys, but not causal launches in 64-row waves."""
    calls = [(257, 90, 3413, 128, 0, 0, 3), (104, 88, 8595, 128, 0, 1, 3), (6, 1443, 10145, 128, 1, 0, 3), (7, 1103, 7699, 128, 1, 0, 2),
             (24, 1223, 17813, 128, 1, 0, 2), (16, 1024, 1024, 128, 0, 0, 3)]
    for call, want, (rc, lines) in zip(calls, (2, 2, 1, 1, 1, 1), fake_hip.backward_calls(tmp_path, calls)):
        sweeps = [line for line in lines if line["what"] == "launch" and "delta" not in line["kernel"]]
        assert rc == 0 and len(sweeps) == want and not any("plan" in line for line in sweeps), (call, sweeps)


def test_plans_at_d64_are_judged_by_the_pairs_that_share_a_compute_unit(tmp_path):
    """D = 64, two workgroups to a compute unit: plans that level the single walks but pair the long ones took up to 1.12 times as long as the
    passes, which pair long with short."""
    without = [(242, 178, 860), (13, 2210, 3580), (88, 1946, 1946)]
    with_plan = [(123, 72, 5938), (153, 80, 3544), (72, 282, 6774), (242, 188, 1284), (93, 1476, 152)]
    shapes = [x + (64, 0, 0, 0) for x in without + with_plan]
    rng, n = random.Random(3), len(shapes)
    for _ in range(150):       # (heads in eights: the mask gives every XCD the same tiles)
        shapes.append((8 * rng.randint(1, 30), rng.randint(64, 4000), rng.randint(64, 4000), 64, rng.randint(0, 1), 0, 0))
    got = [any("plan" in line for line in lines) for _, lines in fake_hip.backward_calls(tmp_path, shapes)]
    assert got[:n] == [False] * len(without) + [True] * len(with_plan)
    seen = {}
    for (heads, s_q, s_kv, d, causal, _, _), planned in zip(shapes, got):
        ratio, first, idx, (by_plan, by_passes, _), cost = plan(heads, s_q, s_kv, d, causal, 1)
        if not by_passes:
            assert not planned
            continue
        cost = cost[:sizes(heads, s_q, s_kv, d, 1)[2]]
        loads, passes = [sum(cost[idx(i)] for i in range(first(m), first(m + 1))) for m in range(64)], [0.0] * 64
        for i, l in enumerate(cost):
            k, m = divmod(i, 64)
            m = 63 - m if k % 2 else m
            passes[31 - m if m < 32 else m] += l       # (BwdQueue::entry)
        pair = lambda w: max(min(x, y) + 0.6 * abs(x - y) for x, y in zip(w[:32], w[32:]))
        short = causal and min(s_q, s_kv) < 1024
        one, two = ratio / (0.8 if short else 0.93), pair(loads) / pair(passes)
        if min(abs(one - 1), abs(two - 1), abs(two / (0.92 if short else 0.96) - 1)) < 1e-4:
            continue       # (on the line)
        want = two < (0.92 if short else 0.96) or (one < 1 and two < 1)
        assert planned == want, (heads, s_q, s_kv, causal, one, two)
        seen[planned, one < 1] = seen.get((planned, one < 1), 0) + 1
    assert all(seen.get(k, 0) >= 2 for k in ((True, True), (True, False), (False, True), (False, False))), seen
