"""The forward tilings whose keys are shared out between two groups of waves (64 query rows, D = 64 and
128), each forced through the debug build on the sizes where it can go wrong: fewer keys than the two groups have
tiles, an odd number of tiles, ragged ends, causal blocks of which the second group's keys are all masked.  Against the
fp64 oracle, bars as in test_parity_gpu.py; and the same shapes through the dispatcher in both element types."""
import numpy as np
import pytest
import torch

import debug_lib
from oracle.attn_oracle import attn_ref
from paper_2512_18134_amd import binding, synth

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 33), (1, 2000), (31, 32), (33, 64), (64, 65), (65, 64), (96, 97), (100, 31), (128, 160), (129, 128),
         (192, 191), (257, 289), (300, 1000), (515, 70)]
TILINGS = [(128, debug_lib.FWD_KEY_GROUPS), (64, debug_lib.FWD_KEY_GROUPS), (64, debug_lib.FWD_D64_4_WAVES),
           (128, debug_lib.FWD_D128_2_WAVES)]


def on_gpu(bits, dt):
    return torch.from_numpy(bits.view(np.int16)).cuda().view(dt)


def f64(t):
    return t.float().cpu().numpy().astype(np.float64)


def check(o, lse, want, o_tol):
    assert np.max(np.abs(f64(o) - want[0])) <= o_tol
    assert np.max(np.abs(f64(lse) - want[1])) <= 1e-3


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("S_q,S_kv", SIZES)
def test_key_groups_against_the_oracle(S_q, S_kv, causal):
    for D in (64, 128):
        scale = synth.default_scale(D)
        for dtype, dt, o_tol in (("bf16", torch.bfloat16, 2e-2), ("f16", torch.float16, 4e-3)):
            q, k, v = synth.make_qkv(1, 3, S_q, S_kv, D, seed=77, sharp=(dtype == "bf16"), dtype=dtype)
            want = attn_ref(q, k, v, causal, scale, dtype=dtype)
            qd, kd, vd = (on_gpu(x, dt) for x in (q, k, v))
            if dtype == "f16":
                o, lse = binding.attn_fwd_f16(qd, kd, vd, causal=causal, scale=scale)
                check(o, lse, want, o_tol)
            for d, variant in TILINGS:
                if d == D:
                    print("S_q", S_q, "S_kv", S_kv, "D", D, "causal", causal, "variant", variant, flush=True)
                    o, lse = debug_lib.attn_fwd_variant(qd, kd, vd, causal, scale, variant)
                    check(o, lse, want, o_tol)


# heads, S_q, S_kv, ranges: one tile per range, ranges of unequal length, every count of lanes of the merge, many rows
SPLITS = [(2, 1, 130, 2), (3, 1, 5000, 3), (2, 64, 5000, 2), (2, 65, 3000, 5), (1, 130, 9000, 17), (2, 257, 4097, 8),
          (40, 129, 2000, 16), (300, 2, 300, 4), (2, 7, 12800, 200), (70, 200, 4200, 2)]


@pytest.mark.parametrize("heads,S_q,S_kv,n_split", SPLITS)
def test_ranges_against_the_oracle(heads, S_q, S_kv, n_split):
    for D in (64, 128):
        scale = synth.default_scale(D)
        for dtype, dt, o_tol, call in (("bf16", torch.bfloat16, 2e-2, binding.attn_fwd_splitkv),
                                       ("f16", torch.float16, 4e-3, binding.attn_fwd_splitkv_f16)):
            q, k, v = synth.make_qkv(1, heads, S_q, S_kv, D, seed=78, sharp=(heads == 3), dtype=dtype)
            qd, kd, vd = (on_gpu(x, dt) for x in (q, k, v))
            print("heads", heads, "S_q", S_q, "S_kv", S_kv, "D", D, dtype, "ranges", n_split, flush=True)
            need = binding.attn_fwd_splitkv_workspace_bytes(1, heads, S_q, D, n_split)
            ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
            o, lse = call(qd, kd, vd, n_split, workspace=ws, scale=scale)
            keep = sorted({0, heads - 1})                     # two heads are enough for the oracle
            sel = lambda x: np.ascontiguousarray(x[:, keep])
            check(o[:, keep], lse[:, keep], attn_ref(sel(q), sel(k), sel(v), False, scale, dtype=dtype), o_tol)


# heads, S_q, S_kv: one tile, one round and several, workgroups that share a CU or not, both sides of the dispatch rules
BOTH_TILINGS = [(1, 64, 64), (3, 300, 200), (70, 515, 515), (130, 520, 520), (300, 100, 700), (520, 129, 131), (600, 70, 90)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads,S_q,S_kv", BOTH_TILINGS)
def test_the_128_row_tilings_give_the_bits_of_the_256_row_ones(heads, S_q, S_kv, causal):
    g = torch.Generator(device="cuda")
    g.manual_seed(heads)
    for D, wide, narrow in ((64, debug_lib.FWD_D64_8_WAVES, debug_lib.FWD_D64_4_WAVES),
                            (128, debug_lib.FWD_D128_ONE_WAVE_PER_SIMD, debug_lib.FWD_D128_2_WAVES)):
        x = [torch.empty((1, heads, S, D), device="cuda").normal_(0, 2, generator=g) for S in (S_q, S_kv, S_kv)]
        for dt in (torch.bfloat16, torch.float16):
            q, k, v = (t.to(dt) for t in x)
            print("heads", heads, "S_q", S_q, "S_kv", S_kv, "D", D, "causal", causal, dt, flush=True)
            want = debug_lib.attn_fwd_variant(q, k, v, causal, synth.default_scale(D), wide)
            for variant in (narrow, debug_lib.FWD_AS_DISPATCHED):
                got = debug_lib.attn_fwd_variant(q, k, v, causal, synth.default_scale(D), variant)
                assert all(torch.equal(a, b) for a, b in zip(got, want)), variant


# queries, keys (with S_q >= 64 one key group works on all keys)
HIDDEN = [(1, 200), (31, 96), (33, 64), (40, 4096), (63, 130), (64, 100)]


@pytest.mark.parametrize("S_q,S_kv", HIDDEN)
def test_keys_that_no_query_sees_leave_no_trace(S_q, S_kv):
    """Causal: the keys from S_q on are masked for every row, so what K holds there reaches no output bit, NaN included."""
    for D in (64, 128):
        for dt, call in ((torch.bfloat16, binding.attn_fwd), (torch.float16, binding.attn_fwd_f16)):
            g = torch.Generator(device="cuda")
            g.manual_seed(S_q)
            q, k, v = (torch.empty((1, 2, S, D), device="cuda").normal_(generator=g).to(dt) for S in (S_q, S_kv, S_kv))
            print("S_q", S_q, "S_kv", S_kv, "D", D, dt, flush=True)
            want = call(q, k, v, causal=True)
            assert all(torch.isfinite(x).all() for x in want)
            for value in (float("nan"), float("inf"), float("-inf")):
                k[:, :, S_q:] = value
                assert all(torch.equal(x, y) for x, y in zip(call(q, k, v, causal=True), want)), value


# queries, keys, keys whose score is -inf, key ranges (0: attn_fwd)
NO_WEIGHT = [(1, 256, (96, 256), 0), (5, 500, (100, 500), 0), (40, 2000, (1000, 1500), 0), (63, 192, (64, 192), 0),
             (1, 1024, (96, 256), 4), (33, 5000, (1280, 1500), 2), (64, 4096, (256, 384), 8)]


@pytest.mark.parametrize("S_q,S_kv,span,n_split", NO_WEIGHT)
def test_keys_with_a_score_of_minus_infinity_weigh_nothing(S_q, S_kv, span, n_split):
    """Finite inputs whose products overflow (a padding key marked by one feature of the lowest value): the first keys of a
    group may then all weigh nothing.  The same as without those keys, in another order of the sums: bars as above."""
    for D in (64, 128):
        scale = synth.default_scale(D)
        g = torch.Generator(device="cuda")
        g.manual_seed(S_q)
        q, k, v = (torch.empty((1, 3, S, D), device="cuda").normal_(generator=g).bfloat16() for S in (S_q, S_kv, S_kv))
        q[..., 0], k[..., 0] = 4.0, 0.0
        k[:, :, span[0]:span[1], 0] = torch.finfo(torch.bfloat16).min
        keep = torch.cat([torch.arange(span[0]), torch.arange(span[1], S_kv)])
        print("S_q", S_q, "S_kv", S_kv, "D", D, "ranges", n_split, flush=True)
        got = ([binding.attn_fwd_splitkv(q, k, v, n_split, scale=scale)] if n_split else
               [binding.attn_fwd(q, k, v, scale=scale),
                debug_lib.attn_fwd_variant(q, k, v, False, scale, debug_lib.FWD_KEY_GROUPS)])
        s = torch.matmul(f64_t(q), f64_t(k)[:, :, keep].transpose(-1, -2)) * scale
        want = (torch.matmul(torch.softmax(s, -1), f64_t(v)[:, :, keep]).numpy(), torch.logsumexp(s, -1).numpy())
        for o, lse in got:
            check(o, lse, want, 2e-2)


def f64_t(t):
    return t.double().cpu()
