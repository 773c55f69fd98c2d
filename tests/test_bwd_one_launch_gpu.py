"""The backward launch that holds both sweeps, on sizes where its tile queue can go wrong: fewer tiles than XCDs, tile
counts that are no multiple of 8 in either sweep (entries between the sweeps that stand for nothing), one more tile than
workgroups, workgroups that pass from one sweep to the other.
Against the compiler-scheduled sweeps of the debug build (one launch each; the bar of the schedule-equivalence test), and
every element of the outputs written."""
import pytest
import torch

import debug_lib
from paper_2512_18134_amd import binding, synth

pytestmark = pytest.mark.gpu

# heads, S_q, S_kv (128-row tiles per sweep)
SIZES = [(1, 1, 1), (1, 100, 900), (1, 900, 100), (3, 129, 385), (5, 640, 129), (11, 1500, 1500), (16, 1025, 1024),
         (17, 1990, 2000), (9, 300, 7000), (9, 7000, 300), (64, 700, 770), (130, 900, 900),
         (56, 100, 1100)]   # (without a mask: one sweep after the other)


def rel(x, y):
    return float((x.float() - y.float()).norm() / y.float().norm())


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads,S_q,S_kv", SIZES)
def test_both_sweeps_in_one_launch(heads, S_q, S_kv, causal):
    for D in (64, 128):
        g = torch.Generator(device="cuda")
        g.manual_seed(S_q + S_kv)
        mk = lambda S: torch.empty((1, heads, S, D), device="cuda").normal_(generator=g).bfloat16()
        q, k, v, d_o = mk(S_q), mk(S_kv), mk(S_kv), mk(S_q)
        scale = synth.default_scale(D)
        print("heads", heads, "S_q", S_q, "S_kv", S_kv, "D", D, "causal", causal, flush=True)
        o, lse = binding.attn_fwd(q, k, v, causal=causal, scale=scale)
        nan = lambda t: torch.full_like(t, float("nan"))
        got = binding.attn_bwd(q, k, v, o, d_o, lse, nan(q), nan(k), nan(v), causal=causal, scale=scale)
        want = debug_lib.attn_bwd_plain(q, k, v, o, d_o, lse, causal, scale)
        for x, y in zip(got, want):
            assert torch.isfinite(x.float()).all()
            # one key, or one query: dS is a difference of equal numbers, its sign is rounding
            assert rel(x, y) <= 1e-2 or float(y.float().abs().max()) <= 2e-2
        if causal and S_kv > S_q:
            assert not got[1][:, :, S_q:].any() and not got[2][:, :, S_q:].any()


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
def test_keys_that_no_query_sees_get_plain_zeros(dt):
    fwd, bwd = ((binding.attn_fwd, binding.attn_bwd) if dt == torch.bfloat16 else
                (binding.attn_fwd_f16, binding.attn_bwd_f16))
    for D in (64, 128):
        q, k, v, d_o = (torch.randn((1, 2, S, D), device="cuda").to(dt) for S in (100, 700, 700, 100))
        o, lse = fwd(q, k, v, causal=True)
        _, dk, dv = bwd(q, k, v, o, d_o, lse, causal=True)
        for t in (dk, dv):      # all bits zero: no negative zeros
            assert not t[:, :, 100:].contiguous().view(torch.int16).any()
