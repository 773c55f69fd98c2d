"""Backward in 64-row waves (owner tiles of 256 rows, and of 128), forced through the debug build: the same bits as in 32-row waves,
at the sizes where tiles, waves, ring stages and the queue end; infinities and NaN reach no element that they do not reach
there."""
import ctypes

import pytest
import torch

import debug_lib
from paper_2512_18134_amd import binding, synth

pytestmark = pytest.mark.gpu

# heads, S_q, S_kv
SIZES = [(1, 1, 1), (1, 31, 33), (2, 64, 65), (1, 255, 257), (3, 256, 256), (2, 300, 97), (1, 97, 300), (5, 513, 700), (9, 1000, 33),
         (17, 777, 1300), (3, 100, 1100), (33, 1025, 1024), (40, 1500, 1900), (130, 260, 260),
         (12, 900, 5000), (100, 128, 1500), (9, 4000, 4000)]    # (these with a plan of the workgroups' walks)


def run(tiling, q, k, v, o, d_o, lse, causal, scale):
    call = debug_lib.lib().attn_bwd_tiling
    call.restype = ctypes.c_int
    call.argtypes = [ctypes.c_void_p] * 10 + [ctypes.c_int] * 6 + [ctypes.c_float, ctypes.c_void_p, ctypes.c_int]
    out = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    ws = torch.empty(2 * lse.numel(), dtype=torch.float32, device="cuda")
    rc = call(*[t.data_ptr() for t in (q, k, v, o, d_o, lse, *out, ws)], q.shape[0], q.shape[1], q.shape[2], k.shape[2],
              int(q.dtype == torch.float16), int(causal), float(scale), torch.cuda.current_stream().cuda_stream, tiling)
    assert rc == 0
    return out


def inputs(heads, S_q, S_kv, dt, sharp):
    g = torch.Generator(device="cuda")
    g.manual_seed(S_q * 3 + S_kv)
    rnd = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
    mk = lambda S, off: (rnd(1, heads, S, 128) + (2 * rnd(1, heads, S, 1) if off else 0)).to(dt)
    return mk(S_q, sharp), mk(S_kv, sharp), mk(S_kv, False), mk(S_q, False)


def bits(t):
    return t.view(torch.int16)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads,S_q,S_kv", SIZES)
def test_same_bits_as_32_row_waves(heads, S_q, S_kv, causal):
    scale = synth.default_scale(128)
    for dt, fwd in ((torch.bfloat16, binding.attn_fwd), (torch.float16, binding.attn_fwd_f16)):
        for sharp in (False, True):
            print("heads", heads, "S_q", S_q, "S_kv", S_kv, "causal", causal, dt, "sharp", sharp, flush=True)
            q, k, v, d_o = inputs(heads, S_q, S_kv, dt, sharp)
            o, lse = fwd(q, k, v, causal=causal, scale=scale)
            want = run(1, q, k, v, o, d_o, lse, causal, scale)
            for tiling in (2, 3):
                got = run(tiling, q, k, v, o, d_o, lse, causal, scale)
                for x, y in zip(got, want):
                    assert torch.isfinite(x.float()).all() and torch.equal(bits(x), bits(y))


@pytest.mark.parametrize("causal", [False, True])
def test_infinite_and_nan_inputs(causal):
    """A masked element's zero weight times an infinity is NaN, within the rows that share a wave: fewer of them here than in a
    tile of 128 rows, never others."""
    scale = synth.default_scale(128)
    q, k, v, d_o = inputs(3, 700, 700, torch.bfloat16, False)
    o, lse = binding.attn_fwd(q, k, v, causal=causal, scale=scale)
    d_o[0, 0, 300, 5], d_o[0, 1, 10, 7], v[0, 2, 650, 3], k[0, 1, 400, 9] = float("inf"), float("nan"), float("-inf"), float("nan")
    want = run(1, q, k, v, o, d_o, lse, causal, scale)
    for x, y in [p for tiling in (2, 3) for p in zip(run(tiling, q, k, v, o, d_o, lse, causal, scale), want)]:
        fine = torch.isfinite(y.float())
        assert torch.equal(bits(x)[fine], bits(y)[fine])
        assert not fine.all()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads,S_q,S_kv", [(60, 100, 2500), (24, 2500, 300), (30, 2900, 2900)])
def test_planned_walks_at_d64(heads, S_q, S_kv, causal):
    """Every tile written once, against the compiler-scheduled sweeps (the bar of the schedule-equivalence test)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(heads + S_q)
    mk = lambda S: torch.empty((1, heads, S, 64), device="cuda").normal_(generator=g).bfloat16()
    q, k, v, d_o = mk(S_q), mk(S_kv), mk(S_kv), mk(S_q)
    scale = synth.default_scale(64)
    print("heads", heads, "S_q", S_q, "S_kv", S_kv, "causal", causal, flush=True)
    o, lse = binding.attn_fwd(q, k, v, causal=causal, scale=scale)
    got = binding.attn_bwd(q, k, v, o, d_o, lse, *[torch.full_like(t, float("nan")) for t in (q, k, v)], causal=causal, scale=scale)
    for x, y in zip(got, debug_lib.attn_bwd_plain(q, k, v, o, d_o, lse, causal, scale)):
        assert torch.isfinite(x.float()).all() and float((x.float() - y.float()).norm()) <= 1e-2 * float(y.float().norm())
