"""Split-KV ranges of many queries (8 waves, 256-row tiles) and partial rows that leave whole (D = 64): sizes at the edges of tiles,
waves and ranges, each head against the fp64 oracle on the first and last rows and in every
element against the unsplit call; the bars are test_splitkv_gpu.py's (fp16: a quarter, as its significand has three bits more)."""
import numpy as np
import pytest
import torch

from oracle.attn_oracle import attn_ref
from paper_2512_18134_amd import binding, synth

pytestmark = pytest.mark.gpu

# heads, S_q, S_kv, D, ranges: more than 256 workgroups, the last range short, waves without rows (129, 200, 300)
CASES = [(24, 129, 2100, 128, 4), (12, 256, 4097, 128, 8), (24, 193, 1100, 128, 2), (9, 300, 6000, 128, 7), (40, 200, 2100, 64, 4),
         (24, 300, 3333, 64, 5)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "H%d_Sq%d_Skv%d_D%d_split%d" % c)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_wide_ranges(case, dtype):
    H, S_q, S_kv, D, n_split = case
    print("case", case, dtype, flush=True)
    q, k, v = synth.make_qkv(1, H, S_q, S_kv, D, seed=S_q + S_kv)
    scale = synth.default_scale(D)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    f32 = [synth.bf16_bits_to_f32(x) for x in (q, k, v)]
    dev = [torch.from_numpy(x).cuda().to(dt) for x in f32]
    if dtype == "f16":       # (the bits that the oracle reads)
        q, k, v = (x.cpu().view(torch.int16).numpy().view(np.uint16) for x in dev)
    split, plain = ((binding.attn_fwd_splitkv, binding.attn_fwd) if dtype == "bf16" else
                    (binding.attn_fwd_splitkv_f16, binding.attn_fwd_f16))
    bar = 2e-2 if dtype == "bf16" else 5e-3
    o, lse = split(*dev, n_split, torch.full_like(dev[0], float("nan")),
                   torch.full((1, H, S_q), float("nan"), device="cuda"), scale=scale)
    o1, lse1 = plain(*dev, scale=scale)
    assert float((o.float() - o1.float()).abs().max()) <= bar and float((lse - lse1).abs().max()) <= 1e-3
    for h in (0, H - 1):
        want, want_lse = attn_ref(q[:, h:h + 1], k[:, h:h + 1], v[:, h:h + 1], False, scale, dtype=dtype)
        got = o[:, h:h + 1].double().cpu().numpy()
        assert np.max(np.abs(got - want)) <= bar
        assert np.max(np.abs(lse[:, h:h + 1].double().cpu().numpy() - want_lse)) <= 1e-3


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_wide_ranges_whose_last_wave_has_one_row(dtype):
    """193 queries in enough workgroups (24 heads of them, above, take the key groups); and the other cases have enough as well."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    case = (40, 193, 1100, 128, 2)
    for H, S_q, S_kv, D, n_split in [case] + [c for c in CASES if c[1] != 193]:
        split_len = -(-(-(-S_kv // n_split)) // 64) * 64
        tiles = H * -(-S_kv // split_len) * -(-S_q // (64 if D == 128 else 128))
        # (what launch_splitkv gives to the 8-wave tiling)
        assert S_q > (64 if D == 128 else 128) and tiles > cus, (H, S_q, S_kv, D, n_split)
    test_wide_ranges(case, dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("sharp", [False, True])
def test_a_row_keeps_its_bits_beside_more_queries(dtype, sharp):
    """Up to 128 queries and above, D = 128 ranges run in the same 32-row waves, whose references come from their own rows: 128
    queries of a call give what they give in a call of their own."""
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    rnd = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
    mk = lambda S, off: (rnd(1, 40, S, 128) + (2 * rnd(1, 40, S, 1) if off else 0)).to(dtype)
    q, k, v = mk(300, sharp), mk(2100, sharp), mk(2100, False)
    split = binding.attn_fwd_splitkv if dtype == torch.bfloat16 else binding.attn_fwd_splitkv_f16
    print("rows", dtype, "sharp", sharp, flush=True)
    o, lse = split(q, k, v, 4)          # (160 ranges: more than 256 workgroups of 64 rows in either call)
    few, few_lse = split(q[:, :, :128].contiguous(), k, v, 4)
    assert torch.equal(o[:, :, :128].contiguous().view(torch.int16), few.view(torch.int16))
    assert torch.equal(lse[:, :, :128], few_lse)
