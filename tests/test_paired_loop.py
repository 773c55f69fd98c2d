"""The forward loop whose waves test their row sums in pairs (gen_attn_loop.PairedGen), on its generated text: the rules the
hardware does not enforce (asm_emit.check_stream) on the main path and through every out-of-line section, the barriers and
direct loads of waves with fewer tiles than their workgroup, and what a wave leaves in LDS for the other one of its pair;
the rule that takes it; and its results against the tiling of 64-row waves, bit for bit."""
import ctypes
import os
import re
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import debug_lib  # noqa: E402
from test_generated_loops import asm_emit, gen_attn_loop, scalar_run  # noqa: E402

PAIRED = [(name, dt) for name in gen_attn_loop.PAIRED for dt in ("bf16", "f16")]


def make(name, dtype="bf16"):
    g = gen_attn_loop.PairedGen(name, dtype=dtype)
    g.generate()
    return g, [l.replace("%=", "") for l in g.lines]


def n_mfma(path):
    return sum(l.startswith("v_mfma") for l in path)


@pytest.mark.parametrize("name,dtype", PAIRED)
def test_main_path_twice_round(name, dtype):
    g, lines = make(name, dtype)
    path = asm_emit.walk(lines, loop_label="BODY0_", loop_visits=2)
    assert n_mfma(path) == g.NQKG + 11 * g.NM
    assert asm_emit.check_stream(path) == len(path)
    # every barrier is met with this wave's LDS accesses done: its sums are there, and it reads no ring stage any more
    for i, l in enumerate(path):
        if l == "s_barrier":
            assert "lgkmcnt(0)" in path[i - 1]


@pytest.mark.parametrize("name", list(gen_attn_loop.PAIRED))
@pytest.mark.parametrize("b", range(4))
def test_out_of_line_sections(name, b):
    g, lines = make(name)
    loads = ["KSLOW%d_" % b, "VSLOW%d_" % b]
    for detour in (["SLOW%d_" % b], ["SPECIAL%d_" % b] + loads, ["SPECIAL%d_" % b, "NOMASK%d_" % b] + loads,
                   ["SPECIAL%d_" % b, "SLOW%d_" % b] + loads):
        path = asm_emit.walk(lines, take=detour, loop_label="BODY0_", loop_visits=2)
        assert asm_emit.check_stream(path) == len(path)
        assert n_mfma(path) == g.NQKG + 11 * g.NM
    last = ["SPECIAL%d_" % b, "TOPL%d_" % b]
    for detour in (last, ["SPECIAL%d_" % b, "NOMASK%d_" % b, "TOPL%d_" % b], last + ["SLOWM%d_" % b], last + ["SLOWL%d_" % b],
                   last + ["SLOWM%d_" % b, "SLOWL%d_" % b]):
        path = asm_emit.walk(lines, take=detour + ["DONE_"], loop_label="BODY0_", loop_visits=2)
        assert asm_emit.check_stream(path) == len(path)
        assert path[-1].startswith("s_nop") and any(l.startswith("s_mov_b32 m0, s") for l in path[-4:])
        # the trailing half, P V of the tile before, P V of the last tile
        tail = path[len(path) - 1 - path[::-1].index("s_barrier"):]
        assert n_mfma(tail) == g.NPVG and not any(l.startswith("global_load_lds") for l in tail)
    # owed loads of this iteration and the next, then two iterations of standing by with loads and one without
    path = asm_emit.walk(lines, take=last + ["OWED%d_" % b, "NEXTOWED%d_" % b, "STANDBYNEXT_"], loop_label="STANDBY_", loop_visits=3)
    assert asm_emit.check_stream(path) == len(path)


@pytest.mark.parametrize("name", list(gen_attn_loop.PAIRED))
def test_single_tile(name):
    g, lines = make(name)
    path = asm_emit.walk(lines, take=["SPECIALF_", "KSLOWF_", "VSLOWF_", "SPECIAL1_", "EXIT1_", "DONE_"])
    assert asm_emit.check_stream(path) == len(path)
    assert n_mfma(path) == g.NQKG + g.NPVG


@pytest.mark.parametrize("name", list(gen_attn_loop.PAIRED))
def test_waves_keep_step(name):
    """n tiles: n + 1 barriers for every wave, whatever its own tile count, and the same loads between them."""
    g, lines = make(name)
    for n in (1, 2, 3, 4, 5, 6, 7, 9, 13):
        for t_full in (n, n - 1):
            for j_mask in sorted({0, n // 2, n - 1, n}):
                full = scalar_run(g, lines, n, n, t_full, j_mask)
                assert len(full) == n + 1
                for j, loads in enumerate(full):     # iteration j brings K(j+4) and V(j+2), the last one nothing
                    want = [("k", j + 4, j % 4)] * g.NLD + [("v", j + 2, (j + 2) % 4)] * g.NLD
                    if j >= n - 1 and n > 1 or j == n:
                        want = []
                    got = sorted((w, t, ((a - ((1 << 20) if w == "k" else (1 << 21))) // g.TB)) for w, t, a in loads)
                    assert got == sorted(want), (n, t_full, j_mask, j)
                for n_wave in range(1, n):
                    part = scalar_run(g, lines, n, n_wave, t_full, j_mask)
                    assert [sorted(x) for x in part] == [sorted(x) for x in full], (n, n_wave, t_full, j_mask)


def exchange(g, lines, n, n_wave):
    """Per barrier interval of a wave's run: its accesses to the row sums in LDS, as (read / write, register, slot)."""
    place = []

    def mark(l):     # as a direct load that the scalar run records, through a pair of its own and with its number as offset
        m = re.match(r"ds_(write|read)_b32 v(\d+), v(\d+)(?: offset:(\d+))?$", l.strip())
        if m is None:    # (m0 stays 0, so that a load's LDS address is its offset)
            return "s_nop 0" if re.search(r"\bm0,", l) else l
        place.append((m.group(1), int(m.group(3 if m.group(1) == "write" else 2)), 1 if m.group(4) else 0))
        return "global_load_lds_dwordx4 v0, s[90:91] offset:%d" % (len(place) - 1)

    sg = {g.s_ntiles: n, g.s_nw: n_wave, g.s_tfull: n, g.s_jmask: n, g.s_skvm1: n * g.BN - 1}
    events = asm_emit.run_scalar([mark(l) for l in lines], sg, g.BN, g.TB,
                                 {"k": (g.s_kbase, g.s_kptr), "v": (g.s_vbase, g.s_vptr), "x": (88, 90)})
    out = [[]]
    for e in events:
        if e[0] == "barrier":
            out.append([])
        elif e[1] == "x":
            out[-1].append(place[e[3]])
    return out


@pytest.mark.parametrize("name", list(gen_attn_loop.PAIRED))
def test_sums_of_every_tile_are_there_for_the_other_wave(name):
    """Tile j's sums are written before barrier j + 1 and read behind it, in the slot of j's parity; a wave with one tile less
    than the other of its pair leaves zeros for that tile, and never before the other has read what was there."""
    g, lines = make(name)
    for n in (1, 2, 3, 4, 5, 6, 9):
        for n_wave in sorted({max(1, n - 1), n}):
            seen = exchange(g, lines, n, n_wave)             # [interval]; interval i lies between barriers i - 1 and i
            assert len(seen) == n + 2
            for i, acc in enumerate(seen):
                j = i - 1                                    # the iteration that barrier i - 1 opens
                want = []
                if 0 <= j < n_wave:
                    want.append(("write", g.TLA, j % 2))
                if j == n_wave and n_wave > 1:               # zeros for the tile that only the other wave has
                    want.append(("write", g.TLB, j % 2))
                if n_wave == 1 and j == 0:
                    want.append(("write", g.TLA, 1))
                if 1 <= j <= n_wave and n_wave > 1:
                    want.append(("read", g.PS, (j - 1) % 2))
                assert sorted(acc) == sorted(want), (n, n_wave, i)


# where the rule of the dispatch was measured: heads, queries, keys, causal, taken
MEASURED = [(16, 128, 128, 1, 1), (16, 777, 777, 1, 1), (16, 1024, 1024, 0, 1), (32, 2048, 2048, 1, 1), (4, 6000, 6000, 1, 1),
            (1, 16384, 16384, 1, 1), (16, 2048, 2048, 0, 1), (24, 2816, 2816, 0, 1), (1, 64, 64, 0, 1), (213, 623, 623, 1, 1),
            (6, 5468, 5468, 0, 0), (128, 2048, 2048, 0, 0), (32, 4096, 4096, 1, 0), (32, 3845, 3845, 1, 0), (16, 16384, 16384, 0, 0),
            (310, 112, 960, 0, 0)]
# ... causal, up to 1024 keys: more than twice as many queries, beyond 160 32-key steps per workgroup and up to that (level), and
# fewer queries, where many tiles and long walks are as often ahead as behind
MEASURED += [(64, 9386, 989, 1, 0), (372, 2742, 832, 1, 0), (128, 10048, 704, 1, 0), (552, 1792, 748, 1, 0), (64, 8192, 512, 1, 1),
             (410, 1024, 1024, 1, 1), (757, 655, 1307, 1, 1), (420, 148, 148, 1, 1), (224, 384, 384, 1, 1), (173, 832, 832, 1, 1),
             (16, 4000, 300, 1, 1)]
# ... one round of the 256-row tiling against two 128-row tiles on some compute units
MEASURED += [(87, 344, 2557, 0, 0), (96, 320, 4494, 0, 0), (56, 557, 3839, 0, 0), (3, 13632, 2779, 1, 0), (6, 8256, 2233, 1, 0),
             (8, 6643, 1856, 1, 0), (32, 2158, 642, 1, 1), (80, 567, 567, 1, 1), (5, 8780, 4736, 1, 1), (4, 9152, 1984, 1, 1),
             (4, 7514, 1353, 0, 1)]


@pytest.mark.parametrize("heads,s_q,s_kv,causal,taken", MEASURED)
def test_taken_where_it_is_the_faster_tiling(heads, s_q, s_kv, causal, taken):
    rule = ctypes.CDLL(debug_lib.PATH).attn_fwd_tiling
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int] * 5
    assert (rule(128, heads, s_q, s_kv, causal) == 4) == bool(taken)


# edges of the 32-row waves and their pairs, of the tiles and of the mask; waves and pairs without rows; one tile, several
# tiles of a workgroup's queue
SHAPES = [(1, 64, 64), (2, 32, 32), (1, 33, 40), (3, 65, 65), (2, 100, 31), (1, 1, 1), (2, 130, 200), (4, 777, 777), (3, 515, 129),
          (2, 300, 1000), (1, 1000, 300), (5, 97, 2000), (300, 300, 300)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("h,s_q,s_kv", SHAPES)
def test_same_bits_as_64_row_waves(h, s_q, s_kv, causal, dtype):
    """... whatever moves the references: offsets of rows and keys that make the test fail often, now and then, or never."""
    import torch
    t = torch.bfloat16 if dtype == "bf16" else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(7 * s_q + s_kv + h)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda")
    for spread in (0.0, 0.6, 2.0):
        q = (normal(1, h, s_q, 128) + spread * normal(1, h, s_q, 1)).to(t)
        k = (normal(1, h, s_kv, 128) + spread * normal(1, h, s_kv, 1)).to(t)
        v = normal(1, h, s_kv, 128).to(t)
        o, lse = debug_lib.attn_fwd_variant(q, k, v, causal, 128 ** -0.5, debug_lib.FWD_D128_2_WAVES)
        o2, lse2 = debug_lib.attn_fwd_variant(q, k, v, causal, 128 ** -0.5, debug_lib.FWD_D128_PAIRED)
        assert torch.equal(o.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, lse2)
        assert not torch.isnan(lse).any()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("what", ["keys", "first keys", "rows", "plus", "nan"])
@pytest.mark.parametrize("h,s_q,s_kv", [(2, 64, 64), (3, 130, 200), (2, 333, 333), (1, 515, 129)])
def test_infinite_and_nan_scores(h, s_q, s_kv, what, causal, dtype):
    """Scores of -inf in the middle and at the start of a walk, for all rows or for some, +inf and NaN.  The same rows are NaN as
    with 64-row waves, and the others the same bits, but for one case: with a causal mask, a row whose scores have all been -inf
    makes the row sums of a 64-row wave NaN also in the tile that its block does not have, and moves the references of
    the rows beside it there, which 32-row waves leave.  Either reference is right: P is rounded to 16 bits (relative error up
    to eps / 2) against either, and O again."""
    import torch
    t = torch.bfloat16 if dtype == "bf16" else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(s_q + 3 * s_kv)
    q, k, v = (torch.randn((1, h, s, 128), generator=gen, device="cuda") for s in (s_q, s_kv, s_kv))
    q[..., 0], k[..., 0] = q[..., 0].abs() + 0.1, k[..., 0].abs() + 0.1   # (a factor of inf in place 0 has a known sign)
    inf = float("inf")
    bad = torch.zeros((1, h, s_q), dtype=torch.bool, device="cuda")
    if what == "keys":
        k[:, :, 32:min(70, s_kv - 1), 0] = -inf
        k[:, :, s_kv - 1, 0] = -inf
    elif what == "first keys":      # a walk that starts with a whole tile of them has no reference that gives numbers
        k[:, :, :7, 0] = -inf
        bad[:, :, :7] = causal      # (rows that see no other key)
    else:
        rows = torch.tensor([3, 31, 32, 40, 63], device="cuda")
        q[:, :, rows, 0] = {"rows": -inf, "plus": inf, "nan": float("nan")}[what]
        bad[:, :, rows] = True
    q, k, v = q.to(t), k.to(t), v.to(t)
    o, lse = debug_lib.attn_fwd_variant(q, k, v, causal, 128 ** -0.5, debug_lib.FWD_D128_2_WAVES)
    o2, lse2 = debug_lib.attn_fwd_variant(q, k, v, causal, 128 ** -0.5, debug_lib.FWD_D128_PAIRED)
    assert torch.equal(torch.isnan(o).all(-1), bad) and torch.equal(torch.isnan(o2).all(-1), bad)
    assert torch.equal(torch.isnan(o).any(-1), bad) and torch.equal(torch.isnan(o2).any(-1), bad)
    assert torch.equal(torch.isnan(lse), torch.isnan(lse2))
    o, o2, v = o.float().nan_to_num(0.0), o2.float().nan_to_num(0.0), v.float()
    lse, lse2 = lse.masked_fill(bad, 0.0), lse2.masked_fill(bad, 0.0)
    assert torch.isfinite(lse).all()
    if causal and what in ("rows", "first keys"):      # rows without a finite score, all in the first 64-row block
        eps = torch.finfo(t).eps
        assert (o - o2).abs().max() <= 2 * eps * v.abs().max()     # (P twice, O twice, half an ulp each)
        assert (lse - lse2).abs().max() <= 1e-5
        o, o2, lse, lse2 = o[:, :, 64:], o2[:, :, 64:], lse[:, :, 64:], lse2[:, :, 64:]
    assert torch.equal(o, o2) and torch.equal(lse, lse2)
