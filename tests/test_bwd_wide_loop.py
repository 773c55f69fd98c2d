"""The backward loops whose waves own 64 rows (gen_attn_bwd_wide_loop.py), on their generated text: the rules the hardware
does not enforce (asm_emit.check_stream) on the main path and through every out-of-line section, and the barriers and
direct loads of waves that stand by in some of their workgroup's tiles; the rule that takes them; the registers of the
compiled kernels."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import debug_lib  # noqa: E402
from test_generated_loops import ROOT, asm_emit  # noqa: E402
import gen_attn_bwd_wide_loop  # noqa: E402

SWEEPS = [(ko, nw, dt) for ko in (True, False) for nw in (2, 4) for dt in ("bf16", "f16")]


def make(key_owner, waves, dtype="bf16"):
    g = gen_attn_bwd_wide_loop.WideGen(key_owner, dtype=dtype, NW=waves)
    g.generate()
    return g, [l.replace("%=", "") for l in g.lines]


def entry(key_owner):
    """Branches of a wave that computes its first tile at once (key owners test the stand-by loop first)."""
    return ["STANDBYEND_"] if key_owner else []


@pytest.mark.parametrize("key_owner,waves,dtype", SWEEPS)
def test_main_path_and_detours(key_owner, waves, dtype):
    g, lines = make(key_owner, waves, dtype)
    path = asm_emit.walk(lines, take=entry(key_owner), loop_label="BODY0_", loop_visits=2)
    assert sum(l.startswith("v_mfma") for l in path) == 16 + 2 * g.NST * g.NM
    assert asm_emit.check_stream(path) == len(path)
    if key_owner:       # a wave whose first tile lies in stage 2, after standing by twice
        path = asm_emit.walk(lines, take=["STANDBYEND_", "PRE2_"], loop_label="BODY0_", loop_visits=2)
        assert sum(l.startswith("v_mfma") for l in path) == 16 + (2 + 2 * g.NST) * g.NM
        assert asm_emit.check_stream(path) == len(path)
    for tag in ["P0"] + [str(b) for b in range(g.NST)]:
        masks = ["MASKLO%s_" % tag, "MASKHI%s_" % tag] if key_owner else ["MASKHI%s_" % tag]
        detours = [[m] for m in masks] + [masks]
        if tag != "P0":
            detours += [["SLOW%s_" % tag], masks + ["SLOW%s_" % tag]]
        for detour in detours:
            path = asm_emit.walk(lines, take=entry(key_owner) + detour, loop_label="BODY0_", loop_visits=2)
            assert asm_emit.check_stream(path) == len(path)
    if key_owner:
        for detour in (["MASKLOP2_"], ["MASKHIP2_"], ["MASKLOP2_", "MASKHIP2_"]):
            path = asm_emit.walk(lines, take=["STANDBYEND_", "PRE2_"] + detour, loop_label="BODY0_", loop_visits=2)
            assert asm_emit.check_stream(path) == len(path)


def intervals(g, lines, n, n_wave, t_full, t_begin=0):
    """Per barrier interval the loads (tensor, tile, ring place) of a wave's run, from the second barrier of the set-up on (two
    waves: the third follows its loads; the intervals on both sides of it are one here)."""
    sg = {g.s_ntiles: n, g.s_nw: n_wave, g.s_tfull: t_full, g.s_tbeg: t_begin, g.s_jlo: 0, g.s_jhi: n, g.s_strm1: 10 ** 6,
          g.s_lds: 1 << 20, g.s_ldsaux: 1 << 24}
    for base, at in ((g.s_t1base, 0), (g.s_t2base, 1 << 28), (g.s_auxbase, 0)):
        sg[base] = at
    # (the far half of a tile goes through one pair for both tensors: told apart by the address)
    bases = {"1": (g.s_t1base, g.s_ptr1), "2": (g.s_t2base, g.s_ptr2), "aux": (g.s_auxbase, g.s_ptra), "far": (200, g.s_far)}
    out = [[]]
    for e in asm_emit.run_scalar(lines, sg, g.BN, g.TB, bases):
        if e[0] == "barrier":
            out.append([])
        elif e[1] == "aux":
            out[-1].append(("aux", (e[3] - (1 << 24)) // 256))
        else:
            which, tile = ("12"[e[2] >= (1 << 28) // g.TB], e[2] % ((1 << 28) // g.TB)) if e[1] == "far" else e[1:3]
            out[-1].append((which, tile, (e[3] - (1 << 20))))
    return out if g.NW == 4 else out[:2] + [out[2] + out[3]] + out[4:]


@pytest.mark.parametrize("waves", [2, 4])
@pytest.mark.parametrize("key_owner", [True, False])
def test_waves_keep_step(key_owner, waves):
    """n tiles: the barriers of the set-up and one per tile for every wave, and between them the same loads, whichever tiles
    the wave computes; iteration j brings tile j + 3 into stage (j + 3) % 4."""
    g, lines = make(key_owner, waves)
    own = [0, 2, 4, 6][:waves]
    for n in (0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 13) if key_owner else (1, 2, 3, 4, 5, 6, 7, 8, 9, 13):
        for t_begin in (0, 3):
            for t_full in sorted({0, t_begin, t_begin + max(n - 1, 0), t_begin + n}):
                whole = intervals(g, lines, n, 0 if key_owner else n, t_full, t_begin)
                assert len(whole) == n + 3
                for j, loads in enumerate(whole[2:], -1):     # (the set-up's tiles 1 and 2 stand in the interval of "j = -1")
                    tiles = (1, 2) if j == -1 else (j + 3,)
                    want = [(t, t_begin + k, k % 4 * g.SB + (t == "2") * g.TB + i * 1024 * waves)
                            for k in tiles for t in ("1", "2") for i in range(g.NLD)]
                    if j == -1 and waves == 2:
                        want += [("2", t_begin, g.TB + i * 2048) for i in range(g.NLD)]
                    assert sorted(l for l in loads if l[0] != "aux") == sorted(want), (n, t_begin, t_full, j)
                    assert [l[1] for l in loads if l[0] == "aux"] == ([k % 4 for k in tiles] if key_owner else [])
                parts = [x for x in own if x < n] + [n] if key_owner else range(0, n)
                for n_wave in parts:
                    part = intervals(g, lines, n, n_wave, t_full, t_begin)
                    assert [sorted(x) for x in part] == [sorted(x) for x in whole], (n, n_wave, t_full)


def test_the_rule_between_the_tilings():
    pick = ctypes.CDLL(debug_lib.PATH).attn_bwd_pick_tiling
    pick.restype, pick.argtypes = ctypes.c_int, [ctypes.c_int] * 5 + [ctypes.POINTER(ctypes.c_float)]
    est = (ctypes.c_float * 3)()
    for heads, s_q, s_kv, causal, cus, want in [
            (128, 4096, 4096, 0, 256, 2), (32, 2048, 2048, 0, 256, 2), (16, 16384, 16384, 0, 256, 2), (128, 1024, 1024, 1, 256, 3),
            (300, 300, 300, 0, 256, 3), (16, 1024, 1024, 0, 256, 1), (1, 1, 1, 0, 256, 1), (1, 1, 1, 1, 256, 1),
            (123, 72, 5938, 0, 256, 3), (128, 4096, 4096, 0, 0, 1)]:
        assert pick(heads, s_q, s_kv, causal, cus, est) == want, (heads, s_q, s_kv, causal, cus, list(est))
    for heads, s_q, s_kv in [(1, 1, 1), (32768, 1, 1), (1 << 20, 64, 64), (3, 8000000, 1), (1, 1, 8000000)]:
        for causal in (0, 1):
            assert pick(heads, s_q, s_kv, causal, 256, est) in (1, 2, 3) and all(0 < x < 1e9 for x in est)


def test_tiles_of_an_xcd_in_its_queues_order():
    tile = ctypes.CDLL(debug_lib.PATH).attn_bwd_xcd_tile
    tile.restype, tile.argtypes = ctypes.c_int, [ctypes.c_int] * 3 + [ctypes.c_longlong] + [ctypes.c_int] * 2 + [ctypes.POINTER(ctypes.c_int)]
    want = ctypes.c_int()
    for heads in (1, 3, 7, 8, 9, 16, 21, 40, 130):
        for n_t in (1, 2, 5, 9, 33):
            for head_bytes in (4 * 256 * 128, 4 * 3000 * 128, 4 * 20000 * 128):
                for causal in (0, 1):
                    for xcd in (0, 3, 7):
                        for i in range((heads * n_t + 7) // 8 + 1):
                            assert tile(heads, n_t, causal, head_bytes, xcd, i, want) == want.value, (heads, n_t, causal, xcd, i)
                        assert want.value == -1


def test_registers_of_the_compiled_kernels(tmp_path):
    """One wave per SIMD with all 512 registers: nothing of a vector register in scratch memory."""
    from paper_2512_18134_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    out = str(tmp_path / "bwd.s")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([hipcc] + flags + ["-S", "--cuda-device-only", "-o", out,
                                      os.path.join(ROOT, "paper_2512_18134_amd", "csrc", "attn_bwd.hip")],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = open(out).read()
    seen = 0
    for block in text[text.index("amdhsa.kernels:"):].split("  - .agpr_count:")[1:]:
        if not re.search(r"\.name:\s+\S*attn_bwd_wide_(planned_)?kernel", block):
            continue
        value = lambda key: int(re.search(r"\.%s:\s+(\d+)" % key, block).group(1))
        assert value("private_segment_fixed_size") == 0 and value("vgpr_spill_count") == 0 and value("vgpr_count") <= 512
        seen += 1
    assert seen == 16         # waves, causal, element type, with a plan or without
