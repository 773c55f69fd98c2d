#!/usr/bin/env python3
"""Emit the main loop of the attention-backward sweeps whose waves own 64 rows (gfx950, D = 128, one wave per SIMD).

The same mathematics, order of sums and results, bit for bit, as the loops of gen_attn_bwd_loop.py, whose waves own 32 rows
and read one 1 KB operand from LDS for every MFMA: four waves at the full matrix rate ask the LDS for all of its 128 bytes a
cycle, and that is what bounds them.  Here a wave owns two blocks of 32 rows (A and B), and every operand read from
LDS feeds two MFMAs.

What makes room for twice the accumulators is that S and dP are not buffered over three stages.  The products of ONE tile
are ordered so that its element-wise work always has other products beside it (slots of one MFMA, iteration j):

    key owners, 64 slots                          query owners, 48 slots
     0-15  dP(j) = dO V^T                          0-15  dP(j) = V dO^T
    16-31  dV += dO^T P(j)                        16-31  S(j+1) = K Q^T   (two buffers)
    32-47  S(j+1) = Q K^T  (P(j) is done with)    32-47  dQ += K^T dS(j)
    48-63  dK += Q^T dS(j)
    VALU:  P(j) from slot 50 of iteration j-1 on,  VALU:  exp2 from slot 34 of iteration j-1 on, dS(j) from
           dS(j) from slot 18 on                          slot 18 on

Registers, key owners: the accumulators take all 256 AGPRs; the owner's K and V rows (128), S, dP (32 each), P in 16 bits,
which dS in 16 bits overwrites (16), four operand buffers (16), two quarters of a tile's LSE' (8), addresses and mask limits (22): 254 VGPRs.
Query owners: accumulators and the owner's Q and dO rows in 256 AGPRs, the rest in VGPRs.

Streamed tiles of 32 rows arrive by direct global->LDS loads in a ring of four stages of 16 KB (both tensors' tile: every
stage lies within the reads' 16-bit offsets, so there is one set of addresses), three tiles ahead of their use, one
barrier per tile.  That barrier stands inside the iteration, ahead of the first read of tile j+1: it publishes that tile and
frees the stage of tile j-1, which tile j+3 then goes into.

Waves that have nothing to do in a tile (key owners whose keys all lie behind the tile's queries, query owners whose
queries all lie before its keys, waves without rows) stand by: the barrier and their share of the loads, no products.

Hazards as in gen_attn_bwd_loop.py; the tests check them on the emitted text (asm_emit.check_stream).

usage: gen_attn_bwd_wide_loop.py <kv|q> <waves: 2|4> <out.inc> [bf16|f16]
"""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from asm_emit import Emitter, parse  # noqa: E402


def deal(ops, fixed_cost, first, n, cost=lambda ins: 2.5 if ins.startswith("v_exp") else 1.0):
    """Deal `ops`, a list of (instruction, earliest slot, slot it has to precede), over the slots first .. first + n - 1
    so that every slot carries about the same issue cost; fixed_cost(slot): what the slot holds already.  In order, but that
    an operation may pass others that have to wait and do not share its registers.  Returns {slot: [instructions]}."""
    total = sum(cost(o[0]) for o in ops) + sum(fixed_cost(s) for s in range(first, first + n))
    left = [o + parse(o[0])[1:] for o in ops]
    out = {s: [] for s in range(first, first + n)}
    done = 0.0
    for s in range(first, first + n):
        done += fixed_cost(s)
        written, read, k = set(), set(), 0           # by the operations passed over
        while k < len(left):
            ins, early, late, dst, src = left[k]
            if done + cost(ins) / 2 > total * (s - first + 1) / n and s < first + n - 1:
                break
            if early <= s and not ((dst | src) & written) and not (dst & read):
                assert s < late, ("too late", ins, s)
                out[s].append(ins)
                done += cost(ins)
                del left[k]
            else:
                written |= dst
                read |= src
                k += 1
    assert not left, left[0]
    return out


class WideGen(Emitter):
    D, BN, NST = 128, 32, 4
    KS, DB, ROWB = 8, 4, 256
    TB = BN * ROWB                  # one tensor's tile
    SB = 2 * TB                     # a stage: tile of the first tensor, tile of the second
    AHEAD = 3                       # tile j + AHEAD is loaded in iteration j

    def __init__(self, key_owner, dtype="bf16", NW=4, NF=None, PFD=None, W=None):
        Emitter.__init__(self)
        self.NW = NW                # waves of a workgroup
        self.NLD = self.TB // (NW * 1024)
        assert dtype in ("bf16", "f16")
        self.KO, self.dtype = bool(key_owner), dtype
        self.mfma = "v_mfma_f32_32x32x16_" + dtype
        self.cvt = "v_cvt_pk_%s_f32" % dtype
        self.NF = NF or (4 if key_owner else 8)
        self.PFD = PFD or (3 if key_owner else 5)
        self.W = W or (1 if key_owner else 2)
        self.NGRP = 2 * self.NLD + (1 if key_owner else 0)
        r = 0
        def take(n):
            nonlocal r
            r += n
            return r - n
        two = lambda n: [take(n), take(n)]
        self.ACC = 0
        if self.KO:                 # AGPRs: dK [block][db], dV [block][db]
            self.NA = 256
            self.B1, self.B2 = two(32), two(32)
            self.S = [two(16)] * 2
        else:                       # AGPRs: dQ [block][db], Q, dO
            self.B1, self.B2, self.NA = [128, 160], [192, 224], 256
            self.S = [two(16), two(16)]
        self.DP = two(16)
        self.P = [two(4), two(4)]   # [chunk][block]: P in 16 bits, then dS (key owners); dS (query owners)
        if not self.KO:
            self.AUXD = two(16)     # the lane's Delta, 16 times
        self.FR = take(4 * self.NF)
        self.AUXL = take(8 if self.KO else 2)
        r += r & 1
        self.ROFF, self.TOFF = take(8), take(8)
        # a wave's direct loads of a tile bring rows 4 NW apart; from 16 rows on the swizzle repeats, and the rest is 4 KB
        # more for every 16 rows
        self.NVOFF = 2
        self.DVOFF = take(self.NVOFF)
        self.AOFF = take(1)
        if self.KO:
            self.AUXV, self.THRLO = take(1), take(1)
        self.THRHI = [take(1)] if self.KO else [take(1), take(1)]
        # temporaries of the clamped loads: key owners have no register left but the LSE' ones, which are idle then
        self.T = self.AUXL if self.KO else take(1)
        self.T2 = self.AUXL + 1
        self.NV = r
        assert r <= 256, r
        # SGPRs: inputs pinned by the asm constraints, the rest clobbered
        self.s_t1base, self.s_t2base, self.s_auxbase = 32, 34, 36
        self.s_c, self.s_ntiles, self.s_nw, self.s_jlo, self.s_jhi = 38, 39, 40, 41, 42
        self.s_tfull, self.s_strm1, self.s_tbeg, self.s_lds, self.s_ldsaux = 43, 44, 45, 46, 47
        self.s_own, self.s_j, self.s_tk = 48, 49, 50
        self.s_ptr1, self.s_ptr2, self.s_ptra = 52, 54, 56
        self.s_row, self.s_255, self.s_dyn, self.s_dyna = 58, 59, 60, 61
        self.s_far = 62             # (a pair) streamed tile plus 4 KB
        self.s_m0 = 64
        self.plan()

    # ------------------------------------------------------------ MFMA program
    def plan(self):
        r = lambda t: [("r", ks, t) for ks in range(self.KS)]
        c = lambda ch, st: [("c", ch, db, st) for db in range(self.DB)]
        if self.KO:
            self.groups = r(1) + c(0, 1) + c(1, 1) + r(0) + c(0, 0) + c(1, 0)
            self.s_done = 48        # slot in which S(j+1) is complete
        else:
            self.groups = r(1) + r(0) + c(0, 0) + c(1, 0)
            self.s_done = 32
        self.NM = 2 * len(self.groups)
        self.first_valu = self.s_done + 2
        self.bar = self.s_done - 16 - 2 * (self.PFD + 1)     # ahead of the first read of tile j+1
        self.dma = self.bar + 2
        assert self.bar >= 0 and len(self.groups) % self.NF == 0 and self.PFD < self.NF
        if self.KO:
            self.deal_key_owner()
        else:
            self.deal_query_owner()

    def frag_loads(self, grp, buf, b):
        """LDS reads of a group's A operand in body b (tile j lies in stage b)."""
        f = self.FR + 4 * buf
        if grp[0] == "r":
            _, ks, t = grp
            st = (b + 1) % self.NST if t == 0 else b
            return ["ds_read_b128 %s, v%d offset:%d" % (self.vr(f, 4), self.ROFF + ks, st * self.SB + t * self.TB)]
        _, ch, db, t = grp
        off = b * self.SB + t * self.TB + ch * 16 * self.ROWB
        return ["ds_read_b64_tr_b16 %s, v%d offset:%d" % (self.vr(f + 2 * h, 2), self.TOFF + 2 * db + h, off) for h in range(2)]

    def mfma_texts(self, grp, buf, b):
        f = self.vr(self.FR + 4 * buf, 4)
        out = []
        own = self.vr if self.KO else self.ar
        if grp[0] == "r":
            _, ks, t = grp
            for k in range(2):
                dst = (self.S[(b + 1) % 2] if t == 0 else self.DP)[k]
                start = "0"
                if t == 1:          # key owners: Delta lies in block A's accumulator, block B (first) starts from it as well
                    start = self.vr(self.DP[0] if self.KO else self.AUXD[k], 16)
                out.append("%s %s, %s, %s, %s" % (self.mfma, self.vr(dst, 16), f, own((self.B1 if t == 0 else self.B2)[k] + 4 * ks, 4),
                                                  start if ks == 0 else self.vr(dst, 16)))
            return out[::-1] if t == 1 and ks == 0 else out
        _, ch, db, t = grp
        for k in range(2):
            acc = self.ar(self.ACC + 128 * t + 64 * k + 16 * db, 16)
            out.append("%s %s, %s, %s, %s" % (self.mfma, acc, f, self.vr(self.P[ch][k], 4), acc))
        return out

    # ------------------------------------------------------------ VALU programs
    # An operation is (instruction, earliest slot, slot it has to precede) in slots of the iteration before (below NM) and
    # of iteration j itself (NM + slot).
    def fixed(self, s):
        """Issue cost of what slot s holds beside the VALU program."""
        s %= self.NM
        c = 1.0
        if s % 2 == 0:
            c += 1.0 if (s // 2) % self.W == 0 else 0.0
        else:
            c += len(self.frag_loads(self.groups[(s // 2 + self.PFD) % len(self.groups)], 0, 0))
        c += {self.bar: 2, self.dma: 6 * self.NLD + 2 + (3 if self.KO else 0), self.dma + 2: 8}.get(s, 0)
        c += {0: 2, self.first_valu - 1: 4 if self.KO else 2}.get(s, 0)
        return c + self.aux_slots.get(s, 0)

    PAIRS = [(k, r) for a in range(4) for k in range(2) for r in (4 * a, 4 * a + 2)]     # (block, first register of a pair)

    def p16(self, k, r):
        return self.P[r // 8][k] + (r % 8) // 2

    def deal_key_owner(self):
        NM, S, DP, w0 = self.NM, self.S[0], self.DP, self.first_valu
        far = 10 ** 6
        lse = lambda r: self.AUXL + 4 * ((r // 4) % 2) + r % 4
        def F(t):
            k, r = self.PAIRS[t]
            e = w0 if r < 8 else self.lse2 + 2 * (self.PFD + 1) + 1
            return [("v_fma_f32 v%d, v%d, s%d, -v%d" % (S[k] + r + i, S[k] + r + i, self.s_c, lse(r + i)), e, far) for i in range(2)]
        def E(t):
            k, r = self.PAIRS[t]
            return [("v_exp_f32 v%d, v%d" % (S[k] + r + i, S[k] + r + i), w0, far) for i in range(2)]
        def C(t):       # into the registers that dK's products of the tile before read dS from
            k, r = self.PAIRS[t]
            early, late = (NM - 7, NM + 16) if r < 8 else (NM + 2, NM + 24)
            return [("%s v%d, v%d, v%d" % (self.cvt, self.p16(k, r), S[k] + r, S[k] + r + 1), early, late)]
        def M(t):
            k, r = self.PAIRS[t]
            return [("v_mul_f32 v%d, v%d, v%d" % (DP[k] + r + i, S[k] + r + i, DP[k] + r + i), NM + 18, NM + 32) for i in range(2)]
        def X(t):       # into the registers that dV's products read P from
            k, r = self.PAIRS[t]
            early, late = (NM + 26, NM + 48) if r < 8 else (NM + 34, NM + 56)
            return [("%s v%d, v%d, v%d" % (self.cvt, self.p16(k, r), DP[k] + r, DP[k] + r + 1), early, late)]
        lag, split = 7, NM + 32
        def first_part():
            ops = []
            for t in range(-3, 16 + lag):      # (the first half's x early: their LSE' registers are needed again)
                f = [x for u in ((2 * t + 6, 2 * t + 7) if t < 1 else (t + 7,)) for x in F(u)] if t + 7 < 16 else []
                ops += f + (E(t) if 0 <= t < 16 else []) + (C(t - lag) if t >= lag else [])
            return ops + [x for t in range(16) for x in M(t)]
        # LSE' of the accumulator's first half before the VALU program begins, of the second into the same registers once
        # the first half's x are made
        self.lse1 = self.s_done - 6
        self.delta = NM - 2 * self.PFD - 3
        half = [o[0] for t in range(8) for o in self.at(F, t)]
        last, self.lse2 = None, w0
        while last is None or self.lse2 != last + 1:
            self.lse2 = w0 if last is None else last + 1
            self.aux_slots = {self.lse1: 2, self.delta: 4}
            self.aux_slots[self.lse2 % NM] = self.aux_slots.get(self.lse2 % NM, 0) + 2
            valu = deal(first_part(), self.fixed, w0, split - w0)
            last = max(s for s, ops in valu.items() if any(o in half for o in ops))
        valu.update(deal([x for t in range(16) for x in X(t)], self.fixed, split, NM + w0 - split))
        # Delta goes into block A's dP, the masks' constant into block B's, once nothing reads the old one any more
        reads = [o[0] for t in range(16) for o in X(t)]
        assert all(s < NM + min(self.delta, w0 - 1) for s, ops in valu.items() if any(o in reads for o in ops))
        assert all(s < NM + self.dma for s, ops in valu.items() if any(o.startswith("v_fma") for o in ops)) and self.dma < self.lse1
        self.valu = lambda b, s: valu[s]

    def at(self, make, t):
        self.lse2 = getattr(self, "lse2", 0)
        return make(t)

    def deal_query_owner(self):
        NM, DP, w0, far = self.NM, self.DP, self.first_valu, 10 ** 6
        self.aux_slots = {}
        pairs = self.PAIRS
        def program(S):
            def F(t):
                k, r = pairs[t]
                return [("v_fma_f32 v%d, v%d, s%d, -v%d" % (S[k] + r + i, S[k] + r + i, self.s_c, self.AUXL + k), w0, far) for i in range(2)]
            def E(t):
                k, r = pairs[t]
                return [("v_exp_f32 v%d, v%d" % (S[k] + r + i, S[k] + r + i), w0, NM + 32) for i in range(2)]
            def M(t):
                k, r = pairs[t]
                return [("v_mul_f32 v%d, v%d, v%d" % (DP[k] + r + i, S[k] + r + i, DP[k] + r + i), NM + 18, far) for i in range(2)]
            def X(t):
                k, r = pairs[t]
                return [("%s v%d, v%d, v%d" % (self.cvt, self.p16(k, r), DP[k] + r, DP[k] + r + 1), NM + 18, NM + (32 if r < 8 else 40))]
            ops = []
            for t in range(17):
                ops += (F(t) if t < 16 else []) + (E(t - 1) if t else [])
            for t in range(17):
                ops += (M(t) if t < 16 else []) + (X(t - 1) if t else [])
            return deal(ops, self.fixed, w0, NM)
        dealt = [program(self.S[0]), program(self.S[1])]
        # (a window slot below NM belongs to the tile of the next body)
        self.valu = lambda b, s: dealt[(b + (s < NM)) % 2].get(s, [])

    def body_valu(self, b):
        """{slot: [instructions]} of body b: the end of tile j's program, the beginning of tile j+1's."""
        return {s: self.valu(b, s if s >= self.first_valu else s + self.NM) for s in range(self.NM)}

    def lse_reads(self, half, stage):
        """Half of a tile's LSE' (rows 8a + 4g + 0..3, a = 2 half, 2 half + 1)."""
        return ["ds_read_b128 %s, v%d offset:%d" % (self.vr(self.AUXL + 4 * i, 4), self.AOFF, stage * 256 + 32 * (2 * half + i))
                for i in range(2)]

    def delta_reads(self, stage):
        """A tile's Delta into block A's dP accumulator."""
        return ["ds_read_b128 %s, v%d offset:%d" % (self.vr(self.DP[0] + 4 * a, 4), self.AOFF, stage * 256 + 128 + 32 * a)
                for a in range(4)]

    # ------------------------------------------------------------------- DMA
    def dma_fast(self, stage):
        out = []
        for far in range(self.NLD // self.NVOFF):
            for t, ptr in ((0, self.s_ptr1), (1, self.s_ptr2)):
                if far:
                    out += ["s_add_u32 s%d, s%d, 4096" % (self.s_far, ptr), "s_addc_u32 s%d, s%d, 0" % (self.s_far + 1, ptr + 1)]
                    ptr = self.s_far
                for k in range(self.NVOFF):
                    i = far * self.NVOFF + k
                    out += ["s_add_u32 m0, s%d, %d" % (self.s_lds, stage * self.SB + t * self.TB + i * self.NW * 1024),
                            "s_nop 0",
                            "global_load_lds_dwordx4 v%d, %s" % (self.DVOFF + k, self.sr(ptr, 2))]
        if self.KO:                 # 32 LSE' (lanes 0-31) and 32 Delta (lanes 32-63) values
            out += ["s_add_u32 m0, s%d, %d" % (self.s_ldsaux, stage * 256),
                    "s_nop 0",
                    "global_load_lds_dword v%d, %s" % (self.AUXV, self.sr(self.s_ptra, 2))]
        return out

    def dma_clamped(self, stage, second=False):
        """Tile s_tk with its rows clamped to the last one; stage None: its ring place is in s_dyn / s_dyna.  second: of the
        second tensor only."""
        e, T = self.e, self.T
        lds = (self.s_lds, self.s_ldsaux) if stage is not None else (self.s_dyn, self.s_dyna)
        at = stage or 0
        e("s_lshl_b32 s%d, s%d, 5" % (self.s_row, self.s_tk))
        e("s_mov_b32 s%d, 255" % self.s_255)
        for i in range(self.NLD):
            if i == self.NVOFF:
                e("s_add_i32 s%d, s%d, 16" % (self.s_row, self.s_row))
            e("v_lshrrev_b32 v%d, 8, v%d" % (T, self.DVOFF + i % self.NVOFF))      # an offset is 256 row + chunk
            e("v_add_u32 v%d, s%d, v%d" % (T, self.s_row, T))
            e("v_min_i32 v%d, s%d, v%d" % (T, self.s_strm1, T))
            e("v_lshlrev_b32 v%d, 8, v%d" % (T, T))
            e("v_and_or_b32 v%d, v%d, s%d, v%d" % (T, self.DVOFF + i % self.NVOFF, self.s_255, T))
            for t, base in ((0, self.s_t1base), (1, self.s_t2base))[1 if second else 0:]:
                e("s_add_u32 m0, s%d, %d" % (lds[0], at * self.SB + t * self.TB + i * self.NW * 1024))
                e("s_nop 0")
                e("global_load_lds_dwordx4 v%d, %s" % (T, self.sr(base, 2)))
        if self.KO and not second:
            if self.NLD > self.NVOFF:
                e("s_sub_i32 s%d, s%d, 16" % (self.s_row, self.s_row))
            e("v_mbcnt_lo_u32_b32 v%d, -1, 0" % self.T2)
            e("v_mbcnt_hi_u32_b32 v%d, -1, v%d" % (self.T2, self.T2))
            e("v_and_b32 v%d, 31, v%d" % (self.T2, self.T2))              # the row that this lane brings
            e("v_add_u32 v%d, s%d, v%d" % (T, self.s_row, self.T2))
            e("v_min_i32 v%d, s%d, v%d" % (T, self.s_strm1, T))
            e("v_sub_u32 v%d, v%d, v%d" % (T, T, self.T2))
            e("v_lshl_add_u32 v%d, v%d, 2, v%d" % (T, T, self.AUXV))
            e("s_add_u32 m0, s%d, %d" % (lds[1], at * 256))
            e("s_nop 0")
            e("global_load_lds_dword v%d, %s" % (T, self.sr(self.s_auxbase, 2)))

    # --------------------------------------------------------------- the loop
    def masks(self, tag):
        """Branches to the mask pre-passes on S of tile s_j."""
        L, out = self.lab, []
        if self.KO:
            out += ["s_cmp_lt_i32 s%d, s%d" % (self.s_j, self.s_jlo), "s_cbranch_scc1 %s" % L("MASKLO%s_" % tag),
                    "%s:" % L("MASKLORET%s_" % tag)]
        return out + ["s_cmp_ge_i32 s%d, s%d" % (self.s_j, self.s_jhi), "s_cbranch_scc1 %s" % L("MASKHI%s_" % tag),
                      "%s:" % L("MASKHIRET%s_" % tag)]

    def body(self, b):
        NST, L = self.NST, self.lab
        self.e("%s:" % L("BODY%d_" % b))
        self.e("s_cmp_ge_i32 s%d, s%d" % (self.s_j, self.s_nw if not self.KO else self.s_ntiles))
        self.e("s_cbranch_scc1 %s" % L("DONE_" if self.KO else "STANDBY_"))
        dst = (b + self.AHEAD) % NST
        extra = {}
        def add(slot, what):
            extra[slot] = extra.get(slot, []) + what
        add(self.bar, ["s_waitcnt vmcnt(%d)" % self.NGRP, "s_barrier"])
        fast = self.dma_fast(dst)
        add(self.dma, ["s_cmp_ge_i32 s%d, s%d" % (self.s_tk, self.s_tfull), "s_cbranch_scc1 %s" % L("SLOW%d_" % b)] + fast +
            ["%s:" % L("SLOWRET%d_" % b)])
        bump = []
        for ptr, n in ((self.s_ptr1, self.TB), (self.s_ptr2, self.TB)) + (((self.s_ptra, 128),) if self.KO else ()):
            bump += ["s_add_u32 s%d, s%d, %d" % (ptr, ptr, n), "s_addc_u32 s%d, s%d, 0" % (ptr + 1, ptr + 1)]
        add(self.dma + 2, bump + ["s_add_i32 s%d, s%d, 1" % (self.s_tk, self.s_tk), "s_add_i32 s%d, s%d, 1" % (self.s_j, self.s_j)])
        add(self.first_valu - 1, self.masks(str(b)))
        lds = {}
        if self.KO:
            nxt = (b + 1) % NST
            lds[self.lse1] = self.lse_reads(0, nxt)
            lds[self.delta] = self.delta_reads(nxt)
            lds[self.lse2 % self.NM] = self.lse_reads(1, nxt if self.lse2 < self.NM else b) + lds.get(self.lse2 % self.NM, [])
        nb = (b + 1) % NST
        self.stream(self.groups, lambda g, buf: self.mfma_texts(g, buf, b), lambda g, buf: self.frag_loads(g, buf, b), self.NF, self.PFD,
                    self.body_valu(b), extra, lambda i, buf: self.frag_loads(self.groups[i], buf, nb), lds_by_slot=lds, wait_every=self.W)
        if b == NST - 1:
            self.e("s_branch %s" % L("BODY0_"))

    def pre(self, b):
        """The first tile of a wave, in stage b: S, and the part of its VALU program that stands in the iteration before."""
        e, L = self.e, self.lab
        before = (b + self.NST - 1) % self.NST
        e("%s:" % L("PRE%d_" % b))
        self.outstanding = []
        lds = {0: self.lse_reads(0, b) + self.delta_reads(b)} if self.KO else {}
        self.stream([g for g in self.groups if g[0] == "r" and g[2] == 0], lambda g, buf: self.mfma_texts(g, buf, before),
                    lambda g, buf: self.frag_loads(g, buf, before), self.NF, self.PFD, {}, {},
                    lambda i, buf: self.frag_loads(self.groups[i], buf, b), prefetched=0, lds_by_slot=lds)
        e("s_nop 15")
        for ins in self.masks("P%d" % b):
            e(ins)
        valu = self.body_valu(before)
        for s in range(self.first_valu, self.NM):
            if self.KO and s == self.lse2:
                for ins in self.lse_reads(1, b):
                    e(ins)
                e("s_waitcnt lgkmcnt(0)")
            for ins in valu.get(s, []):
                e(ins)
        e("s_branch %s" % L("BODY%d_" % b))

    def mask_passes(self, tag, parity):
        """Elements of S that are masked become -inf, so that p = 0 and ds = 0.  Element r of a lane is streamed row
        32 (t_begin + j) + 8 (r / 4) + 4 g + r % 4; block B's owners are 32 rows further than block A's."""
        e, L = self.e, self.lab
        for kind in ("LO", "HI") if self.KO else ("HI",):
            e("%s:" % L("MASK%s%s_" % (kind, tag)))
            e("s_nop 15")
            e("s_lshl_b32 s%d, s%d, 5" % (self.s_row, self.s_j))
            neg = self.DP[1] if self.KO else self.T      # (key owners: nothing reads the old dP any more)
            e("v_mov_b32 v%d, 0xff800000" % neg)
            for k in range(2):
                for r in range(16):
                    const = 8 * (r >> 2) + (r & 3) - (32 * k if kind == "LO" else 0)
                    e("s_add_i32 s%d, s%d, %d" % (self.s_255, self.s_row, const))
                    e("%s vcc, s%d, v%d" % (("v_cmp_ge_i32", self.s_255, self.THRLO) if kind == "LO" else
                                            ("v_cmp_le_i32", self.s_255, self.THRHI[k if not self.KO else 0])))
                    v = self.S[parity][k] + r
                    e("v_cndmask_b32 v%d, v%d, v%d, vcc" % (v, neg, v))
            e("s_branch %s" % L("MASK%sRET%s_" % (kind, tag)))

    def standby(self, limit):
        """Iterations s_j .. limit - 1 of a wave that has nothing to compute in them: the barrier, its share of the loads."""
        e, L = self.e, self.lab
        e("%s:" % L("STANDBY_"))
        e("s_cmp_ge_i32 s%d, s%d" % (self.s_j, limit))
        e("s_cbranch_scc1 %s" % L("STANDBYEND_"))
        e("s_waitcnt vmcnt(%d)" % self.NGRP)
        e("s_barrier")
        e("s_add_i32 s%d, s%d, %d" % (self.s_dyn, self.s_j, self.AHEAD))
        e("s_and_b32 s%d, s%d, %d" % (self.s_dyn, self.s_dyn, self.NST - 1))
        e("s_lshl_b32 s%d, s%d, 8" % (self.s_dyna, self.s_dyn))
        e("s_add_u32 s%d, s%d, s%d" % (self.s_dyna, self.s_dyna, self.s_ldsaux))
        e("s_lshl_b32 s%d, s%d, 14" % (self.s_dyn, self.s_dyn))
        e("s_add_u32 s%d, s%d, s%d" % (self.s_dyn, self.s_dyn, self.s_lds))
        self.dma_clamped(None)
        e("s_add_i32 s%d, s%d, 1" % (self.s_tk, self.s_tk))
        e("s_add_i32 s%d, s%d, 1" % (self.s_j, self.s_j))
        e("s_branch %s" % L("STANDBY_"))
        e("%s:" % L("STANDBYEND_"))

    def start_pointers(self):
        e = self.e
        for ptr, base, sh in ((self.s_ptr1, self.s_t1base, 13), (self.s_ptr2, self.s_t2base, 13)) + (
                ((self.s_ptra, self.s_auxbase, 7),) if self.KO else ()):
            e("s_lshl_b32 s%d, s%d, %d" % (self.s_row, self.s_tk, sh))
            e("s_add_u32 s%d, s%d, s%d" % (ptr, base, self.s_row))
            e("s_addc_u32 s%d, s%d, 0" % (ptr + 1, base + 1))

    def operands(self):
        """The owner rows, which direct loads bring to LDS, into registers, the second tensor's negated: dP starts from Delta and
        becomes t = Delta - dP.  The accumulators are cleared while those loads are on their way."""
        e, T = self.e, self.FR
        for i in range(256 if self.KO else 128):
            e("v_accvgpr_write_b32 a%d, 0" % (self.ACC + i))
        e("s_waitcnt vmcnt(0)")
        e("s_barrier")                       # every wave's part of tile 0 is in LDS
        e("s_mov_b32 s%d, 0x80008000" % self.s_dyn)
        own = self.vr if self.KO else self.ar
        raw = self.B2 if self.KO else self.S[0][0]      # (query owners: 64 registers that nothing lives in yet)
        raw = [raw[0], raw[1]] if self.KO else [raw, raw + 32]
        for ks in range(self.KS):
            t = T + ks                       # (address registers of their own: a read may still be on its way)
            e("v_add_u32 v%d, s%d, v%d" % (t, self.s_own, self.ROFF + ks))
            for k in range(2):
                e("ds_read_b128 %s, v%d offset:%d" % (own(self.B1[k] + 4 * ks, 4), t, 32 * self.ROWB * k))
                e("ds_read_b128 %s, v%d offset:%d" % (self.vr(raw[k] + 4 * ks, 4), t, 64 * self.ROWB + 32 * self.ROWB * k))
        if not self.KO:
            for k in range(2):
                e("ds_read_b32 v%d, v%d offset:%d" % (self.AUXL + k, self.AOFF, 256 * k))
                e("ds_read_b32 v%d, v%d offset:%d" % (self.AUXD[k], self.AOFF, 256 * k + 128))
        e("s_waitcnt lgkmcnt(0)")
        e("s_barrier")                       # every wave has its rows in registers: stages 1 to 3 are free
        if self.NW < 4:                      # ... and the second half of stage 0, which 160 KB have no room for besides
            e("s_mov_b32 s%d, s%d" % (self.s_tk, self.s_tbeg))
            self.dma_clamped(0, second=True)
        e("s_add_i32 s%d, s%d, 1" % (self.s_tk, self.s_tbeg))
        for k in range(2):
            for i in range(32):
                e("v_xor_b32 v%d, s%d, v%d" % (raw[k] + i, self.s_dyn, raw[k] + i))
        if not self.KO:
            for k in range(2):
                for i in range(32):
                    e("v_accvgpr_write_b32 a%d, v%d" % (self.B2[k] + i, raw[k] + i))
                for i in range(1, 16):
                    e("v_mov_b32 v%d, v%d" % (self.AUXD[k] + i, self.AUXD[k]))
        for stage in range(1, self.AHEAD):
            self.dma_clamped(stage)
            e("s_add_i32 s%d, s%d, 1" % (self.s_tk, self.s_tk))
        if self.NW < 4:
            e("s_waitcnt vmcnt(%d)" % (2 * self.NGRP))
            e("s_barrier")                   # all of tile 0 is in LDS

    def generate(self):
        L, e = self.lab, self.e
        e("s_waitcnt lgkmcnt(0)")
        self.save_m0(self.s_m0)
        self.operands()
        e("s_mov_b32 s%d, 0" % self.s_j)
        entries = (0, 2) if self.KO else (0,)
        if self.KO:
            self.standby(self.s_nw)          # (s_nw: the wave's first tile, an even number, or the number of tiles)
            e("s_cmp_ge_i32 s%d, s%d" % (self.s_j, self.s_ntiles))
            e("s_cbranch_scc1 %s" % L("DONE_"))
            self.start_pointers()
            e("s_and_b32 s%d, s%d, %d" % (self.s_row, self.s_j, self.NST - 1))
            e("s_cmp_ge_i32 s%d, 2" % self.s_row)
            e("s_cbranch_scc1 %s" % L("PRE2_"))
        else:                                # (s_nw: the number of tiles that the wave computes)
            e("s_cmp_ge_i32 s%d, s%d" % (self.s_j, self.s_nw))
            e("s_cbranch_scc1 %s" % L("STANDBY_"))
            self.start_pointers()
        for b in entries:
            self.pre(b)
        canonical = [i for i in range(self.PFD) for _ in self.frag_loads(self.groups[i], 0, 0)]
        assert self.outstanding == canonical
        for b in range(self.NST):
            self.body(b)
            assert self.outstanding == canonical
        for b in range(self.NST):
            self.mask_passes(str(b), (b + 1) % 2)
            e("%s:" % L("SLOW%d_" % b))
            self.dma_clamped((b + self.AHEAD) % self.NST)
            e("s_branch %s" % L("SLOWRET%d_" % b))
        for b in entries:
            self.mask_passes("P%d" % b, b % 2)
        if not self.KO:
            self.standby(self.s_ntiles)
        e("%s:" % L("DONE_"))
        e("s_waitcnt vmcnt(0) lgkmcnt(0)")
        self.restore_m0(self.s_m0)
        e("s_nop 15")
        e("s_nop 7")

    # ----------------------------------------------------------- C++ wrapper
    def emit_inc(self):
        self.generate()
        out = ["// Generated by gen_attn_bwd_wide_loop.py %s %d %s -- do not edit.  Main loop of bwd_wide_sweep<%d, *, %s, %s>."
               % ("kv" if self.KO else "q", self.NW, self.dtype, self.NW, "true" if self.KO else "false", "true" if self.dtype == "f16" else "false"),
               "// VGPRs used: %d, AGPRs used: %d.  MFMA slots per iteration: %d." % (self.NV, self.NA, self.NM),
               "asm volatile("]
        out += ['    "%s\\n\\t"' % ln for ln in self.lines]
        outs, ins, pinned = [], [], set()
        for i in range(16 if self.KO else 8):
            outs.append('"={%s}"(acc[%d])' % (self.ar(self.ACC + 16 * i, 16), i))
        def vin(base, n, name):
            ins.append('"{%s}"(%s)' % (self.vr(base, n), name))
            pinned.update(range(base, base + n))
        vin(self.ROFF, 8, "roff_v")
        vin(self.TOFF, 8, "toff_v")
        vin(self.DVOFF, self.NVOFF, "dma_voff_v")
        vin(self.AOFF, 1, "aux_off")
        if self.KO:
            vin(self.AUXV, 1, "aux_voff")
            vin(self.THRLO, 1, "thr_lo_base")
        for k, reg in enumerate(self.THRHI):
            vin(reg, 1, "thr_hi_base[%d]" % k)
        for base, n, name in ((self.s_t1base, 2, "t1_head"), (self.s_t2base, 2, "t2_head"), (self.s_auxbase, 2, "aux_head"),
                              (self.s_c, 1, "c_log2e"), (self.s_ntiles, 1, "n_tiles"), (self.s_nw, 1, "n_wave"), (self.s_jhi, 1, "j_hi"),
                              (self.s_tfull, 1, "t_full"), (self.s_strm1, 1, "str_m1"), (self.s_tbeg, 1, "t_begin"),
                              (self.s_lds, 1, "lds_wave"), (self.s_ldsaux, 1, "lds_aux"), (self.s_own, 1, "own_off")) + (
                              ((self.s_jlo, 1, "j_lo"),) if self.KO else ()):
            ins.append('"{%s}"(%s)' % (self.sr(base, n), name))
        clob = ['"memory"', '"vcc"', '"scc"'] + ['"v%d"' % i for i in range(self.NV) if i not in pinned]
        clob += ['"a%d"' % i for i in range(128, 256)] if not self.KO else []
        clob += ['"s%d"' % i for i in range(self.s_j, self.s_m0 + 1)]
        out += ["    : " + ", ".join(outs), "    : " + ", ".join(ins), "    : " + ", ".join(clob) + ");"]
        return "\n".join(out) + "\n"


if __name__ == "__main__":
    # --nf / --pfd / --w: fragment buffers, groups read ahead, groups per wait; a library build passes none of them
    args, opts = sys.argv[1:], {}
    while len(args) > 3 and args[-2] in ("--nf", "--pfd", "--w"):
        opts[args[-2]] = int(args[-1])
        args = args[:-2]
    text = WideGen(args[0] == "kv", dtype=args[3] if len(args) > 3 else "bf16", NW=int(args[1]), NF=opts.get("--nf"), PFD=opts.get("--pfd"),
                   W=opts.get("--w")).emit_inc()
    with open(args[2], "w") as f:
        f.write(text)
