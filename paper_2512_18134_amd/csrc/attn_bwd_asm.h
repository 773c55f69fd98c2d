// attn_bwd_asm.h -- attention-backward sweeps whose main loop is hand scheduled (one wave per SIMD at D = 128, two at
// D = 64).
//
// Same mathematics and data layout as attn_bwd_sweep_kernel (attn_bwd_kernels.h): a workgroup of four
// waves owns 128 keys (KEY_OWNER) or 128 queries and streams the other side; the owner index is the
// MFMA column = the lane.  The steady-state loop -- the three-stage modulo schedule described in
// gen_attn_bwd_loop.py -- is one inline-asm statement generated by that script, with the accumulators
// and the owner's rows in AGPRs at D = 128.  This file does what surrounds the loop: work decomposition,
// addressing, the start of the stream, S(0)/dP(0), and the epilogue.
//
// Streamed tiles of 32 rows in two 6-stage LDS rings (2 * 6 * 32 * D * 2 bytes) plus a ring of
// 32 LSE' + 32 Delta values per tile (key-owner sweep).  LSE' = LSE * log2(e) and Delta come from
// attn_bwd_delta_kernel through the workspace: ws[0 .. n) = LSE', ws[n .. 2n) = Delta, n = B*H*S_q.
// Requires scale > 0 (masked scores are set to -inf before the multiply by scale*log2e).
//
// Workgroups are persistent, like the forward kernels': a launch has as many workgroups as the chip holds at
// once and each walks the queue of owner tiles of its XCD.  One launch holds both sweeps: the queue is all key-owner
// tiles, then all query-owner tiles (BwdQueue); or one of them, the other count being zero (sweeps_apart in attn_bwd.hip).
#pragma once
#include "attn_bwd_kernels.h"  // BwdParams
#include "attn_common.h"
#include "attn_fwd_asm.h"   // U32Vec
#include "attn_dma.h"       // dma16, wait_vmcnt

namespace attn {

// The queue of a launch: entries [0, n_kv) are key-owner tiles (four products per streamed tile against three, so they go
// first), entries [q_first, q_first + n_q) query-owner tiles; q_first is n_kv rounded up to a multiple of the
// XCD count, so that entry e belongs to XCD e % 8 in both halves.  Entries in between stand for nothing.
struct BwdQueue {
    int n_kv, q_first, n_entries;
    __host__ __device__ BwdQueue(int kv, int q)
        : n_kv(kv), q_first((kv + kNumXcd - 1) / kNumXcd * kNumXcd), n_entries(q ? q_first + q : kv)
    {
    }
    // The entry that workgroup `wg` of a launch of n_slots (a multiple of the XCD count, or >= n_entries) takes up in
    // pass k, or -1.  A pass goes through one entry per workgroup of the XCD, odd passes in reverse, so that a
    // workgroup pairs heavy with light tiles.  Workgroup m of an XCD runs on its compute unit m % cus, also where a unit
    // holds two (measured): the first `cus` of them take their part of a pass in reverse, so that the two on a unit
    // pair heavy with light as well, and the units with the lightest tiles are the ones that a second workgroup joins
    // where there are not enough entries for all.  Entries rise from pass to pass.
    __host__ __device__ int entry(int wg, int n_slots, int cus, int k) const
    {
        const int xcd = wg % kNumXcd, m = wg / kNumXcd;
        const int n_x = (n_entries - xcd + kNumXcd - 1) / kNumXcd;   // queue length of this XCD
        const bool single = n_slots >= n_entries;                    // one entry per workgroup, one pass
        const int per_pass = single ? n_x : n_slots / kNumXcd;
        if (single && (k > 0 || m >= n_x))
            return -1;
        const int first = per_pass < cus ? per_pass : cus;
        const int at = m < first ? first - 1 - m : m;
        const int idx = k * per_pass + (k & 1 ? per_pass - 1 - at : at);
        return idx < n_x ? idx * kNumXcd + xcd : -1;
    }
};

// Which workgroup of an XCD takes up which entries of its queue, for launches of several passes: the host deals the tiles out
// so that the workgroups' walks end together (plan_walks in attn_bwd.hip).  Workgroup m takes up entries idx(first(m)) to
// idx(first(m + 1) - 1) of its XCD's queue, in rising order.  The plan is XCD 0's, whose queue is the longest.
struct BwdPlan {
    static constexpr int kMaxSlots = 64, kMaxEntries = 768;   // per XCD
    // (two 16-bit numbers to a word, which a scalar load can bring)
    uint32_t first[(kMaxSlots + 2) / 2], idx[kMaxEntries / 2];
    static __host__ __device__ int get(const uint32_t *words, int i) { return (int)(words[i >> 1] >> (i & 1) * 16 & 0xffffu); }
    static void set(uint32_t *words, int i, int x)
    {
        words[i >> 1] = (words[i >> 1] & ~(0xffffu << (i & 1) * 16)) | (uint32_t)x << (i & 1) * 16;
    }
};

// The entry that workgroup `wg` takes up in pass k, or -1.  (Kernels of their own for launches with a plan: asking which it is cost
// launches of 10 to 20 us 0.2 to 0.5 us, code that is fetched for the first time)
template <bool PLANNED>
__device__ __forceinline__ int queue_entry(const BwdQueue &queue, const BwdParams &p, const BwdPlan &plan, int wg, int n_slots, int k)
{
    if constexpr (!PLANNED)
        return queue.entry(wg, n_slots, p.cus_per_xcd, k);
    const int m = wg / kNumXcd, at = BwdPlan::get(plan.first, m) + k;
    if (at >= BwdPlan::get(plan.first, m + 1))
        return -1;
    const int entry = BwdPlan::get(plan.idx, at) * kNumXcd + wg % kNumXcd;
    return entry < queue.n_entries ? entry : -1;   // (only the last entry of XCD 0's queue has no counterpart)
}

// LDS of a workgroup: the two rings, the LSE' / Delta ring, and what the waves' owner rows need beyond stage 4 of the rings
// (which no streamed tile occupies before the loop runs)
template <int D>
struct BwdLds {
    static constexpr int NST = 6, TB = 32 * D * 2;
    static constexpr int RING1 = 0, RING2 = NST * TB, AUX = 2 * NST * TB, OWN = AUX + NST * 256, BYTES = OWN + 6 * TB;
};

// One sweep's part of the workgroup's walk: takes up entries from pass `pass` on for as long as they are this sweep's.
// F16: q, k, v, d_o and the gradients are IEEE fp16 instead of bf16 (the element type of the paper's
// Section 6.3 figures); the pointers in BwdParams are then reinterpreted.
template <int D, bool CAUSAL, bool KEY_OWNER, bool F16, bool PLANNED>
__device__ __forceinline__ void bwd_sweep(const BwdParams &p, const BwdPlan &plan, const BwdQueue &queue, const int wave, int &pass)
{
    static_assert(D == 128 || D == 64, "hand-scheduled backward sweeps: D = 64 or 128");
    typedef typename std::conditional<F16, ElemF16, ElemBF16>::type E;
    typedef typename E::t elem_t;
    typedef typename E::x8 ex8;
    constexpr int BN = 32, NW = 4, BO = NW * 32, NST = 6;
    constexpr int CPR = D / 8;
    constexpr int KS = D / 16;
    constexpr int DB = D / 32;
    constexpr int ROWB = D * 2;
    constexpr int TB = BN * ROWB;
    constexpr int NLD = TB / (NW * 1024);
    constexpr int NSET = KEY_OWNER ? 2 : 1;
    // Streamed tiles that go out ahead of S(0).  D = 128: two, the next two behind its products: the address unit takes 64
    // bytes a cycle, 0.25 us for those two (16 heads of 128 rows 12.2 -> 12.0 us, of 512 19.9 -> 19.7, of 1024 37.0 -> 36.7);
    // D = 64, half as many bytes: all four (two: 200 heads of 300 rows, causal, 30.1 -> 30.6)
    constexpr int FIRST = D == 128 ? 2 : 4;
    constexpr int NGRP = 2 * NLD + (KEY_OWNER ? 1 : 0);   // direct loads per wave and streamed tile
    constexpr int NBP = 4 * KS / 16;  // owner fragments packed 16 dwords at a time

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    typedef BwdLds<D> Lds;
    static_assert(Lds::NST == NST && Lds::TB == TB, "one layout");
    constexpr uint32_t RING1 = Lds::RING1, RING2 = Lds::RING2, AUX = Lds::AUX;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(ATTN_LDS_PTR(unsigned char))smem;

    // (the lane number is asked from the hardware again in either sweep, at D = 64 in the epilogue too: no address made
    // from it is kept in registers across a loop)
    auto lane_id = []() -> int {
        int ones = -1;
        asm volatile("" : "+s"(ones));
        return __builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0));
    };
    const int lane = lane_id();
    const int lq = lane & 31;
    const int g = lane >> 5;

    // ---- direct-load addressing
    typename U32Vec<NLD>::type dma_row_v, dma_voff_v;
    uint32_t dma_row[NLD], dma_voff[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int gi = i * NW + wave;
        dma_row[i] = (1024 / ROWB) * gi + lane / CPR;
        dma_voff[i] = dma_row[i] * ROWB + (uint32_t)(((lane % CPR) ^ swz<D>(dma_row[i])) * 16);
        U32Vec<NLD>::set(dma_row_v, i, dma_row[i]);
        U32Vec<NLD>::set(dma_voff_v, i, dma_voff[i]);
    }
    const uint32_t lds_1_wave = lds0 + RING1 + wave * 1024;
    const uint32_t lds_2_wave = lds0 + RING2 + wave * 1024;
    const uint32_t lds_aux = lds0 + AUX;
    const uint32_t aux_row = (uint32_t)lq;
    const uint32_t aux_sel = g ? (uint32_t)(p.n_rows * 4) : 0u;
    auto issue_tile = [&](const elem_t *t1_head, const elem_t *t2_head, const float *aux_head, int S_str, int stage,
                          int t) {  // t: absolute tile index of the streamed tensor
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int r = min(t * BN + (int)dma_row[i], S_str - 1);
            const uint32_t voff = dma_voff[i] + (uint32_t)(r - (int)dma_row[i]) * ROWB;
            dma16(lds_1_wave + stage * TB + i * NW * 1024, t1_head, voff);
            dma16(lds_2_wave + stage * TB + i * NW * 1024, t2_head, voff);
        }
        if (KEY_OWNER) {
            const int r = min(t * BN + lq, p.S_q - 1);
            dma4(lds_aux + stage * 256, aux_head, (uint32_t)r * 4 + aux_sel);
        }
    };

    // This wave's 32 owner rows of both tensors, laid out like a streamed tile.  Whole rows by direct loads: straight into MFMA
    // operand registers they would be 32-byte pieces of 32 rows per load, four times the address unit's work
    const uint32_t own_1 = lds0 + (wave == 0 ? RING1 + 4 * TB : (uint32_t)Lds::OWN + (wave - 1) * TB);
    const uint32_t own_2 = lds0 + (wave == 0 ? RING2 + 4 * TB : (uint32_t)Lds::OWN + (wave + 2) * TB);
    auto issue_own = [&](const elem_t *x1, const elem_t *x2, const float *aux_head, int row0, int last) {
        const int ln = lane_id();
#pragma unroll
        for (int i = 0; i < TB / 1024; ++i) {
            const int r = (1024 / ROWB) * i + ln / CPR;
            const uint32_t voff = (uint32_t)min(row0 + r, last) * ROWB + (uint32_t)(((ln % CPR) ^ swz<D>(r)) * 16);
            dma16(own_1 + i * 1024, x1, voff);
            dma16(own_2 + i * 1024, x2, voff);
        }
        if (!KEY_OWNER)   // LSE' and Delta of the rows, where key owners keep those of the streamed tiles
            dma4(lds_aux + wave * 256, aux_head, (uint32_t)min(row0 + (ln & 31), last) * 4 + (ln >> 5 ? (uint32_t)(p.n_rows * 4) : 0u));
    };

    // ---- operand addressing inside a tile
    uint32_t roff[KS];
    typename U32Vec<KS>::type roff1_v, roff2_v;
    {
        const int sw = swz<D>(lq);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            roff[ks] = lds0 + RING1 + (uint32_t)(lq * ROWB + (((2 * ks + g) ^ sw) * 16));
            roff1_v[ks] = roff[ks];
            roff2_v[ks] = roff[ks] + (RING2 - RING1);
        }
    }
    typename U32Vec<2 * DB>::type toff1_v, toff2_v;
    {
        const int i16 = lane & 15, dh = (lane >> 4) & 1;
        const int rho = i16 >> 2, pi = i16 & 3;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int hlf = 0; hlf < 2; ++hlf) {
                const int row = 4 * g + 8 * hlf + rho;
                const int ch = 4 * db + 2 * dh + (pi >> 1);
                toff1_v[2 * db + hlf] = lds0 + RING1 + (uint32_t)(row * ROWB + ((ch ^ swz<D>(row)) * 16) + (pi & 1) * 8);
                toff2_v[2 * db + hlf] = toff1_v[2 * db + hlf] + (RING2 - RING1);
            }
    }
    const uint32_t aux_off = lds_aux + 16 * g;

    const int n_t = KEY_OWNER ? p.n_t : p.n_tq, total = KEY_OWNER ? p.total_wg : p.total_q;
    auto el = [](const bf16_t *ptr) { return reinterpret_cast<const elem_t *>(ptr); };
    auto locate = [&](int entry, int &bh, int &ot) {
        // a head's sweeps stream Q, dO, K and V between them
        wg_to_tile_n<CAUSAL>(KEY_OWNER ? entry : entry - queue.q_first, total, n_t, 4ll * (p.S_q + p.S_kv) * D, bh, ot);
        if (CAUSAL && KEY_OWNER)
            ot = n_t - 1 - ot;  // early key tiles stream the most queries: heaviest first
    };
    auto issue_own_of = [&](int bh, int ot) {
        const size_t q_head = (size_t)bh * p.S_q * D, k_head = (size_t)bh * p.S_kv * D;
        issue_own(KEY_OWNER ? el(p.k) + k_head : el(p.q) + q_head, KEY_OWNER ? el(p.v) + k_head : el(p.d_o) + q_head,
                  p.lse2 + (size_t)bh * p.S_q, ot * BO + wave * 32, (KEY_OWNER ? p.S_kv : p.S_q) - 1);
    };
    int bh = 0, ot = 0;
    bool own_on_its_way = false;   // the tile's owner rows, and `bh`, `ot` are this tile's
#pragma clang loop unroll(disable)
    for (;; ++pass) {
        const int entry = queue_entry<PLANNED>(queue, p, plan, blockIdx.x, (int)gridDim.x, pass);
        if (entry < 0 || (KEY_OWNER && entry >= queue.n_kv))
            break;   // (entries rise from pass to pass; only the last pass can be short)
        if (!KEY_OWNER && entry < queue.q_first)
            continue;
        if (pass > 0)
            __syncthreads();  // every wave has read the previous tile's staged gradients back: the rings are free
        if (__builtin_expect(!own_on_its_way, 1))
            locate(entry, bh, ot);
        const int S_own = KEY_OWNER ? p.S_kv : p.S_q;
        const int S_str = KEY_OWNER ? p.S_q : p.S_kv;
        const int o0 = ot * BO;
        const int o0w = o0 + wave * 32;
        const int p_lane = lane_id();   // (no lane number is kept in registers across a loop)
        const int own = o0w + (p_lane & 31);

        const size_t q_head = (size_t)bh * p.S_q * D, k_head = (size_t)bh * p.S_kv * D;
        const elem_t *t1_head = KEY_OWNER ? el(p.q) + q_head : el(p.k) + k_head;
        const elem_t *t2_head = KEY_OWNER ? el(p.d_o) + q_head : el(p.v) + k_head;
        const float *aux_head = p.lse2 + (size_t)bh * p.S_q;  // LSE' rows of this head; Delta is n_rows floats further

        // ---- streamed tile range (tiles of 32 rows, absolute indices)
        int t_begin = 0, t_end;
        if (KEY_OWNER) {
            t_end = (p.S_q + BN - 1) / BN;
            if (CAUSAL)
                t_begin = min(o0 / BN, t_end);
        } else {
            int kv_end = p.S_kv;
            if (CAUSAL)
                kv_end = min(kv_end, min(o0 + BO, p.S_q));
            t_end = (kv_end + BN - 1) / BN;
        }
        const int n_tiles = t_end - t_begin;
        const int t_full = S_str / BN;
        const int str_m1 = S_str - 1;
        // tiles j < j_lo touch the causal diagonal from below (key-owner), tiles j >= j_hi touch the ragged
        // end of the streamed tensor or the diagonal from above (query-owner)
        [[maybe_unused]] const int j_lo = CAUSAL ? o0w / BN - t_begin + 1 : 0;
        int j_hi = t_full - t_begin;
        if (!KEY_OWNER && CAUSAL)
            j_hi = min(j_hi, o0w / BN);

        // ---- prologue: the owner rows and tile 0, which S(0) and dP(0) wait for, then the other tiles; zeros for "tile -1",
        // which the first iteration's contraction reads (and multiplies by zeros).  (Owner rows straight into registers, a
        // copy of tile 0 for the zeros and a wait for everything before S(0): 16 heads of 515 rows, D = 64, causal 16.6 -> 15.5
        // us, 200 of 300 rows 32.4 -> 30.0, 16 of 128 rows, D = 128, 13.1 -> 12.4, 128 of 4096 rows 3131 -> 3113; the same bits.)
        if (__builtin_expect(!own_on_its_way, 1))
            issue_own_of(bh, ot);
    #pragma unroll
        for (int t = 0; t < FIRST; ++t)
            issue_tile(t1_head, t2_head, aux_head, S_str, t, t_begin + t);
    #pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const u32x4 zero = {0u, 0u, 0u, 0u};
            const uint32_t at = (NST - 1) * TB + (i * NW + wave) * 1024 + p_lane * 16;
            *(ATTN_LDS_PTR(u32x4))(uintptr_t)(lds0 + RING1 + at) = zero;
            if (KEY_OWNER)
                *(ATTN_LDS_PTR(u32x4))(uintptr_t)(lds0 + RING2 + at) = zero;
        }
        wait_vmcnt<(FIRST - 1) * NGRP>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();   // every wave's part of tile 0 and of the zeros is in LDS
        asm volatile("" ::: "memory");

        // (sums that the compiler cannot take out of the tile loop, where they would cost registers)
        uint32_t from_1 = own_1 - (lds0 + RING1), from_2 = own_2 - (lds0 + RING1);
        asm volatile("" : "+s"(from_1), "+s"(from_2));
        ex8 b1[KS], b2[KS];
    #pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            b1[ks] = *(ATTN_LDS_PTR(const ex8))(uintptr_t)(roff[ks] + from_1);
            b2[ks] = *(ATTN_LDS_PTR(const ex8))(uintptr_t)(roff[ks] + from_2);
        }
        // the second operand is negated and dP starts from Delta: the MFMAs deliver t = Delta - dP (gen_attn_bwd_loop.py)
    #pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            b2[ks] = __builtin_bit_cast(ex8, __builtin_bit_cast(u32x4, b2[ks]) ^ 0x80008000u);
        f32x16 acc[NSET * DB];
    #pragma unroll
        for (int i = 0; i < NSET * DB; ++i)
    #pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][r] = 0.f;

        // LSE' and Delta of tile 0 (key-owner: 16 rows per lane; query-owner: this lane's query)
        typename std::conditional<KEY_OWNER, f32x16, float>::type aux_l;
        f32x16 aux_d;
        if constexpr (KEY_OWNER) {
    #pragma unroll
            for (int a = 0; a < 4; ++a) {
                const f32x4 l4 = *(ATTN_LDS_PTR(const f32x4))(uintptr_t)(aux_off + 32 * a);
                const f32x4 d4 = *(ATTN_LDS_PTR(const f32x4))(uintptr_t)(aux_off + 128 + 32 * a);
    #pragma unroll
                for (int i = 0; i < 4; ++i) {
                    aux_l[4 * a + i] = l4[i];
                    aux_d[4 * a + i] = d4[i];
                }
            }
        } else {
            const uint32_t at = lds_aux + wave * 256 + (p_lane & 31) * 4;
            aux_l = *(ATTN_LDS_PTR(const float))(uintptr_t)at;
            const float delta = *(ATTN_LDS_PTR(const float))(uintptr_t)(at + 128);
    #pragma unroll
            for (int r = 0; r < 16; ++r)
                aux_d[r] = delta;
        }

        // S(0) and t(0)
        f32x16 s_init, dp_init = aux_d;
    #pragma unroll
        for (int r = 0; r < 16; ++r)
            s_init[r] = 0.f;
    #pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const ex8 a1 = *(ATTN_LDS_PTR(const ex8))(uintptr_t)(roff[ks]);
            const ex8 a2 = *(ATTN_LDS_PTR(const ex8))(uintptr_t)(roff[ks] + (RING2 - RING1));
            s_init = E::mfma(a1, b1[ks], s_init);
            dp_init = E::mfma(a2, b2[ks], dp_init);
        }

    #pragma unroll
        for (int t = FIRST; t < 4; ++t)
            issue_tile(t1_head, t2_head, aux_head, S_str, t, t_begin + t);
        typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
        u32x16 b1_pack[NBP], b2_pack[NBP];
    #pragma unroll
        for (int i = 0; i < NBP; ++i) {
            struct Four {
                ex8 a[4];
            } f1 = {{b1[4 * i], b1[4 * i + 1], b1[4 * i + 2], b1[4 * i + 3]}},
              f2 = {{b2[4 * i], b2[4 * i + 1], b2[4 * i + 2], b2[4 * i + 3]}};
            b1_pack[i] = __builtin_bit_cast(u32x16, f1);
            b2_pack[i] = __builtin_bit_cast(u32x16, f2);
        }
        // mask thresholds of this lane, minus the lane-group part of the accumulator row and the first tile
        [[maybe_unused]] const uint32_t thr_lo_base =   // (the key owners' mask from below)
            (uint32_t)(own - 4 * (p_lane >> 5) - BN * t_begin);
        const uint32_t thr_hi_base =
            (uint32_t)((KEY_OWNER ? str_m1 : (CAUSAL ? min(own, str_m1) : str_m1)) - 4 * (p_lane >> 5) - BN * t_begin);
        const float c_log2e = p.c;

        if constexpr (D == 64 && KEY_OWNER && !F16) {
    #include "generated/attn_bwd_loop_kv_d64.inc"
        } else if constexpr (D == 64 && !F16) {
    #include "generated/attn_bwd_loop_q_d64.inc"
        } else if constexpr (D == 64 && KEY_OWNER) {
    #include "generated/attn_bwd_loop_kv_d64_f16.inc"
        } else if constexpr (D == 64) {
    #include "generated/attn_bwd_loop_q_d64_f16.inc"
        } else if constexpr (KEY_OWNER && !F16) {
    #include "generated/attn_bwd_loop_kv_d128.inc"
        } else if constexpr (!KEY_OWNER && !F16) {
    #include "generated/attn_bwd_loop_q_d128.inc"
        } else if constexpr (KEY_OWNER && F16) {
    #include "generated/attn_bwd_loop_kv_d128_f16.inc"
        } else {
    #include "generated/attn_bwd_loop_q_d128_f16.inc"
        }

        // ---- epilogue: dK = -scale * acc[0..], dV = acc[DB..] (or dQ = -scale * acc), 16-bit, row = owner.
        // A lane holds 4-element pieces of ONE owner row: stored directly, a wave-wide store touches 32 rows
        // with 16 bytes each.  So the gradients go through LDS and leave in whole rows: every wave has its own
        // 32 x ROWB bytes of a ring (dK / dQ in the first, dV in the second) and reads back only what it wrote;
        // rows are XOR-swizzled by 16-byte chunk.
        __syncthreads();  // every wave has left the loop (its loads have landed): the rings are free
        if constexpr (D == 128) {
            // the next tile's owner rows travel while this one is written out.  (At D = 64 a second workgroup on the CU
            // does as much, and there are no registers for it.  The tile is located once, here: with a causal mask that is
            // six divisions, and doing it again at the head cost what the early loads win: 373 heads of 33 queries and 940
            // keys 103.6 -> 99.3 us, 451 of 576 rows 269 -> 260, mean over 132 causal calls of several passes -1.3 %.  A tile
            // with none behind it runs straight on, past no code that is not its own: a jump is a fetch more in a short
            // launch.  82 heads of 187 rows 20.0 -> 19.7 us, 134 of 70 rows, causal, 17.0 -> 16.8)
            const int next = queue_entry<PLANNED>(queue, p, plan, blockIdx.x, (int)gridDim.x, pass + 1);
            own_on_its_way = next >= 0 && (KEY_OWNER ? next < queue.n_kv : true);
            if (__builtin_expect(own_on_its_way, 0)) {
                locate(next, bh, ot);
                issue_own_of(bh, ot);
            }
        }
        const int e_lane = D == 64 ? lane_id() : lane;
        const int e_lq = e_lane & 31, e_g = e_lane >> 5;
        auto write_out = [&](const f32x16 *a, auto value, elem_t *out_head, uint32_t ring) {
            typedef typename E::x2 ex2;
            typedef typename E::x4 ex4;
            unsigned char *stage = smem + ring + wave * 32 * ROWB;
    #pragma unroll
            for (int db = 0; db < DB; ++db)
    #pragma unroll
                for (int rb = 0; rb < 4; ++rb) {
                    const f32x2 lo = {value(a[db][4 * rb + 0]), value(a[db][4 * rb + 1])};
                    const f32x2 hi = {value(a[db][4 * rb + 2]), value(a[db][4 * rb + 3])};
                    const ex2 blo = __builtin_convertvector(lo, ex2), bhi = __builtin_convertvector(hi, ex2);  // nearest even
                    const ex4 w = {blo[0], blo[1], bhi[0], bhi[1]};
                    const int chunk = (4 * db + rb) ^ (e_lq & (CPR - 1));
                    *reinterpret_cast<ex4 *>(stage + e_lq * ROWB + chunk * 16 + e_g * 8) = w;
                }
            elem_t *blk = out_head + (size_t)o0w * D;
            const int rows_left = S_own - o0w;  // rows of this wave's block that exist
    #pragma unroll
            for (int i = 0; i < 32 * CPR / 64; ++i) {
                const int idx = i * 64 + e_lane;
                const int r = idx / CPR, c = idx % CPR;
                const u32x4 w = *reinterpret_cast<const u32x4 *>(stage + r * ROWB + ((c ^ (r & (CPR - 1))) * 16));
                if (r < rows_left)
                    *reinterpret_cast<u32x4 *>(blk + (size_t)r * D + c * 8) = w;
            }
        };
        // (+ 0: a zero times -scale is a plain zero, which the keys that no query sees get)
        write_out(acc, [&](float x) { return fmaf(x, -p.scale, 0.f); },
                  reinterpret_cast<elem_t *>(KEY_OWNER ? p.dk : p.dq) + (KEY_OWNER ? k_head : q_head), RING1);
        if constexpr (KEY_OWNER)
            write_out(acc + DB, [](float x) { return x; }, reinterpret_cast<elem_t *>(p.dv) + k_head, RING2);
    }
}

// At D = 64 two workgroups share a CU: 256 registers a wave (all of them VGPRs) must hold either sweep, which a
// test of the compiled kernel checks.  A lone wave per SIMD is bound by the instructions it can issue (matrix pipe 43 %
// busy); two of them fill each other's gaps.  Whole call against one workgroup per CU: 16 heads of 4096 rows 236 -> 223
// us, causal 139 -> 125; 128 heads of 512 rows 46.6 -> 39.9; 512 heads of 300 rows, causal 84 -> 71.  Where one
// workgroup per CU is all there is, the half as many operand buffers cost 2-4 % (16 heads of 1024 rows 22.6 -> 23.1).
template <int D, bool CAUSAL, bool F16, bool PLANNED>
__device__ __forceinline__ void bwd_both_sweeps(const BwdParams &p, const BwdPlan &plan)
{
    const BwdQueue queue(p.total_wg, p.total_q);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int pass = 0;
    bwd_sweep<D, CAUSAL, true, F16, PLANNED>(p, plan, queue, wave, pass);
    bwd_sweep<D, CAUSAL, false, F16, PLANNED>(p, plan, queue, wave, pass);
}

template <int D, bool CAUSAL, bool F16>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_asm_kernel(const BwdParams p)
{
    const BwdPlan none = {};   // (never read)
    bwd_both_sweeps<D, CAUSAL, F16, false>(p, none);
}

template <int D, bool CAUSAL, bool F16>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_asm_planned_kernel(const BwdParams p, const BwdPlan plan)
{
    bwd_both_sweeps<D, CAUSAL, F16, true>(p, plan);
}

}  // namespace attn
