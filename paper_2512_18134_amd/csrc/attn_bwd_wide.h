// attn_bwd_wide.h -- attention-backward sweeps whose waves own 64 rows (D = 128, one wave per SIMD).
//
// The sweeps of attn_bwd_asm.h with owner tiles of 256 rows (four waves) or of 128 (two waves, two workgroups to a CU): the same
// mathematics, the same order of sums, the same bits.  Every operand that a wave reads from LDS feeds two MFMAs, which is
// what the sweeps of 32-row waves are bound by (gen_attn_bwd_wide_loop.py has the schedule; with four waves a streamed tile
// also serves twice as many rows).  Whether and which: pick_tiling in attn_bwd.hip.
//
// Streamed tiles of 32 rows in one 4-stage LDS ring; the owner's rows arrive in LDS as whole rows behind stage 0 and are in
// registers before tiles 1 and 2 go out.  The loop's asm statement takes over once those loads are on their way.
#pragma once
#include "attn_bwd_asm.h"

namespace attn {

// LDS of a workgroup of NW waves: the ring (stage: tile of the first tensor, tile of the second), the owner rows over it from
// OWN on [wave][tensor][64 rows], the LSE' / Delta ring (query owners: those of the owner's rows).  Gradients leave through what
// lies around the owner rows, 32 rows of a wave at a time.  Four waves: the owner rows lie behind stage 0.  Two waves, which
// share the CU's 160 KB with two others: behind the first half of stage 0 (tile 0 of the second tensor goes out later).
template <int NW>
struct BwdWideLds {
    static constexpr int TB = 32 * 128 * 2, STAGE = 2 * TB, OWN = NW == 4 ? STAGE : TB, OWN_TENSOR = 64 * 128 * 2;
    static constexpr int AUX = OWN + NW * 2 * OWN_TENSOR, OUT_1 = NW == 4 ? TB : AUX, OUT_2 = AUX + (NW == 4 ? 0 : TB);
    static constexpr int BYTES = NW * 40 * 1024;
    static __device__ __forceinline__ int out(int wave)   // 8 KB
    {
        return wave == 0 ? 0 : wave == 1 ? OUT_1 : OUT_2 + (wave - 2) * TB;
    }
    static_assert((NW == 4 ? OUT_2 + 2 * TB : OUT_1 + TB) <= BYTES && AUX + NW * 512 <= BYTES && 4 * STAGE <= AUX, "160 KB per CU");
};

// The tile that a workgroup has taken up, and whether its owner rows are on their way to LDS
struct BwdWideTile {
    int bh, ot;
    bool on_its_way;
};

template <int NW, bool CAUSAL, bool KEY_OWNER, bool F16, bool PLANNED>
__device__ __forceinline__ void bwd_wide_sweep(const BwdParams &p, const BwdPlan &plan, const BwdQueue &queue, const int wave,
                                               int &pass, BwdWideTile &tile)
{
    typedef typename std::conditional<F16, ElemF16, ElemBF16>::type E;
    typedef typename E::t elem_t;
    typedef BwdWideLds<NW> Lds;
    constexpr int D = 128, BN = 32, BO = NW * 64, CPR = D / 8, KS = D / 16, DB = D / 32, ROWB = D * 2, TB = Lds::TB;
    constexpr int NLD = TB / (NW * 1024), NVOFF = 2, NSET = KEY_OWNER ? 2 : 1;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(ATTN_LDS_PTR(unsigned char))smem;

    // (asked from the hardware wherever it is needed: the loop leaves no register to keep it in)
    auto lane_id = []() -> int {
        int ones = -1;
        asm volatile("" : "+s"(ones));
        return __builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0));
    };

    auto el = [](const bf16_t *ptr) { return reinterpret_cast<const elem_t *>(ptr); };
    // The place and the owner rows of a tile of either sweep.  (Asked for anew in every tile: what the compiler takes out of
    // the tile loop costs registers that the loop has not)
    auto locate = [&](int entry) {
        const bool keys = entry < queue.n_kv;
        int n_t = keys ? p.n_t : p.n_tq, total = keys ? p.total_wg : p.total_q, rows = p.S_q + p.S_kv;
        asm volatile("" : "+s"(n_t), "+s"(total), "+s"(rows));
        wg_to_tile_n<CAUSAL>(keys ? entry : entry - queue.q_first, total, n_t, 4ll * rows * D, tile.bh, tile.ot);
        if (CAUSAL && keys)
            tile.ot = n_t - 1 - tile.ot;  // early key tiles stream the most queries: heaviest first
    };
    const uint32_t own_1 = lds0 + Lds::OWN + wave * 2 * Lds::OWN_TENSOR, own_2 = own_1 + Lds::OWN_TENSOR;
    // a quarter of the owner rows: 16 rows of both tensors
    auto issue_own = [&](bool keys, int quarter) {
        const size_t head = (size_t)tile.bh * (keys ? p.S_kv : p.S_q) * D;
        const elem_t *x1 = el(keys ? p.k : p.q) + head, *x2 = el(keys ? p.v : p.d_o) + head;
        const int row0 = tile.ot * BO + wave * 64, last = (keys ? p.S_kv : p.S_q) - 1;
        const int ln = lane_id();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * (4 * quarter + i) + ln / CPR;
            const uint32_t voff = (uint32_t)min(row0 + r, last) * ROWB + (uint32_t)(((ln % CPR) ^ swz<D>(r)) * 16);
            dma16(own_1 + (4 * quarter + i) * 1024, x1, voff);
            dma16(own_2 + (4 * quarter + i) * 1024, x2, voff);
        }
    };
#pragma clang loop unroll(disable)
    for (;; ++pass) {
        const int entry = queue_entry<PLANNED>(queue, p, plan, blockIdx.x, (int)gridDim.x, pass);
        if (entry < 0 || (KEY_OWNER && entry >= queue.n_kv))
            break;   // (entries rise from pass to pass; only the last pass can be short)
        if (!KEY_OWNER && entry < queue.q_first)
            continue;
        if (pass > 0)
            __syncthreads();  // every wave has read the previous tile's staged gradients back: the LDS is free
        if (!tile.on_its_way) {
            locate(entry);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                issue_own(KEY_OWNER, i);
        }
        const int bh = tile.bh, ot = tile.ot;
        const int S_own = KEY_OWNER ? p.S_kv : p.S_q;
        const int S_str = KEY_OWNER ? p.S_q : p.S_kv;
        const int o0 = ot * BO, o0w = o0 + wave * 64;
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
        // The wave's own part: key owners begin at tile n_wave (an even number, or n_tiles: none), the first that a query of
        // theirs can be in; query owners compute n_wave tiles.  Tiles j < j_lo touch the causal diagonal from below (key
        // owners), tiles j >= j_hi the ragged end of the streamed tensor or the diagonal from above (query owners).
        int n_wave, j_hi = t_full - t_begin;
        [[maybe_unused]] const int j_lo = CAUSAL ? o0w / BN - t_begin + 2 : 0;
        if (KEY_OWNER) {
            n_wave = o0w < S_own ? (CAUSAL ? min(2 * wave, n_tiles) : 0) : n_tiles;
        } else {
            n_wave = o0w < S_own ? (CAUSAL ? min(o0w / BN + 2, n_tiles) : n_tiles) : 0;
            if (CAUSAL)
                j_hi = min(j_hi, o0w / BN);
        }

        // ---- addresses inside a tile (the loop keeps them in the registers they come in)
        const int lane = lane_id();
        const int lq = lane & 31, g = lane >> 5;
        typename U32Vec<NVOFF>::type dma_voff_v;
#pragma unroll
        for (int i = 0; i < NVOFF; ++i) {
            const int row = 4 * (i * NW + wave) + lane / CPR;
            U32Vec<NVOFF>::set(dma_voff_v, i, row * ROWB + (uint32_t)(((lane % CPR) ^ swz<D>(row)) * 16));
        }
        const uint32_t lds_wave = lds0 + wave * 1024, lds_aux = lds0 + Lds::AUX;
        const uint32_t aux_sel = g ? (uint32_t)(p.n_rows * 4) : 0u;

        // ---- tile 0 (and, query owners, LSE' and Delta of the owner rows)
        if (!KEY_OWNER)
#pragma unroll
            for (int k = 0; k < 2; ++k)
                dma4(lds_aux + wave * 512 + k * 256, aux_head, (uint32_t)min(o0w + 32 * k + lq, S_own - 1) * 4 + aux_sel);
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const uint32_t row = dma_voff_v[i % NVOFF] / ROWB + 4 * NW * NVOFF * (i / NVOFF);
            const uint32_t voff = (uint32_t)min(t_begin * BN + (int)row, str_m1) * ROWB + dma_voff_v[i % NVOFF] % ROWB;
            dma16(lds_wave + i * NW * 1024, t1_head, voff);
            if (NW == 4)
                dma16(lds_wave + TB + i * NW * 1024, t2_head, voff);
        }
        if (KEY_OWNER)
            dma4(lds_aux, aux_head, (uint32_t)min(t_begin * BN + lq, str_m1) * 4 + aux_sel);

        typename U32Vec<KS>::type roff_v;
        typename U32Vec<2 * DB>::type toff_v;
        {
            const int sw = swz<D>(lq);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                roff_v[ks] = lds0 + (uint32_t)(lq * ROWB + (((2 * ks + g) ^ sw) * 16));
            const int i16 = lane & 15, dh = (lane >> 4) & 1;
            const int rho = i16 >> 2, pi = i16 & 3;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int hlf = 0; hlf < 2; ++hlf) {
                    const int row = 4 * g + 8 * hlf + rho;
                    const int ch = 4 * db + 2 * dh + (pi >> 1);
                    toff_v[2 * db + hlf] = lds0 + (uint32_t)(row * ROWB + ((ch ^ swz<D>(row)) * 16) + (pi & 1) * 8);
                }
        }
        // mask thresholds of this lane, minus the lane-group part of the accumulator row and the first tile
        const int own = o0w + lq;
        [[maybe_unused]] const uint32_t thr_lo_base = (uint32_t)(own - 4 * g - BN * t_begin);
        uint32_t thr_hi_base[2];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            thr_hi_base[k] = (uint32_t)((!KEY_OWNER && CAUSAL ? min(own + 32 * k, str_m1) : str_m1) - 4 * g - BN * t_begin);
        const uint32_t aux_off = KEY_OWNER ? lds_aux + 16 * g : lds_aux + wave * 512 + lq * 4;
        [[maybe_unused]] const uint32_t aux_voff = (uint32_t)(lq * 4) + aux_sel;
        const uint32_t own_off = own_1 - lds0;
        const float c_log2e = p.c;
        f32x16 acc[NSET * 2 * DB];

        if constexpr (NW == 4 && KEY_OWNER && !F16) {
#include "generated/attn_bwd_wide_loop_kv_w4.inc"
        } else if constexpr (NW == 4 && !KEY_OWNER && !F16) {
#include "generated/attn_bwd_wide_loop_q_w4.inc"
        } else if constexpr (NW == 4 && KEY_OWNER && F16) {
#include "generated/attn_bwd_wide_loop_kv_w4_f16.inc"
        } else if constexpr (NW == 4 && !KEY_OWNER && F16) {
#include "generated/attn_bwd_wide_loop_q_w4_f16.inc"
        } else if constexpr (NW == 2 && KEY_OWNER && !F16) {
#include "generated/attn_bwd_wide_loop_kv_w2.inc"
        } else if constexpr (NW == 2 && !KEY_OWNER && !F16) {
#include "generated/attn_bwd_wide_loop_q_w2.inc"
        } else if constexpr (NW == 2 && KEY_OWNER && F16) {
#include "generated/attn_bwd_wide_loop_kv_w2_f16.inc"
        } else if constexpr (NW == 2 && !KEY_OWNER && F16) {
#include "generated/attn_bwd_wide_loop_q_w2_f16.inc"
        }

        // ---- epilogue: dK = -scale * acc[0..], dV = acc[2 DB..] (or dQ = -scale * acc), 16-bit, row = owner, through LDS in whole
        // rows: every wave has room for 32 rows and reads back only what it wrote.  Between the steps the owner rows of the
        // workgroup's next tile go out, whichever sweep it belongs to.
        __syncthreads();  // every wave has left the loop (its loads have landed): the LDS is free
        const int next = queue_entry<PLANNED>(queue, p, plan, blockIdx.x, (int)gridDim.x, pass + 1);
        tile.on_its_way = next >= 0 && (next < queue.n_kv || next >= queue.q_first);
        if (tile.on_its_way)
            locate(next);
        const int e_lane = lane_id();
        const int e_lq = e_lane & 31, e_g = e_lane >> 5;
        unsigned char *const stage = smem + Lds::out(wave);
        auto write_out = [&](const f32x16 *a, auto value, elem_t *out_head, int k) {
            typedef typename E::x2 ex2;
            typedef typename E::x4 ex4;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) {
                    const f32x16 &x = a[DB * k + db];
                    const f32x2 lo = {value(x[4 * rb + 0]), value(x[4 * rb + 1])};
                    const f32x2 hi = {value(x[4 * rb + 2]), value(x[4 * rb + 3])};
                    const ex2 blo = __builtin_convertvector(lo, ex2), bhi = __builtin_convertvector(hi, ex2);  // nearest even
                    const ex4 w = {blo[0], blo[1], bhi[0], bhi[1]};
                    const int chunk = (4 * db + rb) ^ (e_lq & (CPR - 1));
                    *reinterpret_cast<ex4 *>(stage + e_lq * ROWB + chunk * 16 + e_g * 8) = w;
                }
            unsigned char *blk = reinterpret_cast<unsigned char *>(out_head + (size_t)(o0w + 32 * k) * D);
            const int rows_left = S_own - o0w - 32 * k;  // rows of this block that exist
#pragma unroll
            for (int i = 0; i < 32 * CPR / 64; ++i) {
                const int r = 4 * i + e_lane / CPR, c = e_lane % CPR;
                const u32x4 w = *reinterpret_cast<const u32x4 *>(stage + r * ROWB + ((c ^ (r & (CPR - 1))) * 16));
                if (r < rows_left) {   // (row r, chunk c; an offset that the compiler makes no 64-bit address of ahead of the branch)
                    uint32_t at = (uint32_t)(i * 1024 + e_lane * 16);
                    asm volatile("" : "+v"(at));
                    *reinterpret_cast<u32x4 *>(blk + at) = w;
                }
            }
        };
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            // (+ 0: a zero times -scale is a plain zero, which the keys that no query sees get)
            write_out(acc, [&](float x) { return fmaf(x, -p.scale, 0.f); },
                      reinterpret_cast<elem_t *>(KEY_OWNER ? p.dk : p.dq) + (KEY_OWNER ? k_head : q_head), k);
            if (tile.on_its_way) {
                issue_own(next < queue.n_kv, 2 * k);
                issue_own(next < queue.n_kv, 2 * k + 1);
            }
            if constexpr (KEY_OWNER)
                write_out(acc + 2 * DB, [](float x) { return x; }, reinterpret_cast<elem_t *>(p.dv) + k_head, k);
        }
    }
}

template <int NW, bool CAUSAL, bool F16, bool PLANNED>
__device__ __forceinline__ void bwd_wide_both_sweeps(const BwdParams &p, const BwdPlan &plan)
{
    const BwdQueue queue(p.total_wg, p.total_q);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int pass = 0;
    BwdWideTile tile = {0, 0, false};
    bwd_wide_sweep<NW, CAUSAL, true, F16, PLANNED>(p, plan, queue, wave, pass, tile);
    bwd_wide_sweep<NW, CAUSAL, false, F16, PLANNED>(p, plan, queue, wave, pass, tile);
}

template <int NW, bool CAUSAL, bool F16>
__global__ __launch_bounds__(NW * 64) void attn_bwd_wide_kernel(const BwdParams p)
{
    const BwdPlan none = {};   // (never read)
    bwd_wide_both_sweeps<NW, CAUSAL, F16, false>(p, none);
}

template <int NW, bool CAUSAL, bool F16>
__global__ __launch_bounds__(NW * 64) void attn_bwd_wide_planned_kernel(const BwdParams p, const BwdPlan plan)
{
    bwd_wide_both_sweeps<NW, CAUSAL, F16, true>(p, plan);
}

}  // namespace attn
