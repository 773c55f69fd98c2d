// attn_fwd_asm.h -- attention-forward kernels whose main loop is hand scheduled.
//
// Transposed products S^T = K Q^T, O^T = V^T P^T on v_mfma_f32_32x32x16_bf16 (a lane
// owns one query: the softmax reductions stay in the lane), online softmax against
// a lazily moved reference, direct global->LDS K/V loads.  The steady-state loop --
// the paper's Fig. 1a in the three-stage modulo schedule described in
// gen_attn_loop.py -- is one inline-asm statement generated by that script, with
// every register assigned by hand: the compiler cannot hold the schedule in the
// registers a wave has.  This file does what surrounds the loop: work
// decomposition, addressing, the start of the K/V stream, the Q load, S(0), and
// the epilogue.
//
// Tilings (template parameters; gen_attn_loop.py CONFIGS holds the matching loops):
//   QB  32-row query blocks per wave     SB  32-key blocks per K/V tile (BN = 32 SB)
//   NW  waves per key group (BM = 32 QB NW query rows)    G  key groups per workgroup
//   <D=64|128, QB=1, SB=2, NW=8>  two waves per SIMD, everything in 256 VGPRs
//   <D=64,     QB=1, SB=2, NW=4>  the same with BM = 128 (two workgroups per CU)
//   <D=128, QB=1, SB=1, NW=2, G=2>, <D=64, QB=1, SB=2, NW=2, G=2>
//                                  launches with few queries: BM = 64, and the keys of a tile cut in two halves that
//                                  two groups of NW waves (each with rings of its own) work on side by side; their
//                                  results meet in LDS (finish_groups).  One wave per SIMD walks half the keys: what
//                                  bounds it is the walk (0.4 us per 32 keys, issue and load latency), not the products
//   <D=128,    QB=2, SB=1, NW=4>  one wave per SIMD, O and Q in AGPRs; a K / V^T fragment
//                                  read from LDS feeds two MFMAs (half the LDS reads)
//   <D=128,    QB=2, SB=1, NW=2>  the same with BM = 128 (two workgroups per CU; the same results)
//   <D=128,    QB=1, SB=1, NW=4>  BM = 128 in 32-row waves (two workgroups per CU, two waves per SIMD) that move their
//                                  references in pairs, as the 64-row waves do (the same results: PairedGen): half the work per
//                                  wave and tile, for launches that a wave's walk bounds
//   <D=256,    QB=1, SB=1, NW=4>  one wave per SIMD, O and Q in AGPRs
// K/V tiles in two 4-stage LDS rings (8 * BN * D * 2 bytes).  The kernel starts S(0) as soon as K(0)
// and Q have landed; the other five tiles of the ring fill behind it.
// Requires scale > 0 (masked scores are set to -inf before the multiply by
// scale*log2e) and S_kv * D * 2 < 2^31.
#pragma once
#include <type_traits>

#include "attn_common.h"
#include "attn_dma.h"  // dma16, wait_vmcnt

namespace attn {

template <int N>
struct U32Vec {
    typedef uint32_t type __attribute__((ext_vector_type(N)));
    static __device__ __forceinline__ void set(type &v, int i, uint32_t x) { v[i] = x; }
};
template <>
struct U32Vec<1> {
    typedef uint32_t type;
    static __device__ __forceinline__ void set(type &v, int, uint32_t x) { v = x; }
};
template <int N>
struct F32Vec {
    typedef float type __attribute__((ext_vector_type(N)));
    static __device__ __forceinline__ float get(const type &v, int i) { return v[i]; }
};
template <>
struct F32Vec<1> {
    typedef float type;
    static __device__ __forceinline__ float get(const type &v, int) { return v; }
};

// Element type of Q, K, V, O: bf16, or IEEE fp16 (the type of the paper's Section 6 evaluation).
// The two differ in the MFMA instruction and in the float -> 16-bit pack, nowhere else.
struct ElemBF16 {
    typedef __bf16 t;
    typedef __attribute__((ext_vector_type(2))) __bf16 x2;
    typedef __attribute__((ext_vector_type(4))) __bf16 x4;
    typedef __attribute__((ext_vector_type(8))) __bf16 x8;
    static __device__ __forceinline__ f32x16 mfma(x8 a, x8 b, f32x16 c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};
struct ElemF16 {
    typedef _Float16 t;
    typedef __attribute__((ext_vector_type(2))) _Float16 x2;
    typedef __attribute__((ext_vector_type(4))) _Float16 x4;
    typedef __attribute__((ext_vector_type(8))) _Float16 x8;
    static __device__ __forceinline__ f32x16 mfma(x8 a, x8 b, f32x16 c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};

// Workgroup shape and LDS budget of a tiling, shared by the kernel and the host code that launches it.
template <int D, int QB, int SB, int NW, bool SPLIT, int G = 1>
struct FwdTiling {
    static constexpr int BN = 32 * SB, BM = NW * 32 * QB;
    static constexpr int THREADS = NW * G * 64;
    static constexpr int RING_BYTES = 8 * BN * D * 2;     // K ring [4] + V ring [4] of one key group
    static constexpr int STAGE_BYTES = BM * D * 2;        // O of one tile, 16-bit
    // A staging area [BM][D] next to the rings when it fits (160 KB of LDS per CU, one workgroup per CU): a tile's
    // Q rows arrive there by direct loads (whole rows, coalesced), the next tile's while the finished one is
    // written out.  Without it Q is loaded straight into registers (32-byte pieces).  O is staged in the rings
    // once the loop has left them.
    static constexpr bool HAS_STAGE = !SPLIT && G == 1 && NW * QB == 8 && RING_BYTES + STAGE_BYTES <= 160 * 1024;
    // 32-row waves that test their tiles' row sums in pairs (gen_attn_loop.py, PairedGen): the sums pass through LDS
    static constexpr bool PAIRED = D == 128 && QB == 1 && SB == 1 && G == 1;
    static constexpr int XCH_SUMS = G * RING_BYTES, XCH_SUMS_BYTES = PAIRED ? 2 * NW * 64 * 4 : 0;
    // fp32 partial rows of a split-KV range leave in whole rows where launches with many queries come (stored by the lanes
    // that hold them, a wave-wide store touches 32 rows with 16 bytes each): 16 heads of 400 queries and 20000 keys, D = 64, 53.2
    // -> 51.3 us; one query: 28.8 -> 29.1, which the 4-wave tiling is for
    static constexpr bool WHOLE_PARTS = SPLIT && D == 64 && NW == 8;
    static constexpr int LDS_BYTES = XCH_SUMS + XCH_SUMS_BYTES + (HAS_STAGE ? STAGE_BYTES : 0);
    // Persistent workgroups (see attn_fwd_asm_kernel) wherever the loop leaves the compiler registers to carry
    // a tile's state across it: the 8-wave D = 128 loop assigns all 256 VGPRs itself, and a split-KV launch
    // has a workgroup per (tile, key range)
    static constexpr bool PERSIST = !SPLIT && !(D == 128 && QB == 1 && SB == 2);
    // the 4-wave D = 64 and paired workgroups are meant to run two to a CU: their waves must fit half a SIMD's registers
    static constexpr int MIN_WAVES_PER_SIMD = ((D == 64 && NW == 4) || PAIRED) ? 2 : 1;
    // ... and the 2-wave D = 128 ones, by their 64 KB of LDS
    static constexpr bool TWO_PER_CU = (D == 64 && NW == 4) || (D == 128 && QB == 2 && NW == 2) || PAIRED;
    static_assert(!(PAIRED && HAS_STAGE), "the row sums lie behind the rings");
    static_assert(SPLIT || STAGE_BYTES <= RING_BYTES, "O staging must fit the rings");
    // the two key groups exchange half of their fp32 accumulators, their row maxima and sums, then stage half rows
    static constexpr int XCH_O = 0, XCH_ML = 2 * NW * 32 * D * 2, XCH_STAGE = XCH_ML + 2 * NW * 64 * 8;
    static_assert(G == 1 || (G == 2 && QB == 1 && XCH_STAGE + 2 * NW * 32 * D <= LDS_BYTES), "the exchange must fit the rings");
};

// SPLIT: the workgroup handles one key range of a split-KV launch (see Params) and writes its
// normalised partial O (fp32) and its log-sum-exp to the workspace instead of o / lse.
//
// Workgroups are persistent (FwdTiling::PERSIST): the launch has at most one workgroup per CU slot (gridDim.x a
// multiple of the XCD count unless every tile has a workgroup of its own), and workgroup `blockIdx.x` walks the
// tile queue of its XCD (persistent_entry), so that no dispatch gap separates two tiles of a CU.
template <int D, int QB, int SB, int NW, bool CAUSAL, bool F16 = false, bool SPLIT = false, int G = 1>
__global__ __launch_bounds__(NW * G * 64, (D == 64 && NW == 4) || (D == 128 && QB == 1 && SB == 1 && G == 1) ? 2 : 1)  // = FwdTiling::MIN_WAVES_PER_SIMD
    void attn_fwd_asm_kernel(const Params p)
{
    static_assert((QB == 1 && SB == 2 && (D == 64 || D == 128) && NW == 8 && G == 1) ||
                      (QB == 1 && SB == 2 && D == 64 && ((NW == 4 && G == 1) || (NW == 2 && G == 2))) ||
                      (QB == 1 && SB == 1 && D == 128 && ((NW == 2 && G == 2) || (NW == 4 && G == 1 && !SPLIT))) ||
                      (QB == 2 && SB == 1 && D == 128 && (NW == 4 || (NW == 2 && !SPLIT)) && G == 1) ||
                      (QB == 1 && SB == 1 && D == 256 && NW == 4 && G == 1 && !SPLIT),
                  "no generated loop for this tiling");
    static_assert(!(SPLIT && CAUSAL), "split-KV launches are not causal");
    typedef typename std::conditional<F16, ElemF16, ElemBF16>::type E;
    typedef typename E::t elem_t;
    typedef typename E::x8 ex8;
    typedef FwdTiling<D, QB, SB, NW, SPLIT, G> T;
    constexpr int BN = T::BN, BM = T::BM, NST = 4;
    constexpr int CPR = D / 8;   // 16-byte chunks per row
    constexpr int KS = D / 16;   // k-steps of K Q^T
    constexpr int DB = D / 32;   // 32-wide blocks of the head dimension
    constexpr int ROWB = D * 2;
    constexpr int TB = BN * ROWB;
    constexpr int NLD = TB / (NW * 1024);
    constexpr int RPG = 1024 / ROWB;
    constexpr int NQP = 4 * QB * KS / 16;  // Q fragments packed 16 dwords at a time
    constexpr bool HAS_STAGE = T::HAS_STAGE;
    constexpr int NQT = BM / BN;           // Q rows of a tile in units of K/V tiles (same LDS layout)

    // K ring [4][TB], V ring [4][TB] (after the loop: O on its way out), then (HAS_STAGE) the staging area [BM][ROWB] of Q
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr uint32_t KRING = 0, VRING = NST * TB;
    constexpr uint32_t STAGE = HAS_STAGE ? T::RING_BYTES : 0;   // Q staging area
    unsigned char *const o_stage = smem;                          // O is staged in the rings, after the loop

    const int tid = threadIdx.x;
    int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = G == 1 ? 0 : wave_wg / NW;    // key group of this wave
    const int wave = G == 1 ? wave_wg : wave_wg % NW;   // ... and its place in the group
    const uint32_t lds0 = (uint32_t)(uintptr_t)(ATTN_LDS_PTR(unsigned char))smem + grp * T::RING_BYTES;
    int lq = lane & 31;
    int g = lane >> 5;

    // ---- this workgroup's walk through the tile queue of its XCD (persistent_entry)
    const int n_slots = T::PERSIST ? (int)gridDim.x : p.total_wg;
    // Where two workgroups share a CU, workgroups m and m + cus_per_xcd of an XCD do (measured): the first ones take their
    // places in the queue in reverse, so that a CU pairs heavy with light tiles of a causal launch (within a pass;
    // persistent_entry does it between passes).  D = 64, causal: 32 heads of 2048 rows 26.1 -> 23.6 us, of 2100 29.6 -> 26.8,
    // 17 of 4096 rows 48.4 -> 43.5, 4 of 16384 rows 163 -> 151; launches with one tile per CU do not change; with many
    // passes either order is a few percent ahead now and then (100 heads of 1352 rows 38.7 -> 36.9, 213 77.7 -> 81.8)
    int place = blockIdx.x;
    if constexpr (CAUSAL && T::TWO_PER_CU) {
        const int xcd = place % kNumXcd, m = place / kNumXcd;
        const int n = n_slots >= p.total_wg ? (p.total_wg - xcd + kNumXcd - 1) / kNumXcd : n_slots / kNumXcd;
        const int first = min(n, p.cus_per_xcd);
        place = (m < first ? first - 1 - m : m) * kNumXcd + xcd;
    }
    auto virtual_wg = [&](int k) -> int { return persistent_entry(place, n_slots, p.total_wg, k); };
    const int n_pass =   // the longest queue of an XCD, in passes of n_slots / 8 entries
        n_slots >= p.total_wg ? 1 : ((p.total_wg + kNumXcd - 1) / kNumXcd + n_slots / kNumXcd - 1) / (n_slots / kNumXcd);

    // ---- one tile of the launch: which head and query rows, which keys
    struct Tile {
        int vb, bh, split, q0, kv0, S_kv, n_tiles, own_tiles, j_mask, t_full, skv_m1;
        const elem_t *qg, *k_head, *v_head;
    };
    auto locate = [&](int vb) -> Tile {
        Tile t;
        t.vb = vb;
        int qt;
        t.split = 0;
        if (SPLIT) {
            // (head, key range) is the slow index: the query tiles that stream one key range are neighbours
            const int logical = xcd_remap(vb, p.total_wg);
            qt = logical % p.n_qt;
            const int hs = logical / p.n_qt;
            t.bh = hs / p.n_split;
            t.split = hs % p.n_split;
        } else {
            wg_to_tile<CAUSAL>(vb, p, D, t.bh, qt);
        }
        t.kv0 = SPLIT ? t.split * p.split_len : 0;                        // first key of this tile's range
        t.S_kv = SPLIT ? min(p.split_len, p.S_kv - t.kv0) : p.S_kv;       // keys of this tile's range
        t.q0 = qt * BM;
        int kv_end = t.S_kv;
        if (CAUSAL)
            kv_end = min(kv_end, min(t.q0 + BM, p.S_q));
        t.n_tiles = (kv_end + BN - 1) / BN;
        const int j_tail = (t.n_tiles * BN > t.S_kv) ? t.n_tiles - 1 : t.n_tiles;
        t.j_mask = CAUSAL ? min(t.q0 / BN, j_tail) : j_tail;  // first K/V tile whose scores need a mask
        t.own_tiles = t.n_tiles;
        if constexpr (G == 2) {
            // the first key group takes the larger half of the tiles; a single tile is computed by both groups and
            // left out of the second one's result (run_tile: idle)
            const int n0 = (t.n_tiles + 1) / 2;
            const int j0 = grp && t.n_tiles > 1 ? n0 : 0;
            t.own_tiles = grp ? max(t.n_tiles - n0, 1) : n0;
            t.n_tiles = n0;
            t.j_mask = max(t.j_mask - j0, 0);
            t.kv0 += j0 * BN;
            t.S_kv -= j0 * BN;
        }
        t.qg = reinterpret_cast<const elem_t *>(p.q) + (size_t)t.bh * p.S_q * D;
        t.k_head = reinterpret_cast<const elem_t *>(p.k) + ((size_t)t.bh * p.S_kv + t.kv0) * D;
        t.v_head = reinterpret_cast<const elem_t *>(p.v) + ((size_t)t.bh * p.S_kv + t.kv0) * D;
        t.t_full = t.S_kv / BN;                               // K/V tiles below this lie inside [0, S_kv)
        t.skv_m1 = t.S_kv - 1;
        return t;
    };
    auto qcol = [&](const Tile &t, int qb) { return t.q0 + (wave * QB + qb) * 32 + lq; };  // query row of this lane

    // ---- direct-load addressing: lane -> (row in tile, 16-byte chunk).  A wave-wide load fills 1 KB of
    // LDS linearly (lane*16); the XOR swizzle is applied on the global side: the lane that fills
    // physical chunk pc of a row fetches logical chunk pc ^ swz(row) (within its group of 16 chunks).
    // A wave fills NLD consecutive KB of a tile: the loop writes m0 once per tile and gives load i the
    // immediate offset i KB, which the hardware adds to the LDS address and to the global address alike,
    // so the loop's offset register of load i (dma_voff_v) holds i KB less (never negative: the rows of
    // load i start i KB into the tile).
    typename U32Vec<NLD>::type dma_row_v, dma_choff_v, dma_voff_v;
    uint32_t dma_row[NLD], dma_choff[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int gi = wave * NLD + i;
        dma_row[i] = RPG * gi + lane / CPR;
        const int ch = lane % CPR;
        dma_choff[i] = (uint32_t)(((ch & ~15) | ((ch & 15) ^ swz<D>(dma_row[i]))) * 16);
        U32Vec<NLD>::set(dma_row_v, i, dma_row[i]);
        U32Vec<NLD>::set(dma_choff_v, i, dma_choff[i]);
        U32Vec<NLD>::set(dma_voff_v, i, dma_row[i] * ROWB + dma_choff[i] - i * 1024);
    }
    // BN rows from row0 on of a [rows][D] tensor into LDS at lds_off (K/V tile layout); rows past `last` re-read it
    auto issue_rows = [&](const elem_t *base, uint32_t lds_off, int row0, int last) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int r = min(row0 + (int)dma_row[i], last);
            dma16(lds0 + lds_off + (wave * NLD + i) * 1024, base, (uint32_t)r * ROWB + dma_choff[i]);
        }
    };
    auto issue_tile = [&](const Tile &t, const elem_t *base, uint32_t ring_off, int stage, int j) {
        issue_rows(base, ring_off + stage * TB, j * BN, t.S_kv - 1);
    };
    const uint32_t lds_k_wave = lds0 + KRING + wave * NLD * 1024;
    const uint32_t lds_v_wave = lds0 + VRING + wave * NLD * 1024;

    // ---- operand addressing inside a tile (ring base folded in, stage offset is an immediate)
    uint32_t koff[KS];
    typename U32Vec<KS>::type koff_v;
    {
        const int sw = swz<D>(lq);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int ch = 2 * ks + g;
            koff[ks] = lds0 + KRING + (uint32_t)(lq * ROWB + (((ch & ~15) | ((ch & 15) ^ sw)) * 16));
            koff_v[ks] = koff[ks];
        }
    }
    // V^T as A operand through ds_read_b64_tr_b16: in a 16-lane block, source lane i supplies the 8-byte
    // piece i%4 of row i/4; lane L receives column L of those four rows
    typename U32Vec<2 * DB>::type voff_v;
    {
        const int i16 = lane & 15, dh = (lane >> 4) & 1;
        const int rho = i16 >> 2, pi = i16 & 3;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int hlf = 0; hlf < 2; ++hlf) {
                const int row = 4 * g + 8 * hlf + rho;
                const int ch = 4 * db + 2 * dh + (pi >> 1);
                voff_v[2 * db + hlf] = lds0 + VRING +
                    (uint32_t)(row * ROWB + (((ch & ~15) | ((ch & 15) ^ swz<D>(row))) * 16) + (pi & 1) * 8);
            }
    }

    // ---- start of a tile's K/V stream and its Q load: K(0) and Q first (S(0) needs nothing else), then
    // K(1), V(0), K(2), and last the two tiles that may still be in flight when the loop starts: K(3), V(1).
    // Q goes to the staging area like K/V tiles do (HAS_STAGE), or straight into registers by asm statements,
    // so that the wait the kernel places is the only wait for it (a load the compiler knows is waited for with
    // vmcnt(0) at its first use, which would also wait for every tile behind it).
    u32x4 q_raw[QB][KS];
    // part k of 2 QB of a tile's Q rows into the staging area
    auto issue_q_part = [&](const Tile &t, int k) {
        constexpr int PER = NQT / (2 * QB);
        static_assert(!HAS_STAGE || NQT % (2 * QB) == 0, "the Q rows go out in 2 QB equal parts");
#pragma unroll
        for (int i = k * PER; i < (k + 1) * PER; ++i)
            issue_rows(t.qg, STAGE + i * TB, t.q0 + i * BN, p.S_q - 1);
    };
    auto issue_q = [&](const Tile &t) {
        if constexpr (HAS_STAGE) {
#pragma unroll
            for (int k = 0; k < 2 * QB; ++k)
                issue_q_part(t, k);
        } else {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const elem_t *src = t.qg + (size_t)min(qcol(t, qb), p.S_q - 1) * D + 8 * g;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=v"(q_raw[qb][ks]) : "v"(src), "n"(32 * ks));
            }
        }
    };
    // q_too: the tile's Q goes out behind K(0); otherwise it is already on its way (see the tile loop)
    auto issue_loads = [&](const Tile &t, auto q_too) {
        issue_tile(t, t.k_head, KRING, 0, 0);
        if constexpr (decltype(q_too)::value)
            issue_q(t);
        issue_tile(t, t.k_head, KRING, 1, 1);
        issue_tile(t, t.v_head, VRING, 0, 0);
        issue_tile(t, t.k_head, KRING, 2, 2);
        issue_tile(t, t.k_head, KRING, 3, 3);
        issue_tile(t, t.v_head, VRING, 1, 1);
    };

    // ---- end of a tile: normalise, write O (16-bit) and the log-sum-exp (fp32)
    typename F32Vec<QB>::type m_ref_v, l_run_v;
    f32x16 o_acc[QB * DB];
    bool idle = false;   // second key group only: this wave's result does not count
    // Two key groups: wave w of either group holds the same 32 query rows, lane for lane.  Each wave hands the other
    // one half of the head dimension (fp32, with its row maxima and sums), combines the half it keeps -- the
    // accumulator rescale of the online softmax, once more -- and writes that half of the rows out.
    auto finish_groups = [&](const Tile &t) {
        constexpr int HB = DB / 2, HCPR = CPR / 2, HROWB = ROWB / 2;
        const float l_lane = F32Vec<QB>::get(l_run_v, 0);
        const float l_own = idle ? 0.f : l_lane + xor32(l_lane);
        const float m_own = idle ? -INFINITY : F32Vec<QB>::get(m_ref_v, 0);
        if (idle) {   // (a weight of zero would not do: keys that no row of this wave sees may hold NaN or infinities)
#pragma unroll
            for (int i = 0; i < DB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    o_acc[i][r] = 0.f;
        }
        float *const xo = reinterpret_cast<float *>(smem + T::XCH_O);
        f32x2 *const xml = reinterpret_cast<f32x2 *>(smem + T::XCH_ML);
        // element r of the half this wave keeps (mine) or hands over
        auto half = [&](bool mine, int r) -> float {
            const float lo = o_acc[r / 16][r % 16], hi = o_acc[HB + r / 16][r % 16];
            return (grp == 0) == mine ? lo : hi;
        };
#pragma unroll
        for (int i = 0; i < 4 * HB; ++i) {
            const f32x4 w = {half(false, 4 * i), half(false, 4 * i + 1), half(false, 4 * i + 2), half(false, 4 * i + 3)};
            *reinterpret_cast<f32x4 *>(xo + ((wave_wg * 4 * HB + i) * 64 + lane) * 4) = w;
        }
        const f32x2 ml = {m_own, l_own};
        xml[wave_wg * 64 + lane] = ml;
        __syncthreads();
        const int other = wave + (1 - grp) * NW;
        const f32x2 ml_o = xml[other * 64 + lane];
        const float m = fmaxf(m_own, ml_o[0]);
        const float w_own = __builtin_amdgcn_exp2f((m_own - m) * p.c), w_oth = __builtin_amdgcn_exp2f((ml_o[0] - m) * p.c);
        const float l_tot = w_own * l_own + w_oth * ml_o[1];
        const float inv = 1.f / l_tot;
        const float a_own = w_own * inv, a_oth = w_oth * inv;
        const float lse_row = m * p.scale + __builtin_amdgcn_logf(l_tot) * 0.69314718055994530942f;
        f32x16 o_half[HB];
#pragma unroll
        for (int i = 0; i < 4 * HB; ++i) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(xo + ((other * 4 * HB + i) * 64 + lane) * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                o_half[i / 4][4 * (i % 4) + r] = half(true, 4 * i + r) * a_own + x[r] * a_oth;
        }
        const int row0 = t.q0 + wave * 32, qrow = row0 + lq;
        if constexpr (SPLIT) {
            const size_t n_rows = (size_t)(p.total_wg / (p.n_qt * p.n_split)) * p.S_q;
            if (qrow < p.S_q) {
                const size_t row = (size_t)t.split * n_rows + (size_t)t.bh * p.S_q + qrow;
                float *orow = p.o_part + row * D + grp * (D / 2);
#pragma unroll
                for (int i = 0; i < 4 * HB; ++i) {
                    const f32x16 &x = o_half[i / 4];
                    const int r = 4 * (i % 4);
                    const f32x4 w = {x[r], x[r + 1], x[r + 2], x[r + 3]};
                    *reinterpret_cast<f32x4 *>(orow + 8 * i + 4 * g) = w;
                }
                if (grp == 0 && g == 0)
                    p.lse_part[row] = lse_row;
            }
        } else {
            unsigned char *stage = smem + T::XCH_STAGE + wave_wg * 32 * HROWB;   // as in finish: whole rows out
#pragma unroll
            for (int i = 0; i < 4 * HB; ++i) {
                const f32x16 &x = o_half[i / 4];
                const int r = 4 * (i % 4);
                const f32x2 lo = {x[r], x[r + 1]}, hi = {x[r + 2], x[r + 3]};
                const typename E::x2 blo = __builtin_convertvector(lo, typename E::x2);  // round to nearest even
                const typename E::x2 bhi = __builtin_convertvector(hi, typename E::x2);
                const typename E::x4 out = {blo[0], blo[1], bhi[0], bhi[1]};
                *reinterpret_cast<typename E::x4 *>(stage + lq * HROWB + ((i ^ (lq & (HCPR - 1))) * 16) + g * 8) = out;
            }
            elem_t *o_blk = reinterpret_cast<elem_t *>(p.o) + ((size_t)t.bh * p.S_q + row0) * D + grp * (D / 2);
            const int rows_left = p.S_q - row0;
#pragma unroll
            for (int i = 0; i < 32 * HCPR / 64; ++i) {
                const int idx = i * 64 + lane;
                const int r = idx / HCPR, c = idx % HCPR;
                const u32x4 w = *reinterpret_cast<const u32x4 *>(stage + r * HROWB + ((c ^ (r & (HCPR - 1))) * 16));
                if (r < rows_left)
                    *reinterpret_cast<u32x4 *>(o_blk + (size_t)r * D + c * 8) = w;
            }
            if (qrow < p.S_q && grp == 0 && g == 0)
                p.lse[(size_t)t.bh * p.S_q + qrow] = lse_row;
        }
        ATTN_TRACE(p, t.vb, 5);
    };
    // between(k), k = 0 .. 2 QB - 1: called after each block's conversion and after each block's stores
    auto finish = [&](const Tile &t, auto between) {
        if constexpr (G == 2) {
            finish_groups(t);
            return;
        }
        if constexpr (T::PAIRED) {
            // the paired loop leaves few registers for what lives across it: the addresses of this part are made from a
            // lane number that the compiler cannot see is the same for every tile
            asm volatile("" : "+v"(lane));
            lq = lane & 31;
            g = lane >> 5;
        }
        float inv[QB], lse_row[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float l_lane = F32Vec<QB>::get(l_run_v, qb);
            const float l_tot = l_lane + xor32(l_lane);
            inv[qb] = 1.f / l_tot;
            lse_row[qb] = F32Vec<QB>::get(m_ref_v, qb) * p.scale + __builtin_amdgcn_logf(l_tot) * 0.69314718055994530942f;
        }
        if constexpr (SPLIT) {
            const size_t n_rows = (size_t)(p.total_wg / (p.n_qt * p.n_split)) * p.S_q;
            if constexpr (T::WHOLE_PARTS) {
                // whole rows through LDS, as below: 32 fp32 rows of a wave at a time, in the rings
                constexpr int FCPR = D / 4, FROWB = D * 4;   // 16-byte chunks, bytes of a row
                static_assert(NW * 32 * FROWB <= T::RING_BYTES, "the partial rows are staged in the rings");
                unsigned char *stage = o_stage + wave * 32 * FROWB;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int rb = 0; rb < 4; ++rb) {
                            const f32x16 &oa = o_acc[qb * DB + db];
                            const f32x4 w = {oa[4 * rb + 0] * inv[qb], oa[4 * rb + 1] * inv[qb], oa[4 * rb + 2] * inv[qb],
                                             oa[4 * rb + 3] * inv[qb]};
                            const int chunk = (8 * db + 2 * rb + g) ^ (lq & (FCPR - 1));
                            *reinterpret_cast<f32x4 *>(stage + lq * FROWB + chunk * 16) = w;
                        }
                    const int row0 = t.q0 + (wave * QB + qb) * 32;
                    const int rows_left = p.S_q - row0;
                    const size_t first = (size_t)t.split * n_rows + (size_t)t.bh * p.S_q + row0;
                    float *blk = p.o_part + first * D;
#pragma unroll
                    for (int i = 0; i < 32 * FCPR / 64; ++i) {
                        const int idx = i * 64 + lane;
                        const int r = idx / FCPR, c = idx % FCPR;
                        const f32x4 w = *reinterpret_cast<const f32x4 *>(stage + r * FROWB + ((c ^ (r & (FCPR - 1))) * 16));
                        if (r < rows_left)
                            *reinterpret_cast<f32x4 *>(blk + (size_t)r * D + c * 4) = w;
                    }
                    if (lq < rows_left && g == 0)
                        p.lse_part[first + lq] = lse_row[qb];
                }
                return;
            }
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int qrow = qcol(t, qb);
                if (qrow >= p.S_q)
                    continue;
                const size_t row = (size_t)t.split * n_rows + (size_t)t.bh * p.S_q + qrow;
                float *orow = p.o_part + row * D;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb) {
                        const f32x16 &oa = o_acc[qb * DB + db];
                        const f32x4 w = {oa[4 * rb + 0] * inv[qb], oa[4 * rb + 1] * inv[qb], oa[4 * rb + 2] * inv[qb],
                                         oa[4 * rb + 3] * inv[qb]};
                        *reinterpret_cast<f32x4 *>(orow + 32 * db + 8 * rb + 4 * g) = w;
                    }
                if (g == 0)
                    p.lse_part[row] = lse_row[qb];
            }
        } else {
            // O goes through LDS so that it leaves in whole rows: a lane holds 4-element pieces of ONE row,
            // stored directly a wave-wide store would touch 32 rows with 16 bytes each.  Every 32-row block
            // has its own 32 x ROWB bytes of the staging area (a wave reads back only what it wrote: no
            // barrier in between); rows are XOR-swizzled by 16-byte chunk.
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                unsigned char *stage = o_stage + (wave * QB + qb) * 32 * ROWB;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb) {
                        const f32x16 &oa = o_acc[qb * DB + db];
                        const f32x2 lo = {oa[4 * rb + 0] * inv[qb], oa[4 * rb + 1] * inv[qb]};
                        const f32x2 hi = {oa[4 * rb + 2] * inv[qb], oa[4 * rb + 3] * inv[qb]};
                        const typename E::x2 blo = __builtin_convertvector(lo, typename E::x2);  // round to nearest even
                        const typename E::x2 bhi = __builtin_convertvector(hi, typename E::x2);
                        const typename E::x4 out = {blo[0], blo[1], bhi[0], bhi[1]};
                        const int chunk = (4 * db + rb) ^ (lq & (CPR - 1));
                        *reinterpret_cast<typename E::x4 *>(stage + lq * ROWB + chunk * 16 + g * 8) = out;
                    }
                between(qb);
            }
            ATTN_TRACE(p, t.vb, 4);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const unsigned char *stage = o_stage + (wave * QB + qb) * 32 * ROWB;
                const int row0 = t.q0 + (wave * QB + qb) * 32;
                elem_t *o_blk = reinterpret_cast<elem_t *>(p.o) + ((size_t)t.bh * p.S_q + row0) * D;
                const int rows_left = p.S_q - row0;  // rows of this block that exist
#pragma unroll
                for (int i = 0; i < 32 * CPR / 64; ++i) {
                    const int idx = i * 64 + lane;
                    const int r = idx / CPR, c = idx % CPR;
                    const u32x4 w = *reinterpret_cast<const u32x4 *>(stage + r * ROWB + ((c ^ (r & (CPR - 1))) * 16));
                    if (r < rows_left)
                        *reinterpret_cast<u32x4 *>(o_blk + (size_t)r * D + c * 8) = w;
                }
                const int qrow = qcol(t, qb);
                if (qrow < p.S_q && g == 0)
                    p.lse[(size_t)t.bh * p.S_q + qrow] = lse_row[qb];
                between(QB + qb);
            }
        }
        ATTN_TRACE(p, t.vb, 5);
    };

    // ---- the work on one tile between its loads and its epilogue
    auto run_tile = [&](const Tile &t) {
#pragma unroll
        for (int i = 0; i < QB * DB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                o_acc[i][r] = 0.f;
        wait_vmcnt<5 * NLD>();  // K(0) and Q have landed; the five tiles behind them may be in flight
        ex8 bq[QB][KS];
        if constexpr (!HAS_STAGE) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    asm volatile("" : "+v"(q_raw[qb][ks]));  // every use of Q stays behind the wait
                    bq[qb][ks] = __builtin_bit_cast(ex8, q_raw[qb][ks]);
                }
        }
        __builtin_amdgcn_s_barrier();  // every wave's part of K(0) (and of Q) is in LDS
        asm volatile("" ::: "memory");  // no LDS read of the compiler's moves above the barrier
        if constexpr (HAS_STAGE) {
            // this lane's query row as MFMA B operand: the K fragment addressing, in the staging area
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int blk = wave * QB + qb;  // 32-row block of the tile
                const uint32_t off = STAGE - KRING + (blk / SB) * TB + (blk % SB) * 32 * ROWB;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    bq[qb][ks] = *(ATTN_LDS_PTR(const ex8))(uintptr_t)(koff[ks] + off);
            }
        }
        ATTN_TRACE(p, t.vb, 1);

        // S(0) = K(0) Q^T
        f32x16 s_init[QB * SB];
#pragma unroll
        for (int i = 0; i < QB * SB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                s_init[i][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) {
                const ex8 a = *(ATTN_LDS_PTR(const ex8))(uintptr_t)((T::PAIRED ? koff_v[ks] : koff[ks]) + sb * 32 * ROWB);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    s_init[qb * SB + sb] = E::mfma(a, bq[qb][ks], s_init[qb * SB + sb]);
            }

        typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
        u32x16 q_pack[NQP];
#pragma unroll
        for (int i = 0; i < NQP; ++i) {
            struct Four {
                ex8 a[4];
            } f;
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4)
                f.a[k4] = bq[(4 * i + k4) / KS][(4 * i + k4) % KS];
            q_pack[i] = __builtin_bit_cast(u32x16, f);
        }
        // Second key group: a wave none of whose rows sees a key of the group (causal; its rows and the group's keys
        // both start at multiples of 32), or a tile too short for two groups: it runs one tile, and its result does not
        // count
        const int last_row = min(t.q0 + (wave + 1) * 32 * QB, p.S_q) - 1;
        if constexpr (G == 2)
            idle = grp && (t.kv0 == (SPLIT ? t.split * p.split_len : 0) ||
                           (CAUSAL && min(t.q0 + wave * 32, last_row) < t.kv0));
        // key index limit of this lane's queries, minus the lane-group part of the accumulator row
        typename U32Vec<QB>::type thr_base_v;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
            U32Vec<QB>::set(thr_base_v, qb,
                            (uint32_t)((CAUSAL ? min(qcol(t, qb) - t.kv0, t.skv_m1) : t.skv_m1) - 4 * g));
        const float c_log2e = p.c;
        const elem_t *k_head = t.k_head, *v_head = t.v_head;
        const int n_tiles = t.n_tiles, j_mask = t.j_mask, t_full = t.t_full, skv_m1 = t.skv_m1;
        // causal: the keys behind this wave's last row are masked for all of its rows; the loop leaves the
        // tiles that hold nothing else to the waves below (it keeps their barriers and issues its loads)
        // a wave without a row below S_q writes nothing: after one tile it only keeps step (barriers, its share of the
        // loads) and leaves the LDS port and the power to the others, in launches where that pays (idle_row in attn_fwd.hip)
        // (a pair of waves has rows or has none: either needs the other's row sums)
        const bool no_rows = G == 1 && !(CAUSAL && D == 64 && NW == 4) &&
                             t.q0 + (T::PAIRED ? wave & ~1 : wave) * 32 * QB >= (CAUSAL ? p.S_q : p.idle_row);
        const int n_tiles_wave =
            idle || no_rows ? 1 : (CAUSAL ? min(t.own_tiles, (last_row - t.kv0) / BN + 1) : t.own_tiles);
        // this lane's place for its tile row sums and the other wave's
        [[maybe_unused]] const uint32_t xch_own = lds0 + T::XCH_SUMS + (wave * 64 + lane) * 4;
        [[maybe_unused]] const uint32_t xch_other = lds0 + T::XCH_SUMS + ((wave ^ 1) * 64 + lane) * 4;
        ATTN_TRACE(p, t.vb, 2);

        if constexpr (T::PAIRED && !F16) {
#include "generated/attn_loop_d128_w4.inc"
        } else if constexpr (T::PAIRED) {
#include "generated/attn_loop_d128_w4_f16.inc"
        } else if constexpr (D == 128 && SB == 2 && !F16) {
#include "generated/attn_loop_d128.inc"
        } else if constexpr (D == 128 && SB == 2 && F16) {
#include "generated/attn_loop_d128_f16.inc"
        } else if constexpr (D == 128 && QB == 2 && NW == 2 && !F16) {
#include "generated/attn_loop_d128a_w2.inc"
        } else if constexpr (D == 128 && QB == 2 && NW == 2) {
#include "generated/attn_loop_d128a_w2_f16.inc"
        } else if constexpr (D == 128 && QB == 2 && !F16) {
#include "generated/attn_loop_d128a.inc"
        } else if constexpr (D == 128 && QB == 2 && F16) {
#include "generated/attn_loop_d128a_f16.inc"
        } else if constexpr (D == 128 && !F16) {
#include "generated/attn_loop_d128_w2.inc"
        } else if constexpr (D == 128) {
#include "generated/attn_loop_d128_w2_f16.inc"
        } else if constexpr (D == 64 && NW == 4 && !F16) {
#include "generated/attn_loop_d64_w4.inc"
        } else if constexpr (D == 64 && NW == 4) {
#include "generated/attn_loop_d64_w4_f16.inc"
        } else if constexpr (D == 64 && NW == 2 && !F16) {
#include "generated/attn_loop_d64_w2.inc"
        } else if constexpr (D == 64 && NW == 2) {
#include "generated/attn_loop_d64_w2_f16.inc"
        } else if constexpr (D == 64 && !F16) {
#include "generated/attn_loop_d64.inc"
        } else if constexpr (D == 64 && F16) {
#include "generated/attn_loop_d64_f16.inc"
        } else if constexpr (D == 256 && !F16) {
#include "generated/attn_loop_d256a.inc"
        } else {
#include "generated/attn_loop_d256a_f16.inc"
        }
        ATTN_TRACE(p, t.vb, 3);
        __syncthreads();  // every wave has left the loop: the rings are free
    };
    auto trace_start = [&](const Tile &t) {
        ATTN_TRACE(p, t.vb, 0);
        ATTN_TRACE_VALUE(p, t.vb, 7, ((unsigned long long)__builtin_amdgcn_s_getreg((31 << 11) | 20) << 32) |   // XCC_ID
                                         __builtin_amdgcn_s_getreg((31 << 11) | 4));                             // HW_ID
        (void)t;
    };

    // the first tile (pass 0 has an entry for every slot), then the queue: only the last pass can be short
    Tile cur = locate(virtual_wg(0));
    trace_start(cur);
    issue_loads(cur, std::true_type{});
    ATTN_TRACE(p, cur.vb, 6);
#pragma clang loop unroll(disable)
    for (int pass = 1;; ++pass) {
        run_tile(cur);
        auto nothing = [](int) {};
        if constexpr (!HAS_STAGE)
            finish(cur, nothing);
        const int vb = pass < n_pass ? virtual_wg(pass) : -1;
        if constexpr (HAS_STAGE) {
            if (vb < 0) {
                finish(cur, nothing);
                break;
            }
            // The staging area is free (every wave took its Q fragments out of it before the loop): the next
            // tile's Q rows travel while the finished tile is normalised, staged in the rings and stored.  Their
            // loads go out in parts between the steps of that work: they miss every cache, and a wave that
            // issues all of them in a row waits for the address unit to take them.
            const Tile nxt = locate(vb);
            finish(cur, [&](int k) { issue_q_part(nxt, k); });
            cur = nxt;
        } else {
            if (vb < 0)
                break;
            cur = locate(vb);
        }
        trace_start(cur);
        __syncthreads();  // every wave has read its staged rows back: the rings are free
        issue_loads(cur, std::integral_constant<bool, !HAS_STAGE>{});
        ATTN_TRACE(p, cur.vb, 6);
    }
}

}  // namespace attn
