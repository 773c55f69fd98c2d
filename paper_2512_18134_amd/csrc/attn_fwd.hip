// attn_fwd.hip -- C ABI of libmi355attn.so (see include/attn_fwd.h) and kernel dispatch.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "attn_fwd.h"
#include "attn_fwd_asm.h"
#include "attn_fwd_simple.h"
#include "attn_launch.h"
#ifdef ATTN_DEBUG_ENTRY_POINTS
#include "attn_probe.h"
#endif
#include "attn_splitkv.h"

namespace {

using attn::Params;

using attn::allow_lds;

// Params::idle_row of a launch.  A wave without a row below S_q (at D = 128 in pairs: a pair without one) that stops after its
// first K/V tile leaves the LDS port and the power to the others, but it leaves the loop by code that the others do not
// run: 0.1 to 0.3 us of instruction fetches, which a short walk does not win back.  Measured without / with, us: D = 64,
// where it is never slower, 512 heads of 300 rows 36.0 / 32.1, 600 heads against 96 keys 27.9 / 26.2; D = 256, 512 of 300 119
// / 113, 600 of 300 rows and 128 keys 75.4 / 76.0, 256 keys 116 / 111, and where all waves but one have no row, 64 heads of 5
// rows, 64 keys 7.6 / 7.7, 135 keys 10.1 / 9.9, 700 keys 18.7 / 18.1.  D = 128, in pairs, 200 heads of 70 rows, 64 keys 5.66 / 5.68, 256
// keys 8.85 / 8.85, 600 of 300 rows and 128 keys 32.5 / 32.2; over 260 launches it is level up to 256 keys and 0.3 to 1.1 %
// ahead beyond with up to 256 tiles, 0.6 to 2.5 % ahead at any length with more than 512.  (The 64-row waves of that size, 200
// heads of 70 rows, 64 keys 7.7 / 7.9, 700 keys 20.4 / 19.0; 128 of 520 rows 35.0 / 33.5.)  Causal: the last query tile
// of a head, which has these waves, walks the most keys (D = 128, in pairs, 128 heads of 520 rows 23.2 / 22.4; 4 of 70 rows 5.64 /
// 5.65; over 300 launches it is level to 2 % ahead), so that these launches always do it (one more argument costs their
// crowded scalar registers as much as it brings), but for the 4-wave D = 64 ones, which never do: 1 head of 192 rows 5.6 /
// 5.8, 32 of 600 rows 9.9 / 10.1, 100 of 256 rows 7.3 / 7.4, 400 of 777 rows 76.7 / 75.5.
int idle_row(const Params &p, int D, long long tiles)
{
    const bool soon = D == 64 || (D == 128 && tiles > 512) || (D == 256 && p.S_q <= 64);
    const int pays_from = soon ? 65 : tiles >= 128 ? 129 : 512;   // keys
    return p.S_kv >= pays_from ? p.S_q : 0x7fffffff;
}

// persistent: as many workgroups as the chip holds at once, each walking the tile queue of its XCD
// (attn_fwd_asm_kernel); otherwise one workgroup per tile
template <typename K>
int launch(K kern, Params p, int BH, int BM, int threads, int lds_bytes, hipStream_t stream, bool persistent = false)
{
    p.n_qt = (p.S_q + BM - 1) / BM;
    const long long total = (long long)BH * p.n_qt;
    if (total > 0x7fffffffLL)
        return ATTN_ERR_SHAPE;
    p.total_wg = (int)total;
    if (!allow_lds(reinterpret_cast<const void *>(kern), lds_bytes))
        return ATTN_ERR_LAUNCH;
    int grid = p.total_wg;
    const int cus = attn::cu_count(attn::kNumXcd);
    p.cus_per_xcd = cus > 0 ? cus / attn::kNumXcd : 32;
    if (persistent) {
        // (a runtime that cannot tell the occupancy gets one workgroup per tile: the kernel takes either)
        const int slots = attn::persistent_slots(reinterpret_cast<const void *>(kern), threads, lds_bytes, attn::kNumXcd);
        if (slots >= attn::kNumXcd && slots < grid)
            grid = slots;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds_bytes, stream, p);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}

template <int D, int BN, int NW>
int launch_simple(const Params &p, int BH, int causal, hipStream_t stream)
{
    constexpr int LDS = 4 * BN * D * 2;
    if (causal)
        return launch(attn::attn_fwd_simple_kernel<D, BN, NW, true>, p, BH, NW * 32, NW * 64, LDS, stream);
    return launch(attn::attn_fwd_simple_kernel<D, BN, NW, false>, p, BH, NW * 32, NW * 64, LDS, stream);
}

// one hand-scheduled tiling: QB 32-row query blocks per wave, SB 32-key blocks per K/V tile, NW waves; persistent
// workgroups where the tiling has them
template <int D, int QB, int SB, int NW, bool F16 = false, int G = 1>
int launch_asm(Params p, int BH, int causal, hipStream_t stream)
{
    typedef attn::FwdTiling<D, QB, SB, NW, false, G> T;
    p.idle_row = idle_row(p, D, (long long)BH * ((p.S_q + T::BM - 1) / T::BM));
    if (causal)
        return launch(attn::attn_fwd_asm_kernel<D, QB, SB, NW, true, F16, false, G>, p, BH, T::BM, T::THREADS, T::LDS_BYTES,
                      stream, T::PERSIST);
    return launch(attn::attn_fwd_asm_kernel<D, QB, SB, NW, false, F16, false, G>, p, BH, T::BM, T::THREADS, T::LDS_BYTES,
                  stream, T::PERSIST);
}

// Below this many queries a launch may use the tilings whose keys are shared out between two groups of waves.  They
// cut the serial walk over the keys in half (D = 128, one query: 8 heads of 1024 keys 22.1 -> 10.6 us, 64 heads of
// 4096 keys 70.5 -> 27.7 us) but add up in another order, and each group rounds P to 16 bits against a reference of its
// own: O moves by up to 3e-3 of its norm in bf16 (64 heads of one query and 8191 keys), which is the rounding of its P and
// of itself, and the dQ that attn_bwd computes from such an O by 2e-2 when the softmax is nearly one-hot (dO . O cancels
// there).  Neither is further from the exact result than one walk's (240 forward + backward calls with 1 to 63 queries,
// bf16, rms: O 2.1e-3, dQ of peaked rows 2.4e-2, either way).  The line is a choice: calls with fewer queries, training
// calls among them, have this order, all others the one that they share with the wide tilings, bit for bit.
constexpr int kKeyGroupMaxQueries = 64;

// D = 64: what a launch of one tiling costs, in us, fitted to launches of one kernel on 1 to 2000 heads of 1 to 16384
// rows (within 10 % where two tilings are close).  `start` for every round of query tiles that a compute unit works
// through (`wgs` workgroups that share a unit overlap theirs; `start_shared` where they do), and `per_tile` for every
// 64-key tile of the query tile with the most of them.  Not causal: a last round that leaves most units idle runs at a
// higher clock.  Causal: heavy and light tiles are handed out in pairs, so that r rounds cost 0.6 r times the heaviest
// tile.
struct Tiling {
    int rows, wgs;
    float start, start_shared, per_tile, per_tile_causal;
};

float tiling_cost(const Tiling &t, int BH, const Params &p, int causal, int cus)
{
    const long long tiles = (long long)BH * ((p.S_q + t.rows - 1) / t.rows);
    const int keys = causal && p.S_q < p.S_kv ? p.S_q : p.S_kv;
    const float n = (float)((keys + 63) / 64);
    const float whole = (float)(tiles / cus), rest = (float)(tiles % cus) / (float)cus;
    const float up = whole + (rest > 0.f ? 1.f : 0.f);   // rounds, the last one counted in full
    if (!causal)
        return (up > 1.f ? t.start_shared * fmaxf(1.f, up / t.wgs) : t.start) + t.per_tile * n * (whole + (rest > 0.f ? 0.65f + 0.35f * rest : 0.f));
    const float r = fmaxf(1.f, 0.5f * (whole + rest + up));
    return t.start * fmaxf(1.f, r / t.wgs) + t.per_tile_causal * n * fmaxf(0.7f + 0.17f * r, 0.6f * r);
}

// Causal launches of 64 queries and more take the 128-row tiling up to 4096 keys, whatever the estimates say: over 876
// launches of 1 to 1024 heads it is 20 % faster than the 256-row one on average, by up to 23 % where that one's last
// round is nearly empty (256 heads of 567 rows 33.8 / 28.7, 96 of 1579 57.3 / 48.8, 128 of 1100 42.4 / 35.4), and slower
// by more than 2 % in six of them, 5.6 % at worst (128 heads of 5504 rows and 576 keys 136.7 / 144.4).  Without a mask
// the 256-row tiling wins wherever it needs as many rounds (96 heads of 320 rows 9.3 / 9.6, 64 of 520 12.3 / 13.0, 64 of
// 777 16.3 / 16.7), and beyond two rounds of its tiles, unless most of their rows do not exist.
int choose_d64(int BH, const Params &p, int causal)
{
    if (causal && p.S_q >= kKeyGroupMaxQueries && p.S_kv <= 4096)
        return 1;
    const int cus = attn::cu_count(1) > 0 ? attn::cu_count(1) : 256;
    // (two 128-row workgroups on a unit stream twice the keys per product of a 256-row one: with a causal mask
    // that shows from long sequences on)
    const Tiling t[3] = {{256, 1, 5.0f, 5.0f, 0.90f, 0.95f},
                         {128, 2, 4.0f, 5.2f, 0.52f, p.S_kv > 4096 ? 0.60f : 0.54f},
                         {64, 1, 4.5f, 4.5f, 0.31f, 0.31f}};
    float best = tiling_cost(t[0], BH, p, causal, cus);
    int tiling = 0;
    const bool wide = p.S_q > 128 && (long long)BH * ((p.S_q + 255) / 256) > 2ll * cus;
    for (int i = 1; i < (wide ? 1 : (p.S_q < kKeyGroupMaxQueries ? 3 : 2)); ++i) {
        const float c = tiling_cost(t[i], BH, p, causal, cus);
        if (c < best) {
            best = c;
            tiling = i;
        }
    }
    return tiling;
}

// D = 64.  tiling: -1 = choose, 0 = 8 waves x 32 rows (two waves per SIMD), 1 = 4 waves x 32 rows (two workgroups
// per CU; the same results), 2 = 2 x 2 waves x 32 rows (64 rows, two key groups).
// Measured, us for tiling 0 / 1: 16 heads of 512 rows 10.6 / 7.8, of 2048 rows 28.6 / 20.8; 32 heads of 2048 rows
// 35.9 / 37.4, causal 31.3 / 25.9; 64 heads of 4096 rows 256 / 267; 2000 heads of 100 rows 40.3 / 24.4.
template <bool F16>
int launch_d64(const Params &p, int BH, int causal, hipStream_t stream, int tiling = -1)
{
    if (tiling < 0)
        tiling = choose_d64(BH, p, causal);
    if (tiling == 2)
        return launch_asm<64, 1, 2, 2, F16, 2>(p, BH, causal, stream);
    if (tiling == 1)
        return launch_asm<64, 1, 2, 4, F16>(p, BH, causal, stream);
    return launch_asm<64, 1, 2, 8, F16>(p, BH, causal, stream);
}

// D = 128: the same estimate for the 256-row tiling (one workgroup per CU) and the 128-row one (two).  A CU with a single
// 128-row workgroup walks a tile's keys at 0.6 us per 32 of them, 0.64 without a mask.  Causal: the sum of the tiles' keys, ragged last
// tiles included, or the walk of the tile with the most of them in an otherwise idle chip, whichever is longer.
// (Launches with at most one 128-row tile per CU take neither: paired_pays.)
float d128_cost(int rows, int BH, const Params &p, int causal, int cus)
{
    const bool two = rows == 128;
    const long long nt = (p.S_q + rows - 1) / rows, tiles = (long long)BH * nt, slots = (two ? 2ll : 1ll) * cus;
    const long long n = ((causal && p.S_q < p.S_kv ? p.S_q : p.S_kv) + 31) / 32;
    const float whole = (float)(tiles / slots), rest = (float)(tiles % slots) / (float)slots;
    if (!causal) {
        const float start = two ? 8.5f : 6.0f, per_tile = two ? 0.86f : 0.80f;
        const float last = two ? (rest > 0.5f ? 0.83f : 0.64f) : per_tile * (0.65f + 0.35f * rest);
        return whole * (start + per_tile * n) + (rest > 0.f ? start + last * n : 0.f);
    }
    const long long step = rows / 32, k = nt < n / step ? nt : n / step;   // tiles below the last keys
    const float sum = (float)(step * k * (k + 1) / 2 + (nt - k) * n);
    const float start = two ? 7.0f : 6.0f, r = fmaxf(1.f, whole + 0.5f * (rest + (rest > 0.f ? 1.f : 0.f)));
    return fmaxf(start + 0.60f * n, start * r + (two ? 0.83f : 0.72f) * sum * BH / (float)slots);
}

// 64 queries and more: the better one of the two tilings of 64-row waves
int choose_d128(int BH, const Params &p, int causal, float *cost = nullptr)
{
    const int cus = attn::cu_count(1) > 0 ? attn::cu_count(1) : 256;
    const float narrow = d128_cost(128, BH, p, causal, cus), wide = d128_cost(256, BH, p, causal, cus);
    const bool two = narrow < (causal ? 1.f : 0.99f) * wide;
    if (cost)
        *cost = two ? narrow : wide;
    return two ? 3 : 1;
}

// D = 128, 64 queries and more: the 128-row tiling of 32-row waves that move their references in pairs.  A wave has half the
// products and half the softmax of a 64-row one, so that the walk over the keys is shorter wherever the launch does not
// fill the chip's SIMDs twice over; it reads twice the LDS operands per product, so that full launches stay with 64-row
// waves (two workgroups of either kind share a CU's matrix pipes: 0.84 us per 32 keys, where a 256-row one takes 0.80).
// us, best tiling of 64-row waves / paired: 16 heads of 128 rows 9.5 / 7.4, of 777 rows, causal, 20.5 / 14.4, of 1024 23.2 /
// 15.8; 32 of 2048, causal, 48.1 / 38.0; 4 of 6000, causal, 98.8 / 70.4; 1 of 16384, causal, 255 / 171; 16 of 2048 41.7 /
// 34.6; 24 of 2816 122 / 115; but 6 of 5468 93 / 120, 128 of 2048 223 / 244, 32 of 4096, causal, 117 / 131.
// Up to one tile per CU it is always ahead (by 10 to 34 % over 950 launches).  Where the 256-row tiling needs one round and
// more 128-row tiles than CUs walk all keys (no mask, or more queries than keys), it is behind from some 500 keys on, by 5
// to 28 %: 87 heads of 344 queries and 2557 keys 47.9 / 59.3, 96 of 320 and 4494 82.5 / 101, causal 6 of 8256 and 2233 50.3 /
// 58.2, 8 of 6643 and 1856 45.5 / 51.1; with fewer keys up to 5 % either way.  Otherwise a CU's second workgroup halves the
// speed of both, so that the line is an estimate again, fitted over 1800 launches of 1 to 600 heads.  Not causal: rounds of
// two tiles per CU, of which the last walks faster where most CUs have one tile or none; heads of a single query tile
// stay out, whose keys come from memory once per workgroup (310 heads of 112 queries and 960 keys 33.8 / 39.7).  Causal: heavy
// and light tiles share a CU and it is ahead (by 14 % on average over 592 launches) up to 2 1/4 tiles per CU.  Up to 1024
// keys the second workgroup on a CU hides the start of every tile, which counts the less the more 32-key steps a workgroup
// walks in all (`per_slot`).  Over 8000 such launches of up to 16000 tiles it is 11 to 13 % ahead up to 20 steps and 7 % at 20
// to 36.  With more than twice as many queries as keys: 4 % ahead at 36 to 60, 2 % at 60 to 110, level at 110 to 160 (146 heads
// of 5519 queries and 361 keys 216 / 212), and 2 to 3 % behind beyond (71 of 7215 and 844 221 / 236, 155 of 10560 and 951
// 782 / 849), which is where the line lies.  With fewer queries it is 1.5 % ahead at 36 to 60 steps and 2 % behind to 2 %
// ahead beyond, but one launch 7 % ahead and the next 8 % behind, by how the queues happen to fall (757 heads of 655 queries and
// 1307 keys 173 / 171, 601 of 755 rows 159 / 145, 495 of 939 and 1790 180 / 215): a line at 80 steps makes 520
// of the 8000 more than 2 % faster and 303 slower, and sizes, remainders and the queues' longest walk tell them apart no
// better than that, so that there is none.  Longer walks: the better of the others has its balance to
// win or lose (32 heads of 3845 rows 107 / 149).
bool paired_pays(int BH, const Params &p, int causal, int cus, float others)
{
    const long long nt = (p.S_q + 127) / 128, tiles = BH * nt, slots = 2ll * cus;
    const long long n = ((causal && p.S_q < p.S_kv ? p.S_q : p.S_kv) + 31) / 32;
    const long long k = causal ? (nt < n / 4 ? nt : n / 4) : 0;   // tiles below the last keys
    if (n > 16 && BH * (nt - k) > cus && (long long)BH * ((p.S_q + 255) / 256) <= cus)
        return false;
    if (4 * tiles <= (causal ? 9 : 4) * cus)
        return true;
    const float whole = (float)(tiles / slots), rest = (float)(tiles % slots) / (float)slots;
    if (!causal) {
        if (nt == 1 && n >= 16)
            return false;
        const float last = rest > 0.5f ? 7.8f + (0.63f + 0.43f * (rest - 0.5f)) * n : rest > 0.f ? 5.0f + (0.31f + 0.29f * rest) * n : 0.f;
        return whole * (5.5f + 0.84f * n) + last < 0.95f * others;
    }
    const float per_slot = (float)(2 * k * (k + 1) + (nt - k) * n) * BH / (float)slots;
    if (n <= 32)
        return p.S_q <= 2ll * p.S_kv || per_slot <= 160.f;
    const float r = fmaxf(1.f, whole + 0.5f * (rest + (rest > 0.f ? 1.f : 0.f)));
    return fmaxf(5.9f + 0.39f * n, 7.0f * r + 0.873f * per_slot + 0.056f * n) < 1.04f * others;
}

int choose_d128_all(int BH, const Params &p, int causal)
{
    const int cus = attn::cu_count(1) > 0 ? attn::cu_count(1) : 256;
    float others;
    const int tiling = choose_d128(BH, p, causal, &others);
    return paired_pays(BH, p, causal, cus, others) ? 4 : tiling;
}

// D = 128.  tiling: -1 = choose, 0 = 8 waves x 32 rows (two waves per SIMD), 1 = 4 waves x 64 rows (one wave
// per SIMD, half the LDS operand reads per MFMA), 2 = 2 x 2 waves x 32 rows (64 rows, two key groups), 3 = 2 waves x 64
// rows (two workgroups per CU; the same results as 1), 4 = 4 waves x 32 rows in pairs (two per CU; the same results as 1).
// Measured, us for tiling 1 / 3 / 4: 96 heads of 640 queries and 2578 keys 112 / 74 / 80; 160 of 320 queries and 7680 keys 280 /
// 198 / 215; causal: 244 of 1088 rows 124 / 109 / 114, 202 of 1871 245 / 206 / 220.  Full rounds of full tiles stay with
// tiling 1: 32 heads of 4096 rows 209 / 222 / 233, causal 116 / 121 / 126.
template <bool F16>
int launch_d128(const Params &p, int BH, int causal, hipStream_t stream, int tiling = -1)
{
    if (tiling < 0)
        tiling = p.S_q < kKeyGroupMaxQueries ? 2 : choose_d128_all(BH, p, causal);
    switch (tiling) {
    case 0:
        return launch_asm<128, 1, 2, 8, F16>(p, BH, causal, stream);
    case 2:
        return launch_asm<128, 1, 1, 2, F16, 2>(p, BH, causal, stream);
    case 3:
        return launch_asm<128, 2, 1, 2, F16>(p, BH, causal, stream);
    case 4:
        return launch_asm<128, 1, 1, 4, F16>(p, BH, causal, stream);
    default:
        return launch_asm<128, 2, 1, 4, F16>(p, BH, causal, stream);
    }
}

// the generic kernel: any scale, heads of any size, program order
int launch_generic(const Params &p, int BH, int D, int causal, hipStream_t st)
{
    switch (D) {
    case 64:
        return launch_simple<64, 64, 8>(p, BH, causal, st);
    case 128:
        return launch_simple<128, 64, 8>(p, BH, causal, st);
    default:
        return launch_simple<256, 32, 4>(p, BH, causal, st);
    }
}

// bf16 dispatch.  The hand-scheduled loops set masked scores to -inf before the multiply by
// scale*log2e (they need scale > 0) and address K/V of one head with 32-bit byte offsets.
int dispatch_fwd(const Params &p, int BH, int D, int causal, hipStream_t st)
{
    const bool asm_ok = p.scale > 0.f && (long long)p.S_kv * D * 2 < (1LL << 31);
    if (!asm_ok)
        return launch_generic(p, BH, D, causal, st);
    switch (D) {
    case 64:
        return launch_d64<false>(p, BH, causal, st);
    case 128:
        return launch_d128<false>(p, BH, causal, st);
    default:
        return launch_asm<256, 1, 1, 4>(p, BH, causal, st);
    }
}

}  // namespace

// host-side validation shared by the entry points; fills `p` on success
static int validate(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int S_q, int S_kv,
                    int D, float scale, Params &p)
{
    if (!q || !k || !v || !o || !lse)
        return ATTN_ERR_NULL;
    if (B < 1 || H < 1 || S_q < 1 || S_kv < 1)
        return ATTN_ERR_SHAPE;
    if (D != 64 && D != 128 && D != 256)
        return ATTN_ERR_UNSUPPORTED_D;
    const long long BH = (long long)B * H;
    if (BH > 0x7fffffffLL || BH * (long long)(S_q > S_kv ? S_q : S_kv) > (1LL << 40) / D)
        return ATTN_ERR_SHAPE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15)
        return ATTN_ERR_ALIGN;
    if ((uintptr_t)lse & 3)
        return ATTN_ERR_ALIGN;
    if (!(scale >= 0.f) || isinf(scale))
        return ATTN_ERR_SCALE;
    p.q = static_cast<const attn::bf16_t *>(q);
    p.k = static_cast<const attn::bf16_t *>(k);
    p.v = static_cast<const attn::bf16_t *>(v);
    p.o = static_cast<attn::bf16_t *>(o);
    p.lse = lse;
    p.S_q = S_q;
    p.S_kv = S_kv;
    p.n_qt = 0;
    p.total_wg = 0;
    p.c = scale * 1.44269504088896340736f;
    p.scale = scale;
    p.idle_row = 0;
    p.cus_per_xcd = 0;
    p.n_split = 1;
#ifdef ATTN_DEBUG_ENTRY_POINTS
    p.trace = nullptr;
    p.trace_entries = 0;
#endif
    p.split_len = 0;
    p.o_part = nullptr;
    p.lse_part = nullptr;
    return ATTN_OK;
}

// key range of one split: a multiple of the 64-key tile; returns the number of non-empty ranges
static int split_plan(int S_kv, int n_split, int &split_len)
{
    const int per = (S_kv + n_split - 1) / n_split;
    split_len = (per + 63) / 64 * 64;
    return (S_kv + split_len - 1) / split_len;
}

extern "C" long long attn_fwd_splitkv_workspace_bytes(int B, int H, int S_q, int D, int n_split)
{
    if (B < 1 || H < 1 || S_q < 1 || n_split < 1 || n_split > 256 || (D != 64 && D != 128))
        return -1;
    return (long long)n_split * B * H * S_q * (D + 1) * 4;
}

// the forward kernel over (query tile, key range) pairs, one workgroup each
template <int D, int QB, int SB, int NW, bool F16, int G>
static int launch_ranges(Params &p, int BH, int n_eff, hipStream_t st)
{
    typedef attn::FwdTiling<D, QB, SB, NW, true, G> T;
    p.n_qt = (p.S_q + T::BM - 1) / T::BM;
    const long long total = (long long)BH * p.n_qt * n_eff;
    if (total > 0x7fffffffLL)
        return ATTN_ERR_SHAPE;
    p.total_wg = (int)total;
    p.idle_row = idle_row(p, D, total);
    auto kern = attn::attn_fwd_asm_kernel<D, QB, SB, NW, false, F16, true, G>;
    if (!allow_lds(reinterpret_cast<const void *>(kern), T::LDS_BYTES))
        return ATTN_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)p.total_wg), dim3(T::THREADS), T::LDS_BYTES, st, p);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}

// Tiling of the ranges.  Up to 64 queries (decode) a 256-row tile is mostly rows that do not exist: 64-row tiles with
// two key groups stream the keys at the rate of a large copy (D = 128, one query, 64 heads of 8191 keys in 8 ranges:
// 69.8 -> 51.6 us; 16 heads of 131072 keys in 64 ranges: 260 -> 187 us), at D = 64 for long ranges or few of them, the
// 128-row workgroups (two to a CU) otherwise (512 ranges of 1024 keys: 42.6 us with 256-row tiles, 28.3 with 128, 29.8
// with 64; 1024 ranges of 2048 keys: 151 / 113 / 96).  With more queries the small tiles win while they find idle
// compute units (256 queries, 8 heads of 8192 keys in 8 ranges: D = 128 28.9 -> 17.5 us, D = 64 19.6 -> 11.2 us), the
// wide ones after that (32 ranges of 4096 keys: 137 against 197 us).  (D = 128: the 64-row waves of
// the unsplit kernel are 4 % faster there in the mean, but take their first reference from 32 keys instead of 64: over 1100
// launches of N(0, 1) inputs the error against 64 bits was larger in 943, by 0.2 % in the mean and 0.5 % for ranges under 700 keys;
// 520 to 640 queries took up to 1.3 times as long, a peaked softmax 1.05 times in the mean.)
template <int D, bool F16>
static int launch_splitkv(Params &p, int BH, int n_eff, void *o, float *lse, hipStream_t st)
{
    typedef typename std::conditional<F16, _Float16, attn::bf16_t>::type out_t;
    const long long n_rows = (long long)BH * p.S_q;
    const int cus = attn::cu_count(1) > 0 ? attn::cu_count(1) : 256;
    const long long ranges = (long long)BH * n_eff;
    const long long wg64 = ranges * ((p.S_q + 63) / 64), wg128 = ranges * ((p.S_q + 127) / 128);
    int rc;
    if constexpr (D == 128) {
        rc = p.S_q <= 64 || wg64 <= cus ? launch_ranges<128, 1, 1, 2, F16, 2>(p, BH, n_eff, st)
                                        : launch_ranges<128, 1, 2, 8, F16, 1>(p, BH, n_eff, st);
    } else {
        const bool groups = p.S_q <= 64 ? p.split_len >= 2048 || (2 * wg64 <= cus && p.split_len >= 512)
                                        : wg64 <= cus && p.split_len >= 512;
        if (groups)
            rc = launch_ranges<64, 1, 2, 2, F16, 2>(p, BH, n_eff, st);
        else if (p.S_q <= 128 || wg128 <= cus)
            rc = launch_ranges<64, 1, 2, 4, F16, 1>(p, BH, n_eff, st);
        else
            rc = launch_ranges<64, 1, 2, 8, F16, 1>(p, BH, n_eff, st);
    }
    if (rc != ATTN_OK)
        return rc;
    const int lanes_log2 = attn::merge_lanes_log2(D, n_eff);
    const int rpb = (attn::kMergeThreads / (D / 4)) >> lanes_log2;
    const long long blocks = (n_rows + rpb - 1) / rpb;
    const unsigned grid = (unsigned)(blocks < 16384 ? blocks : 16384);
    hipLaunchKernelGGL((attn::attn_splitkv_merge_kernel<D, out_t>), dim3(grid), dim3(attn::kMergeThreads), 0, st, p.o_part,
                       p.lse_part, static_cast<out_t *>(o), lse, n_rows, n_eff, lanes_log2);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}

template <bool F16>
static int splitkv_entry(const void *q, const void *k, const void *v, void *o, float *lse, void *workspace,
                         long long workspace_bytes, int n_split, int B, int H, int S_q, int S_kv, int D, int causal,
                         float scale, void *stream)
{
    Params p;
    const int rc = validate(q, k, v, o, lse, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    if (D == 256)
        return ATTN_ERR_UNSUPPORTED_D;
    if (causal)
        return ATTN_ERR_UNSUPPORTED;
    if (!(scale > 0.f))
        return ATTN_ERR_SCALE;
    if (n_split < 1 || n_split > 256 || (long long)S_kv * D * 2 >= (1LL << 31))
        return ATTN_ERR_SHAPE;
    if (!workspace)
        return ATTN_ERR_NULL;
    if ((uintptr_t)workspace & 15)
        return ATTN_ERR_ALIGN;
    if (workspace_bytes < attn_fwd_splitkv_workspace_bytes(B, H, S_q, D, n_split))
        return ATTN_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int n_eff = split_plan(S_kv, n_split, p.split_len);
    if (n_eff == 1) {  // one range: the plain kernel writes o and lse itself
        if (F16)
            return D == 64 ? launch_d64<true>(p, B * H, 0, st) : launch_d128<true>(p, B * H, 0, st);
        return D == 64 ? launch_d64<false>(p, B * H, 0, st) : launch_d128<false>(p, B * H, 0, st);
    }
    const long long n_rows = (long long)B * H * S_q;
    p.n_split = n_eff;
    p.o_part = static_cast<float *>(workspace);
    p.lse_part = p.o_part + (long long)n_eff * n_rows * D;
    return D == 64 ? launch_splitkv<64, F16>(p, B * H, n_eff, o, lse, st)
                   : launch_splitkv<128, F16>(p, B * H, n_eff, o, lse, st);
}

extern "C" int attn_fwd_splitkv(const void *q, const void *k, const void *v, void *o, float *lse, void *workspace,
                                long long workspace_bytes, int n_split, int B, int H, int S_q, int S_kv, int D,
                                int causal, float scale, void *stream)
{
    return splitkv_entry<false>(q, k, v, o, lse, workspace, workspace_bytes, n_split, B, H, S_q, S_kv, D, causal,
                                scale, stream);
}

extern "C" int attn_fwd_splitkv_f16(const void *q, const void *k, const void *v, void *o, float *lse, void *workspace,
                                    long long workspace_bytes, int n_split, int B, int H, int S_q, int S_kv, int D,
                                    int causal, float scale, void *stream)
{
    return splitkv_entry<true>(q, k, v, o, lse, workspace, workspace_bytes, n_split, B, H, S_q, S_kv, D, causal,
                               scale, stream);
}

extern "C" int attn_fwd_f16(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int S_q,
                            int S_kv, int D, int causal, float scale, void *stream)
{
    Params p;
    const int rc = validate(q, k, v, o, lse, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    // fp16 runs on the hand-scheduled kernels only
    if ((long long)S_kv * D * 2 >= (1LL << 31))
        return ATTN_ERR_SHAPE;
    if (!(scale > 0.f))
        return ATTN_ERR_SCALE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (D == 256)
        return launch_asm<256, 1, 1, 4, true>(p, B * H, causal, st);
    return D == 64 ? launch_d64<true>(p, B * H, causal, st) : launch_d128<true>(p, B * H, causal, st);
}

extern "C" int attn_fwd(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int S_q,
                        int S_kv, int D, int causal, float scale, void *stream)
{
    Params p;
    const int rc = validate(q, k, v, o, lse, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    return dispatch_fwd(p, B * H, D, causal, static_cast<hipStream_t>(stream));
}

#ifdef ATTN_DEBUG_ENTRY_POINTS
// Test-only entry point of the debug build of the library (libmi355attn_debug.so): attn_fwd with the
// kernel chosen by the caller.  variant 0: as attn_fwd; 1: the generic program-order kernel;
// 2 / 5: D = 128 on the one-wave-per-SIMD tiling (4 waves x 64 query rows) / on the two-waves-per-SIMD
// tiling (8 waves x 32 rows); 3 / 4: D = 64 with 8-wave / 4-wave workgroups; 6: D = 64 or 128 in 64-row
// workgroups with two key groups; 7 / 8: D = 128 in 128-row workgroups (2 waves x 64 rows / 4 waves x 32 rows in pairs).
// A variant that does not apply to the arguments returns ATTN_ERR_UNSUPPORTED.
template <bool F16>
static int fwd_tiling(const Params &p, int BH, int D, int causal, hipStream_t st, int variant)
{
    if (!(p.scale > 0.f && (long long)p.S_kv * D * 2 < (1LL << 31)))
        return ATTN_ERR_UNSUPPORTED;
    switch (variant) {
    case 2:
        return D == 128 ? launch_d128<F16>(p, BH, causal, st, 1) : ATTN_ERR_UNSUPPORTED;
    case 5:
        return D == 128 ? launch_d128<F16>(p, BH, causal, st, 0) : ATTN_ERR_UNSUPPORTED;
    case 6:
        return D == 128 ? launch_d128<F16>(p, BH, causal, st, 2)
               : D == 64 ? launch_d64<F16>(p, BH, causal, st, 2) : ATTN_ERR_UNSUPPORTED;
    case 7:
    case 8:
        return D == 128 ? launch_d128<F16>(p, BH, causal, st, variant - 4) : ATTN_ERR_UNSUPPORTED;
    case 3:
    case 4:
        return D == 64 ? launch_d64<F16>(p, BH, causal, st, variant - 3) : ATTN_ERR_UNSUPPORTED;
    }
    return ATTN_ERR_UNSUPPORTED;
}

extern "C" int attn_fwd_variant(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H,
                                int S_q, int S_kv, int D, int causal, float scale, void *stream, int variant)
{
    Params p;
    const int rc = validate(q, k, v, o, lse, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (variant) {
    case 0:
        return dispatch_fwd(p, B * H, D, causal, st);
    case 1:
        return launch_generic(p, B * H, D, causal, st);
    default:
        return fwd_tiling<false>(p, B * H, D, causal, st, variant);
    }
}

// The same for attn_fwd_f16 (which has no program-order kernel: variant 1 is refused).
extern "C" int attn_fwd_f16_variant(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H,
                                    int S_q, int S_kv, int D, int causal, float scale, void *stream, int variant)
{
    if (variant == 0)
        return attn_fwd_f16(q, k, v, o, lse, B, H, S_q, S_kv, D, causal, scale, stream);
    Params p;
    const int rc = validate(q, k, v, o, lse, B, H, S_q, S_kv, D, scale, p);
    return rc != ATTN_OK ? rc : fwd_tiling<true>(p, B * H, D, causal, static_cast<hipStream_t>(stream), variant);
}
#endif

#ifdef ATTN_DEBUG_ENTRY_POINTS
// Test-only, host only: the tiling that the dispatcher takes for D = 64 or 128 and at least 64 queries (numbers as in
// launch_d64 and launch_d128).
extern "C" int attn_fwd_tiling(int D, int heads, int S_q, int S_kv, int causal)
{
    Params p;
    p.S_q = S_q;
    p.S_kv = S_kv;
    return D == 128 ? choose_d128_all(heads, p, causal) : choose_d64(heads, p, causal);
}

// Measurement entry point of the debug build: attn_fwd (hand-scheduled kernels) that also records, per
// tile w of the launch's queue, trace[8 w + 0..5] = the 100 MHz constant clock when the tile is taken up, after
// K(0) and Q have landed, before the main loop, after it, after O is staged in LDS, and when O is stored;
// trace[8 w + 6] = the clock when the tile's first loads are all issued; trace[8 w + 7] = XCC_ID << 32 | HW_ID
// (CU, SE, ...) of a wave of the workgroup.  trace: device,
// trace_entries 64-bit values; workgroups whose record would not fit write nothing.
extern "C" int attn_fwd_trace(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int S_q,
                              int S_kv, int D, int causal, float scale, void *stream, unsigned long long *trace,
                              long long trace_entries)
{
    Params p;
    const int rc = validate(q, k, v, o, lse, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    if (!trace || trace_entries < 8)
        return ATTN_ERR_NULL;
    p.trace = trace;
    p.trace_entries = trace_entries;
    return dispatch_fwd(p, B * H, D, causal, static_cast<hipStream_t>(stream));
}

// Measurement entry point of the debug build: n_wg workgroups of waves_per_wg (4 or 8) waves, each wave
// `iters` x 8 MFMAs (32768 FLOP each) on the 8 fragments at `operands` (device, 8 * 64 * 16 bytes: 4 A then 4 B
// fragments, 16 bytes per lane); `out` (device, n_wg * waves_per_wg * 64 floats) receives one value per lane.
extern "C" int attn_probe_mfma(const void *operands, float *out, int n_wg, int waves_per_wg, int iters, void *stream)
{
    if (!operands || !out)
        return ATTN_ERR_NULL;
    if (n_wg < 1 || iters < 1 || (waves_per_wg != 4 && waves_per_wg != 8))
        return ATTN_ERR_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const attn::bf16x8 *ops = static_cast<const attn::bf16x8 *>(operands);
    if (waves_per_wg == 4)
        hipLaunchKernelGGL(attn::attn_probe_mfma_kernel<4>, dim3(n_wg), dim3(256), 0, st, ops, out, iters);
    else
        hipLaunchKernelGGL(attn::attn_probe_mfma_kernel<8>, dim3(n_wg), dim3(512), 0, st, ops, out, iters);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}
#endif

#ifdef ATTN_DEBUG_ENTRY_POINTS
// Measurement entry point of the debug build: attn_probe_mfma with four waves per workgroup and the operand
// pattern of attn_probe_mfma_pattern_kernel (0 .. 5; 5 reads `operands` as IEEE binary16).  Patterns 0-3 and 5
// issue iters x 8 MFMAs of 32768 FLOP per wave, pattern 4 iters x 16 of 16384 FLOP.
extern "C" int attn_probe_mfma_pattern(const void *operands, float *out, int n_wg, int pattern, int iters, void *stream)
{
    if (!operands || !out)
        return ATTN_ERR_NULL;
    if (n_wg < 1 || iters < 1 || pattern < 0 || pattern > 5)
        return ATTN_ERR_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const attn::bf16x8 *ops = static_cast<const attn::bf16x8 *>(operands);
    switch (pattern) {
    case 0: hipLaunchKernelGGL(attn::attn_probe_mfma_pattern_kernel<0>, dim3(n_wg), dim3(256), 0, st, ops, out, iters); break;
    case 1: hipLaunchKernelGGL(attn::attn_probe_mfma_pattern_kernel<1>, dim3(n_wg), dim3(256), 0, st, ops, out, iters); break;
    case 2: hipLaunchKernelGGL(attn::attn_probe_mfma_pattern_kernel<2>, dim3(n_wg), dim3(256), 0, st, ops, out, iters); break;
    case 3: hipLaunchKernelGGL(attn::attn_probe_mfma_pattern_kernel<3>, dim3(n_wg), dim3(256), 0, st, ops, out, iters); break;
    case 4: hipLaunchKernelGGL(attn::attn_probe_mfma_pattern_kernel<4>, dim3(n_wg), dim3(256), 0, st, ops, out, iters); break;
    default: hipLaunchKernelGGL(attn::attn_probe_mfma_pattern_kernel<5>, dim3(n_wg), dim3(256), 0, st, ops, out, iters); break;
    }
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}
#endif

#ifdef ATTN_DEBUG_ENTRY_POINTS
// Measurement entry point of the debug build: the atomic traffic of a single-pass backward's dQ reduction for
// n_heads heads of S_q queries and S_kv keys (D = 128; S_q a multiple of 64, S_kv of 128) into dq (device,
// n_heads * S_q * 128 floats, zeroed by the caller).
extern "C" int attn_probe_dq_atomics(float *dq, int n_heads, int S_q, int S_kv, int causal, void *stream)
{
    if (!dq)
        return ATTN_ERR_NULL;
    if (n_heads < 1 || S_q < 64 || S_kv < 128 || S_q % 64 || S_kv % 128 || (long long)n_heads * (S_kv / 128) > 0x7fffffffLL)
        return ATTN_ERR_SHAPE;
    const int n_kt = S_kv / 128;
    hipLaunchKernelGGL(attn::attn_probe_dq_atomics_kernel, dim3(n_heads * n_kt), dim3(256), 0, static_cast<hipStream_t>(stream),
                       dq, S_q, n_kt, causal);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}
#endif

extern "C" int attn_workgroup_tile(int causal, int workgroup, int n_heads, int n_tiles, long long head_bytes, int *head,
                                   int *tile)
{
    if (!head || !tile)
        return ATTN_ERR_NULL;
    if (n_heads < 1 || n_tiles < 1 || head_bytes < 0 || (long long)n_heads * n_tiles > 0x7fffffffLL || workgroup < 0 ||
        workgroup >= n_heads * n_tiles)
        return ATTN_ERR_SHAPE;
    if (causal)
        attn::wg_to_tile_n<true>(workgroup, n_heads * n_tiles, n_tiles, head_bytes, *head, *tile);
    else
        attn::wg_to_tile_n<false>(workgroup, n_heads * n_tiles, n_tiles, head_bytes, *head, *tile);
    return ATTN_OK;
}

extern "C" int attn_workgroup_queue_entry(int workgroup, int n_workgroups, int n_entries, int pass, int *entry)
{
    if (!entry)
        return ATTN_ERR_NULL;
    if (n_workgroups < 1 || n_entries < 1 || pass < 0 || workgroup < 0 || workgroup >= n_workgroups ||
        (n_workgroups < n_entries && n_workgroups % attn::kNumXcd))
        return ATTN_ERR_SHAPE;
    *entry = attn::persistent_entry(workgroup, n_workgroups, n_entries, pass);
    return ATTN_OK;
}

extern "C" const char *attn_strerror(int status)
{
    switch (status) {
    case ATTN_OK:
        return "ok";
    case ATTN_ERR_NULL:
        return "a required pointer is NULL";
    case ATTN_ERR_SHAPE:
        return "B, H, S_q, S_kv must be >= 1 and the tensors must not exceed 2^40 elements";
    case ATTN_ERR_UNSUPPORTED_D:
        return "head dimension D must be 64, 128 or 256";
    case ATTN_ERR_ALIGN:
        return "q, k, v, o must be 16-byte aligned and lse 4-byte aligned";
    case ATTN_ERR_SCALE:
        return "scale must be finite and >= 0";
    case ATTN_ERR_LAUNCH:
        return "the HIP runtime rejected the kernel launch";
    case ATTN_ERR_UNSUPPORTED:
        return "this entry point does not implement the requested combination (e.g. causal split-KV)";
    case ATTN_ERR_WORKSPACE:
        return "the workspace is too small: smaller than attn_fwd_splitkv_workspace_bytes() asks for, or the shape exceeds "
               "the built-in workspace of attn_bwd_noalloc (B*H*S_q <= 2^21)";
    }
    return "unknown attn_status";
}

extern "C" int attn_version(void) { return 600; }
