// attn_bwd.hip -- C ABI entry point attn_bwd (see include/attn_bwd.h): validation and launches.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "attn_bwd.h"  // the C declaration (include/)
#include "attn_bwd_asm.h"
#include "attn_bwd_kernels.h"
#include "attn_bwd_wide.h"
#include "attn_fwd.h"  // attn_status
#include "attn_launch.h"

// Workspace of attn_bwd_noalloc: one copy per GPU that the library runs on, held until the process ends.
// In host code this name is only a handle for hipGetSymbolAddress; the device address it yields (one per
// device) is what is passed to kernels.
#define ATTN_BWD_NOALLOC_MAX_ROWS (1 << 21)
static __device__ __align__(256) float scratch[2 * ATTN_BWD_NOALLOC_MAX_ROWS];

namespace {

using attn::BwdParams;

// one compiler-scheduled sweep, one workgroup per owner tile
template <typename K>
int launch_sweep(K kern, BwdParams p, int BH, int S_own, int NW, int lds_bytes, hipStream_t stream)
{
    p.n_t = (S_own + NW * 32 - 1) / (NW * 32);
    const long long total = (long long)BH * p.n_t;
    if (total > 0x7fffffffLL)
        return ATTN_ERR_SHAPE;
    p.total_wg = (int)total;
    if (!attn::allow_lds(reinterpret_cast<const void *>(kern), lds_bytes))
        return ATTN_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)p.total_wg), dim3(NW * 64), lds_bytes, stream, p);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}

// Few queries against many keys: the query-owner tiles at the end of the queue are the long ones then, and where they
// begin within a pass over the workgroups and end in the next one, some workgroups walk two of them while others walk
// none.  Such launches run one sweep after the other: 123 heads of 72 queries and 5938 keys, D = 128, 372 -> 315 us, of 1500
// keys 102 -> 90 (D = 64 60 -> 50); 16 heads of 1000 queries and 8000 keys 332 -> 258, causal 80 -> 72 (D = 64 208 -> 155,
// 52 -> 45).  Where the tiles end in the pass they began in, are short, or enough for the workgroups (causal: for half of
// them, as half of the tiles are short), one launch is ahead or level (48 heads of 72 x 1500 49 / 61, 123 of 64 x 512,
// causal, 29 / 33; 48 of 1000 x 8000, causal, D = 64 83 / 92; 400 of 72 x 5938 983 / 1004).
bool sweeps_apart(const BwdParams &p, int causal, int slots)
{
    const attn::BwdQueue queue(p.total_wg, p.total_q);
    const int walk = causal && p.S_q < p.S_kv ? p.S_q : p.S_kv;          // keys of the longest query-owner tile
    if (queue.n_entries <= slots || p.total_q > (causal ? slots / 2 : slots) || p.S_kv / 4 < p.S_q || walk < 1000)
        return false;
    const int per_pass = slots / attn::kNumXcd;                          // entries of an XCD in one pass
    const int first = queue.q_first / attn::kNumXcd, last = (queue.n_entries - 1) / attn::kNumXcd;
    return first % per_pass != 0 && first / per_pass != last / per_pass;
}

// both hand-scheduled sweeps: as many workgroups as the chip holds at once, each walking the queue of owner tiles of its
// XCD
int launch_sweeps(void (*kern)(const BwdParams), int LDS, const BwdParams &p, int causal, hipStream_t stream)
{
    if (!attn::allow_lds(reinterpret_cast<const void *>(kern), LDS))
        return ATTN_ERR_LAUNCH;
    // (a runtime that cannot tell the occupancy gets one workgroup per entry: the kernel takes either)
    int slots = attn::persistent_slots(reinterpret_cast<const void *>(kern), 256, LDS, attn::kNumXcd);
    if (slots < attn::kNumXcd)
        slots = 0x7fffffff;
    const auto run = [&](int n_kv, int n_q) {
        BwdParams r = p;
        r.total_wg = n_kv;
        r.total_q = n_q;
        const int entries = attn::BwdQueue(n_kv, n_q).n_entries;
        hipLaunchKernelGGL(kern, dim3((unsigned)(slots < entries ? slots : entries)), dim3(256), LDS, stream, r);
        return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
    };
    if (!sweeps_apart(p, causal, slots))
        return run(p.total_wg, p.total_q);
    const int rc = run(p.total_wg, 0);
    return rc == ATTN_OK ? run(0, p.total_q) : rc;
}

enum BwdTiling { kAsDispatched, kRows128, kRows256 };

// What a workgroup's walk costs, in us: per owner tile and per streamed tile of either sweep; `launch` + `mean` times the mean
// walk of all compute units is added to the longest one (full compute units take each other's power).  Fitted to 8300
// launches of 1 to 256 heads and 64 to 16384 rows, D = 128, causal or not (root mean square of the error 5 and 6 %).
struct WalkCost {
    float key_tile, key_step, query_tile, query_step, launch, mean;
};
constexpr WalkCost kWalk128 = {4.10f, 0.521f, 3.37f, 0.366f, 5.8f, 0.58f}, kWalk256 = {7.38f, 0.932f, 5.50f, 0.656f, 4.6f, 0.52f};

// Streamed tiles of owner tile t (`rows` rows) of a key-owner or query-owner sweep
int walk_steps(const BwdParams &p, int causal, int rows, bool keys, int t)
{
    if (keys) {
        const int n = (p.S_q + 31) / 32, first = t * (rows / 32);
        return !causal ? n : (first < n ? n - first : 0);
    }
    int end = p.S_kv;
    if (causal) {
        const int last = p.S_q / rows > t ? (t + 1) * rows : p.S_q;
        end = last < end ? last : end;
    }
    return (end + 31) / 32;
}

// Estimated time of a D = 128 launch with owner tiles of `rows` rows: the longest walk among workgroups of one XCD, of which a
// few are followed through the queue, those around the ends of the sweeps among them.
float launch_estimate(const BwdParams &p, int BH, int causal, int rows, const WalkCost &c, int slots)
{
    const int n_t = (p.S_kv + rows - 1) / rows, n_tq = (p.S_q + rows - 1) / rows;
    const attn::BwdQueue queue(BH * n_t, BH * n_tq);
    const int per_pass = slots / attn::kNumXcd;
    // steps of a head's tiles: they fall (key owners) or rise (query owners) by rows / 32 from tile to tile while a mask cuts them
    const auto steps = [&](bool keys, int n) {
        double sum = 0;
        if (!causal)
            return (double)n * walk_steps(p, 0, rows, keys, 0);
        const int cut = (p.S_q < p.S_kv ? p.S_q : p.S_kv) / rows, m = cut < n ? cut : n;    // tiles the mask's edge runs through
        const int d = rows / 32;
        if (keys) {
            const int first = (p.S_q + 31) / 32, all = (first + d - 1) / d < n ? (first + d - 1) / d : n;
            sum = (double)all * first - 0.5 * d * all * (all - 1.0);
        } else {
            sum = 0.5 * d * m * (m + 1.0) + (double)(n - m) * walk_steps(p, causal, rows, keys, n - 1);
        }
        return sum;
    };
    const double all = BH * (n_t * (double)c.key_tile + steps(true, n_t) * c.key_step + n_tq * (double)c.query_tile +
                             steps(false, n_tq) * c.query_step);
    const float mean = (float)(all / slots);
    const float keys = c.key_tile + c.key_step * walk_steps(p, causal, rows, true, 0);
    const float queries = c.query_tile + c.query_step * walk_steps(p, causal, rows, false, n_tq - 1);
    const float heaviest = keys > queries ? keys : queries;
    if (queue.n_entries <= slots)
        return c.launch + heaviest + c.mean * mean;
    if (queue.n_entries > 12 * slots)
        return c.launch + mean + heaviest * (causal ? 0.25f : 0.5f) + c.mean * mean;
    float longest = 0.f;
    const auto follow = [&](int m) {
        float sum = 0.f;
        for (int k = 0;; ++k) {
            const int entry = queue.entry(m * attn::kNumXcd, slots, per_pass, k);
            if (entry < 0)
                break;
            const bool own_keys = entry < queue.n_kv;
            if (!own_keys && entry < queue.q_first)
                continue;
            int bh = 0, t = 0;
            if (causal)
                attn::wg_to_tile_n<true>(own_keys ? entry : entry - queue.q_first, BH * (own_keys ? n_t : n_tq),
                                         own_keys ? n_t : n_tq, 4ll * (p.S_q + p.S_kv) * 128, bh, t);
            if (causal && own_keys)
                t = n_t - 1 - t;
            const int n = walk_steps(p, causal, rows, own_keys, t);
            sum += own_keys ? c.key_tile + c.key_step * n : c.query_tile + c.query_step * n;
        }
        longest = sum > longest ? sum : longest;
    };
    for (int m = 0; m < per_pass; m += (per_pass + 7) / 8)
        follow(m);
    follow(per_pass - 1);
    const int ends[3] = {(queue.n_kv + 7) / 8, queue.q_first / 8 + 1, (queue.n_entries + 7) / 8 - 1};
    for (const int end : ends)
        for (int i = end - 1; i <= end + 1; ++i)
            if (i >= 0 && i < (queue.n_entries + 7) / 8) {
                const int at = i / per_pass & 1 ? per_pass - 1 - i % per_pass : i % per_pass;
                follow(per_pass - 1 - at);
            }
    return c.launch + longest + c.mean * mean;
}

// D = 128: whether owner tiles of 256 rows (64-row waves) are ahead of tiles of 128.  Half the LDS operand reads and half
// the stream per product: long walks on a full chip are 8 to 11 % faster (32 heads of 2048 rows 209 -> 190 us, 128 of 4096
// 3085 -> 2768, causal 1701 -> 1561).  Half the tiles, each with twice as much around its loop and more rows that do not exist:
// launches that do not fill the chip are up to 1.7 times slower (16 heads of 1024 rows 35 -> 44).  Launches that the smaller
// tiles run one sweep after the other stay with them.
bool wide_pays(const BwdParams &p, int BH, int causal, int slots)
{
    if (slots < attn::kNumXcd || 2ll * BH * ((p.S_kv + 255) / 256 + (p.S_q + 255) / 256) < slots)
        return false;   // (no launch of fewer tiles gained)
    BwdParams small = p;
    small.total_wg = BH * ((p.S_kv + 127) / 128);
    small.total_q = BH * ((p.S_q + 127) / 128);
    if (sweeps_apart(small, causal, slots))
        return false;
    // (of 8300 launches 20 % take them, 7 % faster in the mean; 42 of those are more than 2 % slower, 1.16 times at worst: 14 causal
    // heads of 5182 queries and 11160 keys.  A margin of 0.98 with a mask would gain a tenth more and lose in twice as many)
    return launch_estimate(p, BH, causal, 256, kWalk256, slots) <
           (causal ? 0.96f : 0.98f) * launch_estimate(p, BH, causal, 128, kWalk128, slots);
}

template <int D, typename ELEM>
int launch_delta(const BwdParams &p, hipStream_t stream)
{
    const long long blocks = (p.n_rows + (256 / (D / 8)) - 1) / (256 / (D / 8));
    const unsigned grid = (unsigned)(blocks < 4096 ? blocks : 4096);
    hipLaunchKernelGGL((attn::attn_bwd_delta_kernel<D, ELEM>), dim3(grid), dim3(256), 0, stream, p);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}

// Delta, then both hand-scheduled sweeps (scale > 0), in one launch: few owner tiles then fill the chip together, and
// no launch gap or half-empty last round separates the sweeps.  The same bits.  Measured (whole call, one launch per
// sweep -> one for both), D = 128: 16 heads of 128 rows 20.2 -> 13.2 us, of 1024 rows 54.4 -> 38.2, causal 53.5 -> 34.4;
// of 4096 rows 408.8 -> 404.7; 128 heads of 2048 rows 860 -> 850.
template <int D, bool F16>
int launch_hand(BwdParams p, int BH, int causal, hipStream_t stream, BwdTiling tiling = kAsDispatched)
{
    if ((long long)BH * ((p.S_kv + 127) / 128 + (p.S_q + 127) / 128) > 0x7fffffffLL - attn::kNumXcd)
        return ATTN_ERR_SHAPE;
    const bool wide = D == 128 && (tiling == kAsDispatched ? wide_pays(p, BH, causal, attn::cu_count(attn::kNumXcd)) : tiling == kRows256);
    const int rows = wide ? 256 : 128;
    p.n_t = (p.S_kv + rows - 1) / rows;
    p.n_tq = (p.S_q + rows - 1) / rows;
    p.total_wg = BH * p.n_t;
    p.total_q = BH * p.n_tq;
    const int cus = attn::cu_count(attn::kNumXcd);
    p.cus_per_xcd = cus > 0 ? cus / attn::kNumXcd : 32;
    const int rc = launch_delta<D, typename std::conditional<F16, _Float16, attn::bf16_t>::type>(p, stream);
    if (rc != ATTN_OK)
        return rc;
    if constexpr (D == 128) {
        if (wide)
            return launch_sweeps(causal ? attn::attn_bwd_wide_kernel<true, F16> : attn::attn_bwd_wide_kernel<false, F16>,
                                 attn::BwdWideLds::BYTES, p, causal, stream);
    }
    return launch_sweeps(causal ? attn::attn_bwd_asm_kernel<D, true, F16> : attn::attn_bwd_asm_kernel<D, false, F16>,
                         attn::BwdLds<D>::BYTES, p, causal, stream);
}

// plain: run the compiler-scheduled sweeps (always when scale == 0, which the hand-scheduled loops exclude)
template <int D>
int launch_bwd(const BwdParams &p, int BH, int causal, hipStream_t stream, bool plain)
{
    if (!plain && p.scale > 0.f)
        return launch_hand<D, false>(p, BH, causal, stream);
    constexpr int NWK = 4, NWQ = 8;  // waves per workgroup of the key-owner / query-owner sweep
    constexpr int LDSK = 2 * 3 * 64 * D * 2 + 3 * NWK * 256, LDSQ = 2 * 3 * 64 * D * 2 + 3 * NWQ * 256;
    int rc = launch_delta<D, attn::bf16_t>(p, stream);
    if (rc != ATTN_OK)
        return rc;
    rc = causal ? launch_sweep(attn::attn_bwd_sweep_kernel<D, true, true, NWK>, p, BH, p.S_kv, NWK, LDSK, stream)
                : launch_sweep(attn::attn_bwd_sweep_kernel<D, false, true, NWK>, p, BH, p.S_kv, NWK, LDSK, stream);
    if (rc != ATTN_OK)
        return rc;
    return causal ? launch_sweep(attn::attn_bwd_sweep_kernel<D, true, false, NWQ>, p, BH, p.S_q, NWQ, LDSQ, stream)
                  : launch_sweep(attn::attn_bwd_sweep_kernel<D, false, false, NWQ>, p, BH, p.S_q, NWQ, LDSQ, stream);
}

}  // namespace

// host-side validation shared by the entry points; fills `p` on success
static int validate_bwd(const void *q, const void *k, const void *v, const void *o, const void *d_o, const float *lse,
                        void *dq, void *dk, void *dv, float *delta_ws, int B, int H, int S_q, int S_kv, int D,
                        float scale, BwdParams &p)
{
    if (!q || !k || !v || !o || !d_o || !lse || !dq || !dk || !dv || !delta_ws)
        return ATTN_ERR_NULL;
    if (B < 1 || H < 1 || S_q < 1 || S_kv < 1)
        return ATTN_ERR_SHAPE;
    if (D != 64 && D != 128)
        return ATTN_ERR_UNSUPPORTED_D;
    const long long BH = (long long)B * H;
    if (BH > 0x7fffffffLL || BH * (long long)(S_q > S_kv ? S_q : S_kv) > (1LL << 40) / D)
        return ATTN_ERR_SHAPE;
    // one head of any tensor, and the workspace, are addressed with 32-bit byte offsets
    if ((long long)(S_q > S_kv ? S_q : S_kv) * D * 2 >= (1LL << 31) || BH * S_q * 8 >= (1LL << 31))
        return ATTN_ERR_SHAPE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)d_o | (uintptr_t)dq | (uintptr_t)dk |
         (uintptr_t)dv) & 15)
        return ATTN_ERR_ALIGN;
    if (((uintptr_t)lse | (uintptr_t)delta_ws) & 3)
        return ATTN_ERR_ALIGN;
    if (!(scale >= 0.f) || isinf(scale))
        return ATTN_ERR_SCALE;
    p.q = static_cast<const attn::bf16_t *>(q);
    p.k = static_cast<const attn::bf16_t *>(k);
    p.v = static_cast<const attn::bf16_t *>(v);
    p.o = static_cast<const attn::bf16_t *>(o);
    p.d_o = static_cast<const attn::bf16_t *>(d_o);
    p.lse = lse;
    p.lse2 = delta_ws;
    p.delta = delta_ws + BH * S_q;
    p.dq = static_cast<attn::bf16_t *>(dq);
    p.dk = static_cast<attn::bf16_t *>(dk);
    p.dv = static_cast<attn::bf16_t *>(dv);
    p.S_q = S_q;
    p.S_kv = S_kv;
    p.n_t = 0;
    p.total_wg = 0;
    p.cus_per_xcd = 0;
    p.n_tq = 0;
    p.total_q = 0;
    p.n_rows = BH * S_q;
    p.c = scale * 1.44269504088896340736f;
    p.scale = scale;
    return ATTN_OK;
}

extern "C" int attn_bwd(const void *q, const void *k, const void *v, const void *o, const void *d_o, const float *lse,
                        void *dq, void *dk, void *dv, float *delta_ws, int B, int H, int S_q, int S_kv, int D,
                        int causal, float scale, void *stream)
{
    BwdParams p;
    const int rc = validate_bwd(q, k, v, o, d_o, lse, dq, dk, dv, delta_ws, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return D == 64 ? launch_bwd<64>(p, B * H, causal, st, false) : launch_bwd<128>(p, B * H, causal, st, false);
}

// device address of `scratch` on the current device; resolved on the first call on that device
static float *scratch_on_current_device()
{
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static float *ptr[kMaxDev] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *addr = nullptr;
        if (hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch)) != hipSuccess || !addr) {
            (void)hipGetLastError();
            return nullptr;
        }
        ptr[dev] = static_cast<float *>(addr);
    }
    return ptr[dev];
}

extern "C" int attn_bwd_noalloc(const void *q, const void *k, const void *v, const void *o, const void *d_o,
                                const float *lse, void *dq, void *dk, void *dv, int B, int H, int S_q, int S_kv,
                                int D, int causal, float scale, void *stream)
{
    // size check on the host first: the rows must fit the library's own workspace
    if (B >= 1 && H >= 1 && S_q >= 1 && (long long)B * H * S_q > ATTN_BWD_NOALLOC_MAX_ROWS)
        return ATTN_ERR_WORKSPACE;
    BwdParams p;
    float dummy_ws = 0.f;  // validate_bwd only looks at the address
    const int rc = validate_bwd(q, k, v, o, d_o, lse, dq, dk, dv, &dummy_ws, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    float *ws = scratch_on_current_device();
    if (!ws)
        return ATTN_ERR_LAUNCH;
    // every word of the workspace that the sweeps read is written by the Delta kernel of this call:
    // nothing has to start at zero
    p.lse2 = ws;
    p.delta = ws + (long long)B * H * S_q;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return D == 64 ? launch_bwd<64>(p, B * H, causal, st, false) : launch_bwd<128>(p, B * H, causal, st, false);
}

#ifdef ATTN_DEBUG_ENTRY_POINTS
// Test-only, host only: the queue entry that workgroup `wg` of a backward launch of n_slots workgroups takes up in pass
// k, for n_kv key-owner and n_q query-owner tiles (BwdQueue); *first_q = entry number of the first query-owner tile.
extern "C" int attn_bwd_queue_entry(int n_kv, int n_q, int wg, int n_slots, int cus, int k, int *first_q)
{
    const attn::BwdQueue queue(n_kv, n_q);
    *first_q = queue.q_first;
    return queue.entry(wg, n_slots < queue.n_entries ? n_slots : queue.n_entries, cus, k);
}

// Test-only, host only: whether a backward launch of `slots` workgroups runs one sweep after the other (sweeps_apart).
extern "C" int attn_bwd_sweeps_apart(int heads, int S_q, int S_kv, int causal, int slots)
{
    BwdParams p;
    p.S_q = S_q;
    p.S_kv = S_kv;
    p.total_wg = heads * ((S_kv + 127) / 128);
    p.total_q = heads * ((S_q + 127) / 128);
    return sweeps_apart(p, causal, slots);
}

// Test-only, host only: whether a D = 128 launch takes owner tiles of 256 rows; est: the two estimates in us.
extern "C" int attn_bwd_wide_pays(int heads, int S_q, int S_kv, int causal, int slots, float *est)
{
    BwdParams p;
    p.S_q = S_q;
    p.S_kv = S_kv;
    est[0] = launch_estimate(p, heads, causal, 128, kWalk128, slots);
    est[1] = launch_estimate(p, heads, causal, 256, kWalk256, slots);
    return wide_pays(p, heads, causal, slots);
}

// Test-only: attn_bwd / attn_bwd_f16 (D = 128, scale > 0) on owner tiles of 128 (tiling 1) or 256 rows (2).
extern "C" int attn_bwd_tiling(const void *q, const void *k, const void *v, const void *o, const void *d_o,
                               const float *lse, void *dq, void *dk, void *dv, float *delta_ws, int B, int H, int S_q,
                               int S_kv, int f16, int causal, float scale, void *stream, int tiling)
{
    BwdParams p;
    const int rc = validate_bwd(q, k, v, o, d_o, lse, dq, dk, dv, delta_ws, B, H, S_q, S_kv, 128, scale, p);
    if (rc != ATTN_OK)
        return rc;
    if (!(scale > 0.f))
        return ATTN_ERR_SCALE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return f16 ? launch_hand<128, true>(p, B * H, causal, st, (BwdTiling)tiling)
               : launch_hand<128, false>(p, B * H, causal, st, (BwdTiling)tiling);
}

// Test-only entry point of the debug build of the library: attn_bwd on the compiler-scheduled sweeps
// (the reference of the schedule-equivalence test).
extern "C" int attn_bwd_plain(const void *q, const void *k, const void *v, const void *o, const void *d_o,
                              const float *lse, void *dq, void *dk, void *dv, float *delta_ws, int B, int H, int S_q,
                              int S_kv, int D, int causal, float scale, void *stream)
{
    BwdParams p;
    const int rc = validate_bwd(q, k, v, o, d_o, lse, dq, dk, dv, delta_ws, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return D == 64 ? launch_bwd<64>(p, B * H, causal, st, true) : launch_bwd<128>(p, B * H, causal, st, true);
}
#endif

extern "C" int attn_bwd_f16(const void *q, const void *k, const void *v, const void *o, const void *d_o,
                            const float *lse, void *dq, void *dk, void *dv, float *delta_ws, int B, int H, int S_q,
                            int S_kv, int D, int causal, float scale, void *stream)
{
    BwdParams p;
    const int rc = validate_bwd(q, k, v, o, d_o, lse, dq, dk, dv, delta_ws, B, H, S_q, S_kv, D, scale, p);
    if (rc != ATTN_OK)
        return rc;
    // fp16 runs on the hand-scheduled sweeps only
    if (!(scale > 0.f))
        return ATTN_ERR_SCALE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return D == 64 ? launch_hand<64, true>(p, B * H, causal, st) : launch_hand<128, true>(p, B * H, causal, st);
}
