// attn_bwd.hip -- C ABI entry point attn_bwd (see include/attn_bwd.h): validation and launches.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
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
// causal, 29 / 33; 48 of 1000 x 8000, causal, D = 64 83 / 92; 400 of 72 x 5938 983 / 1004).  Most of them now take a plan
// (plan_walks), which is asked first; these are left where it does not pay or has too many entries.  64-row waves (one after the
// other / one launch): no mask 257 heads of 90 x 3413 337 / 387, 201 of 121 x 5021 404 / 497, 75 of 459 x 13920 911 / 1148; causal
// 6 of 1443 x 10145 101 / 66, 7 of 1103 x 7699 84 / 53: those run in one launch.
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

enum BwdTiling { kAsDispatched, kRows128, kRows256, kRows128TwoWaves };

// What a workgroup's walk costs, in us: per owner tile and per streamed tile of either sweep; `launch` + `mean` times the mean
// walk of all workgroups is added to the longest one (full compute units take each other's power).  Fitted to 7200 launches
// of 1 to 256 heads and 64 to 16384 rows, D = 128, causal or not (root mean square of the error 5, 6 and 5 %).
struct WalkCost {
    int rows, per_cu;   // of an owner tile; workgroups that a compute unit holds
    float key_tile, key_step, query_tile, query_step, launch, mean, plan_pays, alone = 1.f;
    float key(int steps) const { return key_tile + key_step * steps; }
    float query(int steps) const { return query_tile + query_step * steps; }
};
constexpr WalkCost kWalk128 = {128, 1, 4.18f, 0.522f, 3.55f, 0.367f, 5.76f, 0.535f, 0.95f},
                   kWalk256 = {256, 1, 7.26f, 0.924f, 5.56f, 0.644f, 4.83f, 0.503f, 0.95f},
                   kWalk128TwoWaves = {128, 2, 7.27f, 0.920f, 6.32f, 0.654f, 4.72f, 0.551f, 0.95f};
// D = 64 (two workgroups to a CU): what the tiles' walks cost beside each other, and what share of it the longer walk's rest takes once the
// other has ended (`alone`), is all that is asked of it
constexpr WalkCost kWalkD64 = {128, 2, 4.0f, 0.60f, 3.5f, 0.45f, 0.f, 0.f, 0.93f, 0.6f};

// Streamed tiles of owner tile t (`rows` rows) of a key-owner or query-owner sweep
int walk_steps(const BwdParams &p, int causal, int rows, bool keys, int t)
{
    if (keys) {
        const int n = (p.S_q + 31) / 32, first = t * (rows / 32);
        return !causal ? n : (first < n ? n - first : 0);
    }
    int end = p.S_kv;
    if (causal) {
        const long long last = (t + 1ll) * rows < p.S_q ? (t + 1ll) * rows : p.S_q;
        end = last < end ? (int)last : end;
    }
    return (end + 31) / 32;
}

// The tiles of one sweep that an XCD takes up, in its queue's order: what wg_to_tile_n gives for entries xcd, xcd + 8, xcd + 16,
// ..., without its divisions.  each(t, n) per n tiles t.
template <typename F>
void xcd_tiles(int heads, int n_t, int causal, long long head_bytes, int xcd, F &&each)
{
    using attn::kNumXcd;
    const int a = heads / kNumXcd, r = heads % kNumXcd, n_left = r * n_t;
    if (!causal) {
        each(0, (int)(((long long)heads * n_t - xcd + kNumXcd - 1) / kNumXcd));   // (all alike)
        return;
    }
    for (int i = 0; kNumXcd * i + xcd < n_left; ++i)
        each(n_t - 1 - (kNumXcd * i + ((i & 1) && kNumXcd * (i + 1) <= n_left ? kNumXcd - 1 - xcd : xcd)) / r, 1);
    if (a == 0)
        return;
    const int want = attn::causal_group_heads(n_t, head_bytes), ng = a > want ? a / want : 1;
    for (int g = 0; g < ng; ++g)
        for (int t = n_t - 1; t >= 0; --t)
            each(t, a / ng + (g < a % ng));
}

// The walks of a launch's workgroups in one tiling, from what every entry of an XCD's queue costs
struct BwdWalks {
    static constexpr int kMax = attn::BwdPlan::kMaxEntries;
    int n, first_q, per_xcd;   // entries of XCD 0, the first of a query owner, workgroups of an XCD
    int xcds;                  // 2: heads are dealt out tile by tile and give the XCDs different tiles
    // by place in the queue: XCD 0's entries and XCD 7's, which have the heaviest tile of each place between them (heaviest first,
    // every other row of eight in reverse); 0 where XCD 7 has none
    float cost[2][kMax];
    // The longest walk of a workgroup.  D = 64: also of a compute unit's pair of them; while both run each takes its time, the rest of the
    // longer one takes `alone` of it
    struct Longest {
        float one, pair;
    };
    Longest passes;   // where the queue is taken pass by pass (BwdQueue::entry)
    Longest least;    // no plan's are shorter (with a mask, by pairs: none was)
    float alone, pays_one, pays_pair;
    bool keys_first;   // the key owners' tiles are the longer ones

    // Of per_xcd walks in the order of a pass, whose first and last, second and last but one, ... share a compute unit
    void longest(const float *walk, Longest &most) const
    {
        for (int m = 0; m < per_xcd; ++m)
            most.one = std::max(most.one, walk[m]);
        for (int i = 0; alone < 1.f && i < per_xcd / 2; ++i) {
            const float x = walk[i], y = walk[per_xcd - 1 - i], less = std::min(x, y);
            most.pair = std::max(most.pair, less + (std::max(x, y) - less) * alone);
        }
    }

    // Whether a launch takes the plan whose longest walks these are.  Time by plan over time by passes: D = 128, 190 launches, 0.73 to 0.98
    // where the longest walk is under 0.95 of the passes' (one of 97 1.02), 0.96 to 1.05 above.  D = 64 by single walks, under 0.93 (short
    // causal ones, whose costs are less sure, 0.8): 3000 drawn launches 0.964 in the mean, but 56 of them more than 2 % slower than by
    // passes, 1.12 times at worst: their plans level the single walks and pair long ones, where the passes pair long with short (13 heads of
    // 2210 x 3580 113.5 -> 119.5 us).  By pairs as well, which have to be under 0.96 (0.92), or under the passes' where the single walks are level:
    // 0.954, 38 and 1.07 times.
    bool pays(const Longest &l) const
    {
        const bool level = l.one < pays_one * passes.one;
        return alone < 1.f ? l.pair < pays_pair * passes.pair || (level && l.pair < passes.pair) : level;
    }

    // false: a single pass, or too many entries
    bool fill(const BwdParams &p, int BH, int causal, const WalkCost &c, int slots)
    {
        using attn::kNumXcd;
        const attn::BwdQueue queue(p.total_wg, p.total_q);
        if (queue.n_entries <= slots || slots % kNumXcd || slots / kNumXcd > attn::BwdPlan::kMaxSlots ||
            queue.n_entries > kMax * kNumXcd || !p.total_wg || !p.total_q)
            return false;
        n = (queue.n_entries + kNumXcd - 1) / kNumXcd;
        first_q = queue.q_first / kNumXcd;
        per_xcd = slots / kNumXcd;
        xcds = causal && BH % kNumXcd ? 2 : 1;
        const long long head_bytes = 4ll * (p.S_q + p.S_kv) * p.D;
        const float first_key = c.key(walk_steps(p, causal, c.rows, true, 0)),
                    last_query = c.query(walk_steps(p, causal, c.rows, false, p.n_tq - 1));   // the heaviest of either sweep
        keys_first = first_key >= last_query;
        alone = c.alone;
        const bool unsure = p.D == 64 && causal && std::min(p.S_q, p.S_kv) < 1024;
        pays_one = unsure ? 0.8f : c.plan_pays;
        pays_pair = unsure ? 0.92f : 0.96f;
        passes = {};
        least.one = std::max(first_key, last_query);
        least.pair = alone * least.one;
        for (int x = 0; x < xcds; ++x) {
            float *const of = cost[x], *at = of;
            if (causal) {
                xcd_tiles(BH, p.n_t, causal, head_bytes, x * (kNumXcd - 1),
                          [&](int t, int m) { at = std::fill_n(at, m, c.key(walk_steps(p, causal, c.rows, true, p.n_t - 1 - t))); });
                std::fill(at, of + first_q, 0.f);
                at = of + first_q;
                xcd_tiles(BH, p.n_tq, causal, head_bytes, x * (kNumXcd - 1),
                          [&](int t, int m) { at = std::fill_n(at, m, c.query(walk_steps(p, causal, c.rows, false, t))); });
                std::fill(at, of + n, 0.f);
            } else {
                std::fill(of, of + first_q, first_key);
                std::fill(of + first_q, of + n, last_query);
            }
            float walk[attn::BwdPlan::kMaxSlots] = {}, sum = 0.f;
            for (int k = 0, first = 0; first < n; ++k, first += per_xcd) {
                const int m = std::min(per_xcd, n - first);
                if (k & 1)
                    for (int i = 0; i < m; ++i)
                        walk[per_xcd - 1 - i] += of[first + i];
                else
                    for (int i = 0; i < m; ++i)
                        walk[i] += of[first + i];
            }
            longest(walk, passes);
            for (int m = 0; m < per_xcd; ++m)
                sum += walk[m];
            least.one = std::max(least.one, sum / per_xcd);
            least.pair = std::max(least.pair, sum / per_xcd);   // (a pair takes at least its mean: alone >= 0.5)
        }
        least.pair += 0.02f * passes.pair;   // (of 970 causal plans taken none came closer to the bound)
        if (!causal)
            least = two_costs(keys_first ? first_q : n - first_q, std::max(cost[0][0], cost[0][n - 1]),
                              keys_first ? n - first_q : first_q, std::min(cost[0][0], cost[0][n - 1]));
        return true;
    }

    // plan_walks's longest walks where there are only two costs: n1 tiles of l1, then n2 of l2.  Workgroups in two classes, the first
    // `more` of them one l1 apart from the others; the class that is free first takes a tile each, as far as they go
    Longest two_costs(int n1, float l1, int n2, float l2) const
    {
        const int more = n1 % per_xcd, first[2] = {more, 0}, end[2] = {per_xcd, more};
        float load[2] = {}, walk[attn::BwdPlan::kMaxSlots];
        for (int k = 0; k < n1 / per_xcd; ++k)
            load[0] += l1;
        load[1] = load[0] + l1;
        int i = 0, m = 0;   // the last tile goes to class i, up to its workgroup m
        while (n2 > 0) {
            i = load[1] <= load[0] && more > 0;
            m = std::min(first[i] + n2, end[i]);
            n2 -= m - first[i];
            if (n2 > 0 || m == end[i]) {
                load[i] += l2;
                m = 0;
            }
        }
        for (int k = 0; k < per_xcd; ++k)
            walk[k] = load[k < more];
        for (int k = first[i]; k < m; ++k)
            walk[k] += l2;
        Longest most = {};
        longest(walk, most);
        return most;
    }
};

// The plan of a launch's walks (BwdPlan): list scheduling.  The sweep with the longer tiles first, every entry of an XCD's queue, in the
// queue's order, to the workgroup that is free first.  Taking one pass through the queue after the other, odd ones backwards, leaves walks up to
// a third apart where tiles differ, by the mask or by the sweep they belong to.  By passes -> by plan, in us: D = 128, 40 causal heads
// of 1500 rows 106.7 -> 95, 12 of 6000 1.17 times as fast, 123 heads of 72 x 5938 1.12 (against one sweep after the other), 16 causal of
// 1000 x 8000 1.36; D = 64, 123 of 72 x 5938 1.36, 16 of 1000 x 8000 1.28.  The queue is sorted within a group of heads only: where
// many groups follow each other a plan can be longer than the passes (and is not taken).  Returns the longest walks.
BwdWalks::Longest plan_walks(attn::BwdPlan &plan, const BwdWalks &w, int cus)
{
    using attn::BwdPlan;
    plan = {};   // (all of it goes to the device, and set() keeps the other half of a word)
    const int per_xcd = w.per_xcd;
    // (load, workgroup) at the leaves of a tree whose nodes hold the lesser of their two: its root is free first, and one path to it is
    // renewed per entry, without branches to guess (10 ns; a binary heap takes 30).  (The bits of floats that are not negative have the
    // floats' order)
    int leaves = 1;
    while (leaves < per_xcd)
        leaves *= 2;
    uint64_t tree[2 * BwdPlan::kMaxSlots];
    for (int m = 0; m < leaves; ++m)
        tree[leaves + m] = m < per_xcd ? (uint64_t)m : ~0ull;
    for (int i = leaves - 1; i > 0; --i)
        tree[i] = std::min(tree[2 * i], tree[2 * i + 1]);
    uint8_t owner[BwdPlan::kMaxEntries];
    int of_slot[BwdPlan::kMaxSlots] = {};
    for (const bool keys : {w.keys_first, !w.keys_first})
        for (int at = keys ? 0 : w.first_q; at < (keys ? w.first_q : w.n); ++at) {
            const int m = (int)(uint32_t)tree[1];
            owner[at] = (uint8_t)m;
            ++of_slot[m];
            uint32_t bits = (uint32_t)(tree[1] >> 32);
            float load;
            memcpy(&load, &bits, sizeof load);
            load += w.xcds > 1 ? std::max(w.cost[0][at], w.cost[1][at]) : w.cost[0][at];
            memcpy(&bits, &load, sizeof load);
            uint64_t least = (uint64_t)bits << 32 | (uint32_t)m;
            for (int i = leaves + m; i > 1; i /= 2) {
                tree[i] = least;
                least = std::min(least, tree[i ^ 1]);
            }
            tree[1] = least;
        }
    // the workgroups that begin with the heaviest tiles share their compute units with those that begin with the lightest
    // (BwdQueue::entry)
    const auto place = [&](int m) { return m < cus ? m : per_xcd - 1 - (m - cus); };
    int first[BwdPlan::kMaxSlots + 1] = {};
    for (int m = 0; m < per_xcd; ++m)
        first[place(m) + 1] = of_slot[m];
    for (int m = 0; m < per_xcd; ++m)
        first[m + 1] += first[m];
    for (int m = 0; m <= per_xcd; ++m)
        BwdPlan::set(plan.first, m, first[m]);
    BwdWalks::Longest longest = {};
    for (int x = 0; x < w.xcds; ++x) {
        float walk[BwdPlan::kMaxSlots] = {};
        for (int at = 0; at < w.n; ++at)
            walk[owner[at]] += w.cost[x][at];
        w.longest(walk, longest);
    }
    for (int at = 0; at < w.n; ++at)
        BwdPlan::set(plan.idx, first[place(owner[at])]++, at);
    return longest;
}

// A launch in one tiling: its walks, the plan of them if it has one, and (D = 128) what it is estimated to take.  In three steps, as
// the host's time counts: set() asks no walks, walk() makes no plan, and `us` is the least that the next step could leave.
struct BwdLaunch {
    BwdParams p;
    const WalkCost *c;
    BwdWalks walks;
    attn::BwdPlan plan;
    float rest, us;   // what is added to the longest walk; the sum
    enum { kSet, kWalked, kDone } step;
    bool planned;

    // estimate: between tilings (D = 128); a launch that has no choice takes its walks only
    void set(const BwdParams &of, int BH, int causal, const WalkCost &cost, int cus, bool estimate)
    {
        p = of;
        c = &cost;
        p.n_t = (p.S_kv + cost.rows - 1) / cost.rows;
        p.n_tq = (p.S_q + cost.rows - 1) / cost.rows;
        p.total_wg = BH * p.n_t;
        p.total_q = BH * p.n_tq;
        planned = false;
        rest = us = 0.f;
        const int slots = cus * cost.per_cu, entries = attn::BwdQueue(p.total_wg, p.total_q).n_entries;
        step = cus <= 0 || entries <= slots || entries > BwdWalks::kMax * attn::kNumXcd ? kDone : kSet;
        if (!estimate || cus <= 0)
            return;
        // steps of a head's tiles: they fall (key owners) or rise (query owners) by rows / 32 from tile to tile while a mask cuts them
        const auto steps = [&](bool keys, int n) {
            if (!causal)
                return (double)n * walk_steps(p, 0, cost.rows, keys, 0);
            const int d = cost.rows / 32, top = (p.S_q + 31) / 32;
            if (keys) {
                const int all = (top + d - 1) / d < n ? (top + d - 1) / d : n;
                return (double)all * top - 0.5 * d * all * (all - 1.0);
            }
            const int cut = (p.S_q < p.S_kv ? p.S_q : p.S_kv) / cost.rows, m = cut < n ? cut : n;   // tiles the mask's edge runs through
            return 0.5 * d * m * (m + 1.0) + (double)(n - m) * walk_steps(p, causal, cost.rows, keys, n - 1);
        };
        const double all = BH * (p.n_t * (double)cost.key_tile + steps(true, p.n_t) * cost.key_step + p.n_tq * (double)cost.query_tile +
                                 steps(false, p.n_tq) * cost.query_step);
        const float mean = (float)(all / slots);
        const float heaviest = std::max(cost.key(walk_steps(p, causal, cost.rows, true, 0)),
                                        cost.query(walk_steps(p, causal, cost.rows, false, p.n_tq - 1)));
        rest = cost.launch + cost.mean * mean;
        us = rest + std::max(mean, heaviest);
        if (step == kDone)
            us = rest + (entries <= slots ? heaviest : mean + heaviest * (causal ? 0.25f : 0.5f));
    }
    void walk(int BH, int causal, int cus)
    {
        step = kDone;
        if (!walks.fill(p, BH, causal, *c, cus * c->per_cu))
            return;
        if (walks.pays(walks.least))
            step = kWalked;
        us = rest + (step == kWalked ? walks.least.one : walks.passes.one);
    }
    // makes the plan, and takes it if it pays
    void close()
    {
        const BwdWalks::Longest longest = plan_walks(plan, walks, p.cus_per_xcd);
        planned = walks.pays(longest);
        us = rest + (planned ? longest.one : walks.passes.one);
        step = kDone;
    }
    // the next step; false: there is none
    bool go_on(int BH, int causal, int cus)
    {
        if (step == kDone)
            return false;
        if (step == kSet)
            walk(BH, causal, cus);
        else
            close();
        return true;
    }
};

// both hand-scheduled sweeps: as many workgroups as the chip holds at once, each walking the queue of owner tiles of its
// XCD, or what a plan gives it
struct BwdKernels {
    void (*plain)(const BwdParams);
    void (*planned)(const BwdParams, const attn::BwdPlan);
};
int launch_sweeps(const BwdKernels &kern, int threads, int LDS, const BwdLaunch &l, int causal, hipStream_t stream)
{
    // Workgroups of a kernel that the chip holds, 0 if its LDS is refused.  (A runtime that cannot tell the occupancy gets one
    // workgroup per entry: the kernel takes either)
    const auto slots_of = [&](const void *k) {
        if (!attn::allow_lds(k, LDS))   // (ahead of the occupancy, which it is part of)
            return 0;
        const int n = attn::persistent_slots(k, threads, LDS, attn::kNumXcd);
        return n < attn::kNumXcd ? 0x7fffffff : n;
    };
    // (all of a plan's workgroups have to run at once: as many as the planned kernel fits)
    if (l.planned && slots_of(reinterpret_cast<const void *>(kern.planned)) == l.walks.per_xcd * attn::kNumXcd) {
        hipLaunchKernelGGL(kern.planned, dim3((unsigned)(l.walks.per_xcd * attn::kNumXcd)), dim3(threads), LDS, stream, l.p, l.plan);
        return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
    }
    const int slots = slots_of(reinterpret_cast<const void *>(kern.plain));
    if (slots == 0)
        return ATTN_ERR_LAUNCH;
    const auto run = [&](int n_kv, int n_q) {
        BwdParams r = l.p;
        r.total_wg = n_kv;
        r.total_q = n_q;
        const int entries = attn::BwdQueue(n_kv, n_q).n_entries;
        hipLaunchKernelGGL(kern.plain, dim3((unsigned)(slots < entries ? slots : entries)), dim3(threads), LDS, stream, r);
        return (int)(hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH);
    };
    const bool rows64 = l.c == &kWalk256 || l.c == &kWalk128TwoWaves;
    if ((rows64 && causal) || !sweeps_apart(l.p, causal, slots))
        return run(l.p.total_wg, l.p.total_q);
    const int rc = run(l.p.total_wg, 0);
    return rc == ATTN_OK ? run(0, l.p.total_q) : rc;
}

// D = 128: which owner tiles a launch takes.  64-row waves read half the LDS operands per product: in tiles of 256 rows (four
// waves, half the stream as well) long walks on a full chip are 8 to 11 % faster than in tiles of 128 rows and 32-row waves (32
// heads of 2048 rows 206 -> 187 us, 128 of 4096 3026 -> 2691); in tiles of 128 rows (two waves, two workgroups to a CU that
// fill each other's gaps) causal and ragged launches (128 causal heads of 4096 rows 1673 -> 1516, of 1024 147 -> 140, 300 of
// 300 rows 91 -> 84).  A 64-row wave takes 1.6 times as long for a tile as a 32-row one: launches that do not fill the chip are
// up to 1.7 times slower (16 heads of 1024 rows 35 -> 44).  The estimate rests on the
// walk that the launch then has, by plan or by passes.  Of 6170 launches (1 to 256 heads, 64 to 16384 rows) 29 % take 64-row waves, 8 % faster in the
// mean; 12 of those 1795 are more than 2 % slower, 1.08 times at worst.  (Where any of them was taken to have a plan little above its mean
// walk, 62 were, 1.12 times at worst.)
BwdTiling pick_tiling(const BwdParams &p, int BH, int causal, int cus, BwdLaunch (&l)[3])
{
    const bool all = cus >= attn::kNumXcd && 2ll * BH * ((p.S_kv + 255) / 256 + (p.S_q + 255) / 256) >= cus;   // (no launch of fewer tiles gained)
    l[0].set(p, BH, causal, kWalk128, cus, all);
    if (all) {
        l[1].set(p, BH, causal, kWalk256, cus, true);
        l[2].set(p, BH, causal, kWalk128TwoWaves, cus, true);
    }
    for (;;) {   // the least estimate, worked out only where it could be that
        // (the two factors by the same launches: 1.3 % of them are left more than 3 % behind their best tiling, 1.8 % at 0.975 and 1)
        const float t32 = 0.98f * l[0].us, t256 = (l[1].planned ? 1.01f : 1.f) * l[1].us;
        const int i = !all || (t32 <= t256 && t32 <= l[2].us) ? 0 : t256 <= l[2].us ? 1 : 2;
        if (!l[i].go_on(BH, causal, cus))
            return i == 0 ? kRows128 : i == 1 ? kRows256 : kRows128TwoWaves;
    }
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
    const int cus = attn::cu_count(attn::kNumXcd);
    p.cus_per_xcd = cus > 0 ? cus / attn::kNumXcd : 32;
    const int rc = launch_delta<D, typename std::conditional<F16, _Float16, attn::bf16_t>::type>(p, stream);
    if (rc != ATTN_OK)
        return rc;
    // (while the Delta kernel runs)
    BwdLaunch launch[3];
    if (D == 128 && tiling == kAsDispatched) {
        tiling = pick_tiling(p, BH, causal, cus, launch);
    } else {
        tiling = D == 128 ? tiling : kRows128;
        BwdLaunch &l = launch[tiling - kRows128];
        l.set(p, BH, causal, D == 64 ? kWalkD64 : tiling == kRows128 ? kWalk128 : tiling == kRows256 ? kWalk256 : kWalk128TwoWaves, cus, false);
        while (l.go_on(BH, causal, cus)) {
        }
    }
    const BwdLaunch &l = launch[tiling - kRows128];
    const auto run = [&](const BwdKernels &kern, int threads, int lds) { return launch_sweeps(kern, threads, lds, l, causal, stream); };
    using namespace attn;
    if constexpr (D == 128) {
        if (tiling == kRows256)
            return causal ? run({attn_bwd_wide_kernel<4, true, F16>, attn_bwd_wide_planned_kernel<4, true, F16>}, 256, BwdWideLds<4>::BYTES)
                          : run({attn_bwd_wide_kernel<4, false, F16>, attn_bwd_wide_planned_kernel<4, false, F16>}, 256, BwdWideLds<4>::BYTES);
        if (tiling == kRows128TwoWaves)
            return causal ? run({attn_bwd_wide_kernel<2, true, F16>, attn_bwd_wide_planned_kernel<2, true, F16>}, 128, BwdWideLds<2>::BYTES)
                          : run({attn_bwd_wide_kernel<2, false, F16>, attn_bwd_wide_planned_kernel<2, false, F16>}, 128, BwdWideLds<2>::BYTES);
    }
    return causal ? run({attn_bwd_asm_kernel<D, true, F16>, attn_bwd_asm_planned_kernel<D, true, F16>}, 256, BwdLds<D>::BYTES)
                  : run({attn_bwd_asm_kernel<D, false, F16>, attn_bwd_asm_planned_kernel<D, false, F16>}, 256, BwdLds<D>::BYTES);
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
    p.D = D;
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

// Test-only, host only: a launch's plan; the longest walk over that of the passes, 1 without walks (BwdWalks::fill).  walks, in us: the longest
// by plan and by passes, what no order goes below, then XCD 0's entries.
extern "C" float attn_bwd_plan_walks(int heads, int S_q, int S_kv, int D, int causal, int tiling, int cus, uint32_t *first, uint32_t *idx,
                                     float *walks)
{
    const WalkCost &c = D == 64 ? kWalkD64 : tiling == kRows256 ? kWalk256 : tiling == kRows128 ? kWalk128 : kWalk128TwoWaves;
    BwdParams p;
    p.S_q = S_q;
    p.S_kv = S_kv;
    p.D = D;
    p.n_t = (S_kv + c.rows - 1) / c.rows;
    p.n_tq = (S_q + c.rows - 1) / c.rows;
    p.total_wg = heads * p.n_t;
    p.total_q = heads * p.n_tq;
    attn::BwdPlan plan;
    BwdWalks w;
    if (!w.fill(p, heads, causal, c, cus * c.per_cu))
        return 1.f;
    walks[0] = plan_walks(plan, w, cus / attn::kNumXcd).one;
    walks[1] = w.passes.one;
    walks[2] = w.least.one;
    std::copy(w.cost[0], w.cost[0] + w.n, walks + 3);
    for (int i = 0; i < (int)(sizeof plan.first / 4); ++i)
        first[i] = plan.first[i];
    for (int i = 0; i < (int)(sizeof plan.idx / 4); ++i)
        idx[i] = plan.idx[i];
    return walks[0] / walks[1];
}

extern "C" float attn_bwd_plan(int heads, int S_q, int S_kv, int D, int causal, int tiling, int cus, uint32_t *first, uint32_t *idx)
{
    float walks[3 + BwdWalks::kMax];
    return attn_bwd_plan_walks(heads, S_q, S_kv, D, causal, tiling, cus, first, idx, walks);
}

// Test-only, host only: the i-th tile that an XCD takes up of a sweep (xcd_tiles), -1 behind the last, and the same from
// wg_to_tile_n in *want.
extern "C" int attn_bwd_xcd_tile(int heads, int n_t, int causal, long long head_bytes, int xcd, int i, int *want)
{
    int at = 0, got = -1, bh = 0, t = -1;
    const long long entry = (long long)attn::kNumXcd * i + xcd;
    xcd_tiles(heads, n_t, causal, head_bytes, xcd, [&](int x, int n) {
        got = at <= i && i < at + n ? x : got;
        at += n;
    });
    if (causal && entry < (long long)heads * n_t)
        attn::wg_to_tile_n<true>((int)entry, heads * n_t, n_t, head_bytes, bh, t);
    *want = causal ? t : entry < (long long)heads * n_t ? 0 : -1;
    return got;
}

// Test-only, host only: the tiling that a D = 128 launch on `cus` compute units takes (1: tiles of 128 rows and 32-row waves, 2: of
// 256 rows, 3: of 128 rows and 64-row waves) and the three estimates in us, of the others the least that they could come to.
// walk: the longest walk that the taken tiling's estimate rests on, and whether it has a plan.
extern "C" int attn_bwd_picked_walk(int heads, int S_q, int S_kv, int causal, int cus, float *est, float *walk)
{
    BwdParams p;
    p.S_q = S_q;
    p.S_kv = S_kv;
    p.D = 128;
    p.cus_per_xcd = cus / attn::kNumXcd;
    BwdLaunch l[3];
    l[1].us = l[2].us = -1.f;
    const BwdTiling t = pick_tiling(p, heads, causal, cus, l);
    if (l[1].us < 0.f) {
        l[0].set(p, heads, causal, kWalk128, cus, true);
        l[1].set(p, heads, causal, kWalk256, cus, true);
        l[2].set(p, heads, causal, kWalk128TwoWaves, cus, true);
    }
    for (int i = 0; i < 3; ++i)
        est[i] = l[i].us;
    walk[0] = l[t - kRows128].us - l[t - kRows128].rest;
    walk[1] = l[t - kRows128].planned;
    return t;
}

extern "C" int attn_bwd_pick_tiling(int heads, int S_q, int S_kv, int causal, int cus, float *est)
{
    float walk[2];
    return attn_bwd_picked_walk(heads, S_q, S_kv, causal, cus, est, walk);
}

// Test-only: attn_bwd / attn_bwd_f16 (D = 128, scale > 0) in the tiling that is asked for (BwdTiling).
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
