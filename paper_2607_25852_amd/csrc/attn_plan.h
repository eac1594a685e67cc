// Work plan of the persistent verify-attention kernel, built by one workgroup.
//
// Every kv-head has the same work, so the plan is made for one head. A unit is a (request, row
// block), a run of 64-token tiles of the request's context; the units are laid end to end on a
// line and the line is cut into ranges of equal cost. A work item is one range of one head, one
// item per compute unit: the end of one unit, any number of whole units, the start of another.
// A unit that a cut falls into leaves one fp32 partial result per piece, which the merge kernel
// combines; an uncut unit is written directly. So the chip is filled evenly whatever the
// lengths are, and at most one unit per cut needs a merge. The heads of a range are
// neighbouring items, which run at the same time and read the same pages.
// Used by the attention call's own plan kernel and by the round set-up kernel
// (sv_prepare_round), so both build the same plan.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "rows.h"

namespace sv {

constexpr int kAttnTile = 64;       // KV tokens per tile of the attention kernel
constexpr int kPlanMinTiles = 6;    // no range is shorter unless the line is
constexpr int kPlanGrid = 256;      // compute units
constexpr int kPlanUnits = 2 * kPlanGrid;  // from this many units on the work is a list (attn_list.hip)
constexpr int kPlanSnapTiles = 2;   // a cut this close to a unit's end is moved onto it
// Cost of a unit, in sixteenths of the time of one tile of a unit of at most 64 query rows
// (bound by its K/V stream): its start and end (descriptors, page ids, queries, the first
// tile's latency, the merge of the token halves: 6.3 us, 9.8 us above 64 rows) and its tiles.
// Above 64 rows the tile's matrix and vector work shows (1.3 against 1.05 us), and above 128
// rows (whole-tile waves) the chain of dependent steps bounds the tile (1.9 us).
constexpr unsigned kCostStart = 100, kCostStart65 = 144, kCostTile = 16, kCostTile65 = 20, kCostWideTile = 32;
// Workgroups on the odd XCDs end 3 to 4% later than those on the even ones with the same work
// (attention over 188 MB to 6.4 GB, several cards), so their ranges are this many 1024ths
// shorter and the others' longer.
constexpr unsigned kOddXcd = 17;
static_assert(kPlanUnits * (kCostStart65 + (uint64_t)kCostWideTile * ((1 << 22) / kAttnTile)) < 1u << 31,
              "the cost of a line, and a step more, fit 32 bits");

// one cut of the line: the range starts at this tile of this unit. The request's packing and
// key count go with it, which saves the readers a dependent load.
struct __attribute__((aligned(16))) AttnRange {
    int32_t req, block, tile, q0;
    int32_t k, kv, pad0, pad1;
};

struct AttnPlanArgs {
    int R, block, total_q, max_kv_len, G, nrb;
    int rb_rows;       // query rows per row block
    int ranges;        // most ranges per head the workspace holds
    int heads;         // kv-heads
    AttnRange* recs;   // [ranges + 1]
    int32_t* ctr;      // {ranges per head, claim counter, finished workgroups}
};

// ranges per head of a plan whose count reads `stored` (any word, where no plan was built): never
// negative, so that its product with the heads is at most that of `most`, which the host checks
__device__ inline int plan_ranges(int stored, int most) { return stored < 0 ? 0 : stored < most ? stored : most; }

// tiles of request i's context, 0 when its packing is malformed
__device__ inline int plan_tiles(int block, int total_q, int max_kv_len, int q0, int k_i, int kv_len) {
    if (kv_len > max_kv_len) kv_len = max_kv_len;
    const int nt = (int)((unsigned)(kv_len + kAttnTile - 1) / kAttnTile);
    return (rows_in_batch(q0, k_i, block, total_q) & (kv_len >= k_i)) ? nt : 0;
}

// cost per tile and of the start of a unit with M query rows
__device__ inline unsigned plan_tile_cost(int M) { return M > 128 ? kCostWideTile : M > 64 ? kCostTile65 : kCostTile; }
__device__ inline unsigned plan_start_cost(int M) { return M > 64 ? kCostStart65 : kCostStart; }
__device__ inline unsigned plan_unit_cost(int M, int nt) {
    if (M <= 0 || nt <= 0) return 0;
    return plan_start_cost(M) + (unsigned)nt * plan_tile_cost(M);
}
__device__ inline unsigned plan_head_cost(const AttnPlanArgs& a, int k_i, int nt) {
    unsigned c = 0;
    for (int rb = 0; rb < a.nrb; rb++) c += plan_unit_cost(a.G * k_i - rb * a.rb_rows, nt);
    return c;
}

// NT threads of one workgroup. pre: R + 1 entries of LDS, wsum: NT / 64 entries of LDS.
// req(i, q0, k_i, kv_len) gives request i's packing and key count. The caller's kernel end
// publishes the plan. Costs are 32 bits: ranges are for fewer than kPlanUnits units, each of at
// most 2^16 tiles.
template <int NT, typename ReqFn>
__device__ inline void build_attn_plan(const AttnPlanArgs& a, ReqFn req, uint32_t* pre, uint32_t* wsum) {
    static_assert(NT % 64 == 0, "plan threads");
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // 1. cost before each request, one request per thread at a time
    uint32_t W = 0;  // the cost of the line so far
    for (int i0 = 0; i0 < a.R; i0 += NT) {
        const int i = i0 + tid;
        uint32_t cost = 0;
        if (i < a.R) {
            int q0, k_i, kv;
            req(i, q0, k_i, kv);
            cost = plan_head_cost(a, k_i, plan_tiles(a.block, a.total_q, a.max_kv_len, q0, k_i, kv));
        }
        uint32_t incl = cost;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t v = __shfl_up(incl, off, 64);
            if (lane >= off) incl += v;
        }
        uint32_t before = W;
        if constexpr (NT == 64) {
            W += __shfl(incl, 63, 64);
        } else {
            if (lane == 63) wsum[w] = incl;
            __syncthreads();
            for (int k = 0; k < NT / 64; k++) {
                if (k < w) before += wsum[k];
                W += wsum[k];
            }
            __syncthreads();  // (the sums of the next requests go to the same place)
        }
        if (i < a.R) pre[i] = before + incl - cost;
    }
    __syncthreads();
    // 2. the size of the ranges
    constexpr uint32_t least = kCostStart + kPlanMinTiles * kCostTile;
    const uint32_t even = (W + (uint32_t)a.ranges - 1) / (uint32_t)a.ranges;
    // A line too short for that (far below the longest contexts the host allows for) leaves compute
    // units idle: there a range starts at every unit, and only long units are cut.
    const uint32_t step = even < least / 2 ? least / 2 : even;
    const bool brief = step < least;
    const int n = (int)((W + step - 1) / step);  // (at most a.ranges)
    // the items of a range share an XCD when its workgroups hold whole ranges (attn.hip)
    const bool skewed = n > 0 && n % 8 == 0 && n * a.heads <= kPlanGrid;
    // 3. the cuts: the request by binary search over the costs, then row block and tile
    for (int r = tid; r <= n; r += NT) {
        uint32_t at = (uint32_t)r * step;
        if (skewed) {  // (per XCD the ranges' sizes sum to per * step on average over two XCDs)
            const unsigned per = (unsigned)n / 8, x = (unsigned)r / per, k = (unsigned)r % per;
            at += (x & 1 ? per - k : k) * (step * kOddXcd / 1024);
        }
        AttnRange rec{a.R, 0, 0, 0, 0, 0, 0, 0};
        if (r < n && at < W) {
            int lo = 0, hi = a.R - 1;  // the last request whose cost starts at or before `at`
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (pre[mid] <= at) lo = mid;
                else hi = mid - 1;
            }
            int q0, k_i, kv;
            req(lo, q0, k_i, kv);
            const int nt = plan_tiles(a.block, a.total_q, a.max_kv_len, q0, k_i, kv);
            unsigned x = at - pre[lo];
            int rb = 0;
            unsigned uc = plan_unit_cost(a.G * k_i, nt);
            while (x >= uc && rb + 1 < a.nrb) {
                x -= uc;
                rb++;
                uc = plan_unit_cost(a.G * k_i - rb * a.rb_rows, nt);
            }
            const unsigned start = plan_start_cost(a.G * k_i - rb * a.rb_rows);
            int t = x > start ? (int)((x - start) / plan_tile_cost(a.G * k_i - rb * a.rb_rows)) : 0;
            if (t <= kPlanSnapTiles || (brief && nt < 2 * kPlanMinTiles)) t = 0;
            if (t >= nt || (nt - t <= kPlanSnapTiles && t > 0)) {
                t = 0;
                rb++;
            }
            rec = AttnRange{lo, rb, t, q0, k_i, kv, 0, 0};
        }
        a.recs[r] = rec;
    }
    if (tid == 0) {
        a.ctr[0] = n;
        a.ctr[1] = 0;
        a.ctr[2] = 0;
    }
}

// A grid takes n items in one pass when it has a workgroup for each of them on every XCD, that is
// for 8 * ceil(n / 8) of them; else its workgroups go on claiming items.
__device__ inline bool plan_one_pass(int n, int grid) { return n <= grid / 8 * 8; }

// The item of workgroup (or claim) `index`, -1 past the last. Workgroups go to the 8 XCDs
// round-robin: in one pass each XCD takes a contiguous part of the items, so that the heads of a
// range, whose K/V blocks are neighbours in every page, run on one XCD and share its address
// translations.
__device__ inline int plan_item(int index, int n, bool one_pass) {
    const unsigned per_xcd = ((unsigned)n + 7) / 8, x = (unsigned)index;
    const unsigned item = !one_pass ? x : x / 8 < per_xcd ? x % 8 * per_xcd + x / 8 : 0xFFFFFFFFu;
    return item < (unsigned)n ? (int)item : -1;
}

// Calls piece(i, row0, q0, k_i, kv_len, t0, t1, nt) for each piece of the range between two cuts:
// request i's rows from row0 of the kv-head group on (row block row0 / rb_rows) against tiles
// t0 .. t1-1 of the nt tiles of its context. req(i, q0, k_i, kv_len) gives the packing and key
// count of the requests after the first, which the cut itself carries. The cuts may hold any
// words: every piece lies in its request and its request in the batch.
template <typename Args, typename ReqFn, typename PieceFn>
__device__ __forceinline__ void walk_range(const Args& a, const AttnRange& r0, const AttnRange& r1, int rb_rows,
                                           ReqFn req, PieceFn piece) {
    int rb = r0.block, t = r0.tile;
    for (int i = max(r0.req, 0); i <= r1.req && i < a.R; i++, rb = 0, t = 0) {
        int q0 = r0.q0, k_i = r0.k, kv_len = r0.kv;
        if (i != r0.req) req(i, q0, k_i, kv_len);
        kv_len = min(kv_len, a.max_kv_len);
        const int nt = plan_tiles(a.block, a.total_q, a.max_kv_len, q0, k_i, kv_len);
        if (nt == 0) continue;
        const int rb_end = i == r1.req ? min(r1.block, a.nrb - 1) : a.nrb - 1;  // (the last unit, cut or whole)
        for (rb = max(rb, 0); rb <= rb_end; rb++, t = 0) {
            const int row0 = rb * rb_rows;
            const int t0 = max(t, 0), t1 = i == r1.req && rb == r1.block ? min(r1.tile, nt) : nt;
            if (t0 >= t1 || a.G * k_i <= row0) continue;
            piece(i, row0, q0, k_i, kv_len, t0, t1, nt);
        }
    }
}

}  // namespace sv
