// The plan of the streaming attention kernel: whose its spans are, where they are cut, and what each of them reads first.
// Included by attn_mfma.hip (a kernel of its own) and attn_unit.hip (workgroups behind those of a short call).
#pragma once

#include "common.h"
#include "span_cuts.h"

namespace ss {
namespace {

// ---------------------------------------------------------------------------------------------
// plan: workgroup (p, g0) writes the flat list of tile pair addresses of some units (KV heads g0 .. g0 + heads - 1 of the request at
// place p of the layout) and the descriptors of the waves whose span starts inside them; (p, 0) publishes the request's record, one
// workgroup the plan's.
//
// Where the spans are cut.  A wave (a workgroup, in the team kernels) pays a fixed price for every unit it opens (query loads, a
// drained ring of pairs, the partial of the unit before), so equal pair counts do not finish together: on a ragged batch the
// waves that cross ten short units were 10 % late.  The cuts are therefore equal in a weighted coordinate in which every unit is
// what opening it costs followed by its pairs; a cut that falls into a unit's opening becomes the unit's first
// pair.  The cuts depend on the batch's lengths only, so results do not vary from run to run.
//
// Classes.  A team kernel has code for every number of row blocks up to its own, and the requests of a call usually differ in it
// (their depths are chosen one by one).  The plan lays the requests out by row blocks, the most first, so that a span is one run of
// units of equal row blocks, seldom two.  96 requests of 512..8192 tokens, e4m3, 64 heads over 8, depth 2..8 (two to five row blocks):
// a call took 238 us with every unit walked by the code for five, 221 this way; 128 requests of 128..16384, 32 heads over 8, depth 0..8
// (one to three): 280 either way (bound by memory); decode step of two layers of trees of 4..8 nodes, e4m3: 145 and 132.
//
// What a unit's place needs to know of the other requests: up to kPlanLanes requests every wavefront reads all of them, up to eight
// to a lane (four with classes), and sums for itself, with one barrier for what the descriptors look up; a larger batch is laid out
// by a kernel of one workgroup in front (attn_layout_kernel), where every workgroup of the plan would walk the whole batch.  Measured
// with three row blocks, against a sort in rounds of 256 requests by every workgroup: 65 requests over 8 KV heads 9.2 -> 7.3 us, 256
// 13.2 -> 8.3, 300 18.7 -> 4.7 and 6.4 (two kernels), 1000 over two 25.4 -> 12.4, 4096 over one 177 -> 22.  (Without classes, cuts
// and layout by one prefix of the batch took 6.5, 9.0, 10.7, 12.3 and 39.6.)  Where the layout kernel begins to pay, eight to a lane
// against layout and plan: without classes 257 requests over one KV head 7.6 / 4.2 + 5.9 us, 400 over one 6.4 / 4.2 + 4.6, 257 over
// eight 10.7 / 4.8 + 8.1, 512 over eight 10.9 / 4.7 + 8.8, and a launch less; with classes 300 over eight 12.4 / 4.8 + 7.6, 400 over
// two 10.9 / 4.7 + 4.9 (the call 36.1 / 35.0).
// ---------------------------------------------------------------------------------------------
constexpr int kPlanLanes = 512, kPlanLanesClasses = 256, kPlanGroups = 512;

// Inclusive scan over a wavefront's lanes (values >= 0, 0 is neutral for `op`) by data-parallel moves: a scan by shuffles is six
// LDS round trips, 0.3 us of the plan's 5.
template <typename Op>
__device__ __forceinline__ int wave_scan_int(int x, Op op)
{
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));   // row_shr 1, 2, 4, 8: inside each row of 16 lanes
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));   // row_bcast 15: row 0 to row 1, row 2 to row 3
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));   // row_bcast 31: rows 0 and 1 to rows 2 and 3
    return x;
}
struct Add {
    __device__ __forceinline__ int operator()(int x, int y) const { return x + y; }
};
struct Max {
    __device__ __forceinline__ int operator()(int x, int y) const { return max(x, y); }
};
template <typename Op>
__device__ __forceinline__ int wave_total(int x, Op op)
{
    return __builtin_amdgcn_readlane(wave_scan_int(x, op), 63);
}

// Costs for the cuts of the class kernels, in eighths of a pair of a unit with one row block: of a pair and of opening a unit, with
// 1 .. 5 row blocks, for bf16 and e4m3 caches.  For teams measured by sweeps over nine bf16 and seven e4m3 batches (uniform and mixed row blocks, short
// and long units); half or twice the opening costs are 1 to 4 % slower, pair costs between equal and 8 : 12 within 3 %.  For wavefronts by
// themselves over 90 batches of 80 to 256 requests: half of these opening costs 2 % slower, twice 1 %.
constexpr int kPairCost[2][kMaxClasses] = {{8, 8, 8, 9, 9}, {8, 8, 9, 9, 10}};
constexpr int kOpenCost[2][kMaxClasses] = {{32, 48, 80, 100, 128}, {64, 96, 160, 220, 280}};
constexpr int kOpenCostAlone[kMaxClasses] = {24, 32, 44, 52, 68};
// Packed for SpanClasses, class 0 being five row blocks.
constexpr uint64_t pack_costs(const int (&v)[kMaxClasses], int bits)
{
    uint64_t x = 0;
    for (int k = 0; k < kMaxClasses; ++k) x |= (uint64_t)v[kMaxClasses - 1 - k] << (bits * k);
    return x;
}

// Request i: pairs per KV head, and its class (the most row blocks first; a kernel of one or two row blocks has one class).
__device__ __forceinline__ void plan_request(const AttnArgs &a, int L, int q_len, int &n, int &cls)
{
    n = window_pairs(L, q_len, a.q_lo);
    const int blocks = (window_q_len(q_len, a.q_lo, a.q_win) * (a.num_q_heads / a.num_kv_heads) + 15) >> 4;
    cls = a.team_blocks ? a.team_blocks - max(blocks, 1) : 0;
}

// How a call is cut: filled in from the classes' requests and pairs and the longest unit's pairs.
struct Cut {
    SpanClasses classes;
    SpanCuts cuts;
    long long total;   // pairs of all units
    int mode;

    __device__ __forceinline__ void choose(const AttnArgs &a, int longest)
    {
        const bool kv8 = a.kv_dtype == SS_FP8_E4M3;
        total = (long long)classes.x[kMaxClasses - 1] * a.num_kv_heads;
        const SpanChoice c = choose_spans(total, longest, (long long)a.batch * a.num_kv_heads, a.launch_waves, a.team_blocks > 0, kv8);
        mode = c.mode;
        cuts.nw = c.spans;
        constexpr uint64_t every = 0x001001001001001ull;   // one weight for all classes
        if (c.whole) {   // a unit counts one, whatever its pairs
            classes.cost = 0;
            classes.weight = every;
        } else if (a.team_blocks) {
            const int skip = kMaxClasses - a.team_blocks;   // classes with more row blocks than the kernel has
            classes.cost = (kv8 ? pack_costs(kPairCost[1], 8) : pack_costs(kPairCost[0], 8)) >> (8 * skip);
            if (a.auto_weight)
                classes.weight = (mode == kSpanAlone ? pack_costs(kOpenCostAlone, 12) : kv8 ? pack_costs(kOpenCost[1], 12) : pack_costs(kOpenCost[0], 12)) >> (12 * skip);
            else
                classes.weight = every * (uint64_t)(a.unit_weight * 8 * (mode == kSpanTeam ? kWavesPerWg : 1));
        } else {   // What a team pays for opening a unit: 4 to 8 pairs are level with one or two row blocks.
            classes.cost = 1;
            classes.weight = (uint64_t)(mode == kSpanTeam ? a.unit_weight * 2 : a.unit_weight);
        }
        cuts.total_w = classes.total() * a.num_kv_heads;
    }
    __device__ __forceinline__ void publish(const AttnArgs &a) const
    {
        AttnPlan &plan = *a.plan;
        plan.total_pairs = (int)total;
        plan.mode = mode;
        plan.spans = (int)cuts.nw;
        plan.total_cost = cuts.total_w;
#pragma unroll
        for (int c = 0; c < kMaxClasses; ++c) {
            plan.class_req[c] = classes.end[c];
            plan.class_x[c] = classes.x[c] * a.num_kv_heads;
            plan.class_cost[c] = classes.cost_of(c);
            plan.class_weight[c] = classes.weight_of(c);
        }
    }
};

// The work of workgroup `block` of the plan, done by the first 256 threads of a workgroup.
//   SLOTS   requests to a lane; 0: the batch has been laid out by attn_layout_kernel
//   places  LDS: of the requests, in layout order (SLOTS * 64)
struct Place {
    int b, L, n;
};
template <int SLOTS>
__device__ __forceinline__ void plan_block(const AttnArgs &a, int heads, int block, Place *places)
{
    constexpr bool LAID = SLOTS == 0;
    constexpr int N = LAID ? 1 : SLOTS;
    const int groups = a.num_kv_heads / heads;
    const int p = block / groups, g0 = block % groups * heads;   // place in the layout, first KV head
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    Cut cut;
    AttnReq own;
    if constexpr (LAID) {
        own = a.req[p];
        const AttnPlan &plan = *a.plan;
        cut.total = plan.total_pairs;
        cut.mode = plan.mode;
        cut.cuts.nw = plan.spans;
        cut.cuts.total_w = plan.total_cost;
    } else {
        int L[N], q0[N], q1[N], n[N], c[N], place[N];
#pragma unroll
        for (int s = 0; s < N; ++s) {   // (all of them on their way before the first is used)
            const int i = min(s * 64 + lane, a.batch - 1);
            L[s] = a.kv_len[i];
            q0[s] = a.q_indptr[i];
            q1[s] = a.q_indptr[i + 1];
        }
        int longest = 0;
#pragma unroll
        for (int s = 0; s < N; ++s) {
            plan_request(a, L[s], q1[s] - q0[s], n[s], c[s]);
            if (s * 64 + lane >= a.batch) {
                n[s] = 0;
                c[s] = kMaxClasses;
            }
            longest = max(longest, n[s]);
            place[s] = -1;
        }
        const int classes = max(a.team_blocks, 1);
        int end = 0, x = 0;
#pragma unroll
        for (int k = 0; k < kMaxClasses; ++k) {
            if (k < classes) {
                int pairs = 0;
                const int before = end;
#pragma unroll
                for (int s = 0; s < N; ++s) {
                    const unsigned long long m = __ballot(c[s] == k);
                    if (c[s] == k) {
                        place[s] = end + __popcll(m & ((1ull << lane) - 1));
                        pairs += n[s];
                    }
                    end += __popcll(m);
                }
                if (end > before) x += wave_total(pairs, Add());
            }
            cut.classes.end[k] = end;
            cut.classes.x[k] = x;
        }
        cut.choose(a, wave_total(longest, Max()));
        own.cls = cut.classes.of(p);
        int pre = 0;
#pragma unroll
        for (int s = 0; s < N; ++s) {
            if (place[s] >= 0 && place[s] < p) pre += n[s];
            const unsigned long long m = __ballot(place[s] == p);
            if (m) {
                const int from = __builtin_ctzll(m);
                own.b = s * 64 + from;
                own.L = __builtin_amdgcn_readlane(L[s], from);
                own.q0 = __builtin_amdgcn_readlane(q0[s], from);
                own.q1 = __builtin_amdgcn_readlane(q1[s], from);
                own.n = __builtin_amdgcn_readlane(n[s], from);
            }
            if ((s & 3) == wave && place[s] >= 0) places[place[s]] = Place{s * 64 + lane, L[s], n[s]};
        }
        __syncthreads();   // (`places`; nothing but LDS is on its way)
        own.pre = wave_total(pre, Add());
        own.cpre = cut.classes.start(p, own.pre, own.cls);
        if (g0 == 0 && tid == 0) {
            a.req[p] = own;
            if (p == a.batch - 1) cut.publish(a);
        }
    }
    const int per = cut.mode == kSpanTeam ? kWavesPerWg : 1;   // wavefronts that share a span
    const int n = own.n;
    // (a pair whose second tile lies past the cache's end repeats the first; its slots are never visible)
    auto pair_at = [&](int b, int L, int t, int gg) {
        const int32_t *table = a.block_table + (long long)b * a.max_blocks;
        const int b0 = table[2 * t], b1 = 2 * t + 1 < (L + kTile - 1) / kTile ? table[2 * t + 1] : b0;
        return make_int2(b0 * a.num_kv_heads + gg, b1 * a.num_kv_heads + gg);
    };
    const long long off0 = (long long)own.pre * a.num_kv_heads;   // the request's place in the flat list
    for (int t = 255 - tid; t < n; t += 256) {   // (from the last wavefront on: the first one has the descriptors)
        const int2 addr = pair_at(own.b, own.L, t, 0);
        for (int g = g0; g < g0 + heads; ++g) a.pair_addr[off0 + (long long)g * n + t] = make_int2(addr.x + g, addr.y + g);
    }

    // waves (or teams) whose cut falls into this unit's stretch [ya, ye) of the weighted coordinate
    const SpanCuts &cuts = cut.cuts;
    int cost, weight, class_end;
    if constexpr (LAID) {
        cost = a.plan->class_cost[own.cls];
        weight = a.plan->class_weight[own.cls];
        class_end = a.plan->class_x[own.cls];
    } else {
        cost = cut.classes.cost_of(own.cls);
        weight = cut.classes.weight_of(own.cls);
        class_end = 0;
#pragma unroll
        for (int k = 0; k < kMaxClasses; ++k)
            if (k == own.cls) class_end = cut.classes.x[k] * a.num_kv_heads;
    }
    for (int g = g0; g < g0 + heads; ++g) {
        const long long off = off0 + (long long)g * n;
        const long long ya = own.cpre * a.num_kv_heads + (long long)g * (weight + (long long)n * cost), ye = ya + weight + (long long)n * cost;
        const long long w_lo = cuts.first_cut_at_or_after(ya);   // first w with w*total_w/nw >= ya
        const long long w_hi = min(cuts.first_cut_at_or_after(ye), cuts.nw);   // first w at or past the unit's end
        // Descriptor: {place in the layout, KV head, first pair, class, span begin, end of the span's first class, kv_len, first query
        // row, end query row, addresses of the first kDescPairs tile pairs the wave reads, team, request, pairs of the unit}: everything
        // the wave's first loads depend on, so that they go out after a single read.
        for (long long i = w_lo * per + tid; i < w_hi * per; i += 256) {
            const long long w = i / per;
            const int t0 = SpanCuts::first_pair(cuts.cut(w), ya, weight, cost);
            int32_t *d = a.wave_desc + i * kDescInts;
            d[0] = p; d[1] = g; d[2] = t0; d[3] = own.cls;
            d[4] = (int)(off + t0); d[5] = class_end;
            d[6] = own.L; d[7] = own.q0; d[8] = own.q1;
            d[15] = cut.mode; d[16] = own.b; d[17] = n;
            // walk forward from (p, g, pair) over unit boundaries; past the last unit repeat the unit's pair
            Place at = {own.b, own.L, n};
            int pp = p, gg = g, tt = t0 + (int)(i - w * per);
            Place from[kDescPairs];
            int pair[kDescPairs], head[kDescPairs];
#pragma unroll
            for (int j = 0; j < kDescPairs; ++j) {
                while (pp < a.batch && tt >= at.n) {
                    tt -= at.n;
                    if (++gg == a.num_kv_heads) {
                        gg = 0;
                        if (++pp < a.batch) {
                            if constexpr (LAID) {
                                const AttnReq r = a.req[pp];
                                at = Place{r.b, r.L, r.n};
                            } else {
                                at = places[pp];
                            }
                        }
                    }
                }
                const bool in = pp < a.batch;
                from[j] = in ? at : Place{own.b, own.L, n};
                pair[j] = in ? tt : t0;
                head[j] = in ? gg : g;
                tt += per;
            }
#pragma unroll
            for (int j = 0; j < kDescPairs; ++j) {
                const int2 addr = pair_at(from[j].b, from[j].L, pair[j], head[j]);
                d[9 + 2 * j] = addr.x;
                d[10 + 2 * j] = addr.y;
            }
        }
    }
    if (block == 0) {   // Launched waves without a span, and the end of the last span (the descriptor behind the last wave's).
        for (long long w = cuts.nw * per + tid; w <= a.launch_waves; w += 256) {
            int32_t *d = a.wave_desc + w * kDescInts;
            d[4] = (int)cut.total;
            d[15] = cut.mode;   // (read before the span is seen to be empty)
        }
    }
}

// KV heads to a workgroup of the plan.  Every workgroup sums over the batch, so several KV heads share one where there are more units than the
// chip needs workgroups (8 KV heads, the plan kernel: 128 requests 7.7 us with one head each and 6.8 us, 256 requests 12.6 and 8.3).
inline int plan_heads(const AttnArgs &a)
{
    int heads = 1;
    while (a.num_kv_heads % (2 * heads) == 0 && (long long)a.batch * a.num_kv_heads / (2 * heads) >= kPlanGroups) heads *= 2;
    return heads;
}
// The batch needs attn_layout_kernel in front.
inline bool plan_laid_out(const AttnArgs &a) { return a.batch > (a.team_blocks ? kPlanLanesClasses : kPlanLanes); }

}  // namespace
}  // namespace ss
