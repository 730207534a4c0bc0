// Verify attention on the matrix cores (gfx950), head_dim 128, bf16 queries, bf16 or e4m3 cache.
//
// The work decomposition and the tile arithmetic are described in attn_mfma_kernels.h; here are the plan kernel,
// the workspace layout and the dispatch.
#include "common.h"
#include "span_cuts.h"

namespace ss {
namespace {

// ---------------------------------------------------------------------------------------------
// plan: workgroup (p, g) writes the flat list of tile pair addresses of one unit (KV head g of the request at place p of the
// layout) and the descriptors of the waves whose span starts inside it; (p, 0) publishes the request's record, the last one
// the plan's.
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
// The sort costs the plan kernel 1.3 us of 6.5.
static_assert(kSpansPerWg == kWavesPerWg, "one span per wavefront");
constexpr int kPlanMaxBatch = 4096;   // requests whose prefixes fit the plan kernel's LDS; beyond that the cuts are unweighted
constexpr int kMaxPairCost = 16, kMaxOpenCost = 32 * kWavesPerWg * 8;   // of the tables below / of the option's largest weight

// Inclusive scan over a wavefront's lanes (values >= 0, 0 is neutral for `op`) by data-parallel moves: a scan by shuffles is six
// LDS round trips, 0.3 us of the plan's 5.
template <class Op>
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

// Costs for the cuts of a team kernel, in eighths of a pair of a unit with one row block: of a pair and of opening a unit, with
// 1 .. 5 row blocks, for bf16 and e4m3 caches.  Measured by sweeps over nine bf16 and seven e4m3 batches (uniform and mixed row blocks, short
// and long units); half or twice the opening costs are 1 to 4 % slower, pair costs between equal and 8 : 12 within 3 %.
constexpr int kPairCost[2][kMaxClasses] = {{8, 8, 8, 9, 9}, {8, 8, 9, 9, 10}};
constexpr int kOpenCost[2][kMaxClasses] = {{32, 48, 80, 100, 128}, {64, 96, 160, 220, 280}};
// Packed for SpanClasses, class 0 being five row blocks.
constexpr uint64_t pack_costs(const int (&v)[kMaxClasses], int bits)
{
    uint64_t x = 0;
    for (int k = 0; k < kMaxClasses; ++k) x |= (uint64_t)v[kMaxClasses - 1 - k] << (bits * k);
    return x;
}

// SORTED: for a team kernel, a batch whose prefixes fit: the requests are laid out by class (the most row blocks first).
template <bool SORTED>
__global__ __launch_bounds__(256) void attn_plan_kernel(AttnArgs a)
{
    // (for a batch whose prefix fits LDS: pairs and costs per KV head in front of each request of the layout, and the order)
    extern __shared__ int32_t plan_lds[];
    int32_t *prefix = plan_lds;
    uint32_t *cprefix = reinterpret_cast<uint32_t *>(plan_lds + a.batch + 1);   // (SORTED)
    uint16_t *order = reinterpret_cast<uint16_t *>(plan_lds + 2 * (a.batch + 1));
    __shared__ int sh[4], csh[4], longest_sh[4], counts[4][kMaxClasses];
    const int p = blockIdx.x / a.num_kv_heads, g = blockIdx.x % a.num_kv_heads;   // place in the layout, KV head
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = a.num_q_heads / a.num_kv_heads;
    const bool fits = a.plan_fits;

    SpanCuts cuts;
#pragma unroll
    for (int c = 0; c < kMaxClasses; ++c) cuts.classes.end[c] = a.batch;
    cuts.classes.cost = cuts.classes.weight = 0;
    if constexpr (SORTED) {
        const bool kv8 = a.kv_dtype == SS_FP8_E4M3;
        const int skip = kMaxClasses - a.team_blocks;   // classes with more row blocks than the kernel has
        cuts.classes.cost = (kv8 ? pack_costs(kPairCost[1], 8) : pack_costs(kPairCost[0], 8)) >> (8 * skip);
        cuts.classes.weight = a.auto_weight ? (kv8 ? pack_costs(kOpenCost[1], 12) : pack_costs(kOpenCost[0], 12)) >> (12 * skip)
                                            : 0x001001001001001ull * (uint64_t)(a.unit_weight * kWavesPerWg * 8);
    }
    // request i: pairs per KV head, and its class (the most row blocks first)
    auto request = [&](int i, int &n, int &cls) __attribute__((always_inline)) {
        const int q_len = a.q_indptr[i + 1] - a.q_indptr[i];
        n = window_pairs(a.kv_len[i], q_len, a.q_lo);
        const int blocks = (window_q_len(q_len, a.q_lo, a.q_win) * G + 15) >> 4;
        cls = SORTED ? a.team_blocks - max(blocks, 1) : 0;
    };

    int longest = 0;   // (pairs of the longest unit)
    auto note_longest = [&](int n) {
        n = wave_scan_int(n, [](int x, int y) { return max(x, y); });
        if (lane == 63) longest_sh[wave] = n;
    };
    int b = p, pre = 0;
    long long total = 0;
    if (fits && a.batch <= 64) {
        // A request to a lane: each wavefront does all of it by itself and waits once, for the prefixes in LDS, where the loops
        // below wait five times (three times without classes) and read the other wavefronts' counts in between.  A call is 0.6 us
        // shorter with classes (16 requests of 20..60 tokens 31.9 -> 31.3 us, 32 trees 69.4 -> 68.7) and 0.3 without (110.3 -> 110.0).
        const bool real = lane < a.batch;
        int t = 0, c = 0, req = lane;
        if (real) request(lane, t, c);
        if constexpr (SORTED) {
            int place = lane, end = 0;
#pragma unroll
            for (int k = 0; k < kMaxClasses; ++k) {
                const unsigned long long m = __ballot(real && c == k);
                if (real && c == k) place = end + __popcll(m & ((1ull << lane) - 1));
                end += __popcll(m);
                cuts.classes.end[k] = end;
            }
            t = __builtin_amdgcn_ds_permute(place << 2, t);   // (`place` is a permutation of the lanes)
            req = __builtin_amdgcn_ds_permute(place << 2, lane);
        }
        longest = t;
        auto add = [](int x, int y) { return x + y; };
        const int incl = wave_scan_int(t, add);
        if (wave == 0 && real) prefix[lane] = incl - t;
        if (wave == 0 && lane == 63) prefix[a.batch] = incl;
        if constexpr (SORTED) {
            const int cls = cuts.classes.of(lane);
            const int u = real ? t * cuts.classes.cost_of(cls) + cuts.classes.weight_of(cls) : 0;
            const int cincl = wave_scan_int(u, add);
            if (wave == 0 && real) {
                cprefix[lane] = (uint32_t)(cincl - u);
                order[lane] = (uint16_t)req;
            }
            if (wave == 0 && lane == 63) cprefix[a.batch] = (uint32_t)cincl;
        }
        note_longest(longest);
        __syncthreads();
        pre = prefix[p];
        if constexpr (SORTED) b = order[p];
        total = (long long)__builtin_amdgcn_readfirstlane(prefix[a.batch]) * a.num_kv_heads;
    } else if (fits) {
        // the first 256 requests stay in registers between the passes
        int n0 = 0, c0 = 0;
        if (tid < a.batch) request(tid, n0, c0);
        longest = n0;
        int carry = 0, ccarry = 0;
        if constexpr (SORTED) {
            // how many of each class there are, then each request's place: stable, class by class
            int mine[kMaxClasses] = {0, 0, 0, 0, 0};
            for (int base = 0; base < a.batch; base += 256) {
                const int i = base + tid;
                int n = n0, c = c0;
                if (base && i < a.batch) request(i, n, c);
#pragma unroll
                for (int k = 0; k < kMaxClasses; ++k) mine[k] += __popcll(__ballot(i < a.batch && c == k));
            }
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < kMaxClasses; ++k) counts[wave][k] = mine[k];
            }
            __syncthreads();
            int next[kMaxClasses], end = 0;   // the next free place of each class
#pragma unroll
            for (int k = 0; k < kMaxClasses; ++k) {
                next[k] = end;
                end += __builtin_amdgcn_readfirstlane(counts[0][k] + counts[1][k] + counts[2][k] + counts[3][k]);
                cuts.classes.end[k] = end;
            }
            for (int base = 0; base < a.batch; base += 256) {
                const int i = base + tid;
                int n = n0, c = c0;
                if (base && i < a.batch) request(i, n, c);
                if (a.batch > 256) {   // (else `counts` is of this chunk already)
                    __syncthreads();
#pragma unroll
                    for (int k = 0; k < kMaxClasses; ++k) {
                        const int m = __popcll(__ballot(i < a.batch && c == k));
                        if (lane == 0) counts[wave][k] = m;
                    }
                    __syncthreads();
                }
                int place = 0;
#pragma unroll
                for (int k = 0; k < kMaxClasses; ++k) {
                    const unsigned long long m = __ballot(i < a.batch && c == k);
                    int before = next[k];
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const int m_w = counts[w][k];
                        if (w < wave) before += m_w;
                        next[k] += m_w;
                    }
                    if (c == k) place = before + __popcll(m & ((1ull << lane) - 1));
                }
                if (i < a.batch) {
                    order[place] = (uint16_t)i;
                    prefix[place] = n;
                }
            }
            __syncthreads();
        }
        // exclusive prefixes of pairs and costs in layout order
        for (int base = 0; base < a.batch; base += 256) {
            const int i = base + tid;
            int t = n0, c = 0;
            if constexpr (SORTED) {
                t = i < a.batch ? prefix[i] : 0;
            } else if (base) {
                t = 0;
                if (i < a.batch) request(i, t, c);
            }
            longest = max(longest, t);
            auto add = [](int x, int y) { return x + y; };
            const int incl = wave_scan_int(t, add);
            int u = 0, cincl = 0;
            if constexpr (SORTED) {
                const int cls = cuts.classes.of(i);
                u = i < a.batch ? t * cuts.classes.cost_of(cls) + cuts.classes.weight_of(cls) : 0;
                cincl = wave_scan_int(u, add);
            }
            if (lane == 63) {
                sh[wave] = incl;
                csh[wave] = cincl;
            }
            __syncthreads();
            int before = carry, cbefore = ccarry;
            for (int wv = 0; wv < wave; ++wv) {
                before += sh[wv];
                if constexpr (SORTED) cbefore += csh[wv];
            }
            if (i < a.batch) {
                prefix[i] = before + incl - t;
                if constexpr (SORTED) cprefix[i] = (uint32_t)(cbefore + cincl - u);
            }
            const int chunk_total = sh[0] + sh[1] + sh[2] + sh[3], cchunk = csh[0] + csh[1] + csh[2] + csh[3];
            __syncthreads();
            carry += chunk_total;
            ccarry += cchunk;
        }
        if (tid == 0) {
            prefix[a.batch] = carry;
            if constexpr (SORTED) cprefix[a.batch] = (uint32_t)ccarry;
        }
        note_longest(longest);
        __syncthreads();
        pre = prefix[p];
        if constexpr (SORTED) b = order[p];
        total = (long long)__builtin_amdgcn_readfirstlane(prefix[a.batch]) * a.num_kv_heads;   // (uniform: scalar arithmetic below)
    } else {   // a batch too large for that: just the sums in front of and from request p on, in the batch's order
        int before = 0, rest = 0;
        for (int i = tid; i < a.batch; i += 256) {
            int t, c;
            request(i, t, c);
            longest = max(longest, t);
            if (i < p) before += t; else rest += t;
        }
        for (int off = 32; off; off >>= 1) {
            before += __shfl_xor(before, off);
            rest += __shfl_xor(rest, off);
        }
        note_longest(longest);
        if (lane == 0) {
            sh[wave] = before;
            csh[wave] = rest;
        }
        __syncthreads();
        pre = sh[0] + sh[1] + sh[2] + sh[3];
        total = (long long)(pre + csh[0] + csh[1] + csh[2] + csh[3]) * a.num_kv_heads;
    }
    longest = __builtin_amdgcn_readfirstlane(max(max(longest_sh[0], longest_sh[1]), max(longest_sh[2], longest_sh[3])));
    const SpanCount count = count_spans(total, longest, a.launch_waves, a.team_blocks == 0);
    const bool team = a.team_blocks > 0 || count.spans < a.launch_waves;   // (kernels of one or two row blocks: when the chip is not full)
    const int per = team ? kWavesPerWg : 1;   // wavefronts that share a span
    const long long nw = team ? count_team_spans(total, longest, a.launch_waves / kWavesPerWg) : count.spans;   // spans to cut

    const int L = a.kv_len[b], q0 = a.q_indptr[b], q1 = a.q_indptr[b + 1];
    const int n = window_pairs(L, q1 - q0, a.q_lo);
    const long long off = (long long)pre * a.num_kv_heads + (long long)g * n;   // this unit's place in the flat list
    const int32_t *bt = a.block_table + (long long)b * a.max_blocks;
    const int blocks = (L + kTile - 1) / kTile;
    // (a pair whose second tile lies past the cache's end repeats the first; its slots are never visible)
    auto pair_at = [](const int32_t *table, int t, int nblk, int hkv, int gg) {
        const int b0 = table[2 * t], b1 = 2 * t + 1 < nblk ? table[2 * t + 1] : b0;
        return make_int2(b0 * hkv + gg, b1 * hkv + gg);
    };
    int2 *dst = a.pair_addr + off;
    for (int t = tid; t < n; t += 256) dst[t] = pair_at(bt, t, blocks, a.num_kv_heads, g);

    // waves (or teams) whose cut falls into this unit's stretch [ya, ye) of the weighted coordinate
    cuts.prefix = prefix;   // (read only if they were built)
    cuts.cprefix = SORTED ? cprefix : nullptr;
    cuts.batch = a.batch;
    cuts.hkv = a.num_kv_heads;
    // Without classes a pair costs one.  What a team pays for opening a unit: 4 to 8 pairs are level with one or two row blocks.
    cuts.weight = !fits ? 0 : !team ? a.unit_weight : a.team_blocks ? a.unit_weight * kWavesPerWg : a.unit_weight * 2;
    cuts.total = total;
    cuts.total_w = SORTED ? (long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)cprefix[a.batch]) * a.num_kv_heads
                          : total + (long long)cuts.weight * a.batch * a.num_kv_heads;
    cuts.nw = nw;
    const int cls = SORTED ? cuts.classes.of(p) : 0, cost = SORTED ? cuts.classes.cost_of(cls) : 1;
    const int weight = SORTED ? cuts.classes.weight_of(cls) : cuts.weight;
    const uint32_t cpre = SORTED ? cprefix[p] : (uint32_t)pre + (uint32_t)weight * (uint32_t)p;
    const long long ya = (long long)cpre * a.num_kv_heads + (long long)g * (weight + (long long)n * cost), ye = ya + weight + (long long)n * cost;
    const long long w_lo = cuts.first_cut_at_or_after(ya);   // first w with w*total_w/nw >= ya
    const long long w_hi = cuts.first_cut_at_or_after(ye);   // first w at or past the unit's end
    // Descriptor: {place in the layout, kv head, first pair, class, span begin, span end, kv_len, first query row, end query
    // row, addresses of the first kDescPairs tile pairs the wave reads, team, request, pairs of the unit,
    // end of the span's first class}: everything
    // the wave's first loads depend on, so that they go out after a single read.
    for (long long i = w_lo * per + tid; i < w_hi * per && i < nw * per; i += 256) {
        const long long w = i / per;
        const int t0 = SpanCuts::first_pair(cuts.cut(w), ya, weight, cost);
        const long long x0 = off + t0;
        const long long x1 = cuts.span_end(w);
        int32_t *d = a.wave_desc + i * kDescInts;
        d[0] = p; d[1] = g; d[2] = t0; d[3] = cls;
        d[4] = (int)x0; d[5] = (int)x1;
        d[6] = L; d[7] = q0; d[8] = q1;
        d[15] = team; d[16] = b; d[17] = n;
        if constexpr (SORTED) d[18] = min((int)x1, prefix[cuts.classes.end_of(cls)] * a.num_kv_heads);
        else d[18] = (int)x1;
        // walk forward from (p, g, pair) over unit boundaries; past the last unit repeat the last pair
        int pp = p, gg = g, tt = t0 + (int)(i - w * per), nn = n, nblk = blocks;
        int2 last = pair_at(bt, t0, blocks, a.num_kv_heads, g);
        const int32_t *tb = bt;
        for (int j = 0; j < kDescPairs; ++j) {
            while (pp < a.batch && tt >= nn) {
                tt -= nn;
                if (++gg == a.num_kv_heads) {
                    gg = 0;
                    if (++pp < a.batch) {
                        const int bb = SORTED ? order[pp] : pp;
                        nn = window_pairs(a.kv_len[bb], a.q_indptr[bb + 1] - a.q_indptr[bb], a.q_lo);
                        nblk = (a.kv_len[bb] + kTile - 1) / kTile;
                        tb = a.block_table + (long long)bb * a.max_blocks;
                    }
                }
            }
            if (pp < a.batch) last = pair_at(tb, tt, nblk, a.num_kv_heads, gg);
            d[9 + 2 * j] = last.x;
            d[10 + 2 * j] = last.y;
            tt += per;
        }
    }
    if (blockIdx.x == 0) {   // launched waves beyond the partition count get an empty span
        for (long long w = nw * per + tid; w < a.launch_waves; w += 256) {
            int32_t *d = a.wave_desc + w * kDescInts;
            d[4] = 0;
            d[5] = 0;
            d[15] = team;   // (read before the span is seen to be empty)
        }
    }
    if (g == 0 && tid == 0) {
        AttnReq r;
        r.b = b; r.L = L; r.q0 = q0; r.q1 = q1; r.n = n; r.cls = cls; r.pre = pre;
        r.cpre = cpre;
        a.req[p] = r;
        if (p == a.batch - 1) {
            a.plan->total_pairs = (int)total;
            a.plan->num_waves = (int)count.spans;
            a.plan->unit_weight = fits ? a.unit_weight : 0;
            a.plan->chain = count.chain;
            a.plan->cuts = (int)nw;
            a.plan->team = team;
            a.plan->total_cost = cuts.total_w;
#pragma unroll
            for (int c = 0; c < kMaxClasses; ++c) {
                a.plan->class_req[c] = cuts.classes.end[c];
                a.plan->class_x[c] = SORTED ? prefix[cuts.classes.end[c]] * a.num_kv_heads : (int)total;
                a.plan->class_cost[c] = SORTED ? cuts.classes.cost_of(c) : 1;
                a.plan->class_weight[c] = SORTED ? cuts.classes.weight_of(c) : weight;
            }
        }
    }
}

}  // namespace

size_t attn_workspace_bytes(int batch, int max_blocks, int num_q_heads, int num_kv_heads, int head_dim, int launch_waves,
                            int max_q_len)
{
    const int G = num_q_heads / num_kv_heads;
    const size_t rows_pad = (size_t)attn_rows_pad(max_q_len, G);
    const size_t slots = (size_t)launch_waves + (size_t)batch * num_kv_heads;
    size_t n = 256;
    n += align_up(sizeof(AttnReq) * (size_t)batch, 256);
    n += align_up(sizeof(int32_t) * kDescInts * (size_t)launch_waves, 256);
    n += align_up(sizeof(int2) * (size_t)batch * (((size_t)max_blocks + 1) / 2) * num_kv_heads, 256);
    n += align_up(slots * rows_pad * 2 * sizeof(float), 256);
    n += align_up(slots * rows_pad * (size_t)head_dim * sizeof(float), 256);
    return n;
}

bool attn_mfma_supported(const AttnArgs &a)
{
    const int G = a.num_q_heads / a.num_kv_heads;
    return a.head_dim == kMfmaHeadDim && a.q_dtype == SS_BF16 && (a.kv_dtype == SS_BF16 || a.kv_dtype == SS_FP8_E4M3) &&
           (G == 1 || G == 2 || G == 4 || G == 8) && a.launch_waves % kWavesPerWg == 0;
}

int32_t attn_mfma_launch(const AttnArgs &a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1)
{
    const int G = a.num_q_heads / a.num_kv_heads;
    if (G != 1 && G != 2 && G != 4 && G != 8) return fail(SS_ERR_UNSUPPORTED, "head grouping not built for the MFMA kernel");
    // A wavefront holds at most 16 * kMaxRowBlocks query rows of a KV head.  A batch whose row bound
    // exceeds that is served in several passes over equal windows of query tokens, each a full
    // plan / stream / merge sequence on the same workspace (the stream orders them).
    const int win_max = 16 * kMaxRowBlocks / G;
    const int passes = (a.max_q_len + win_max - 1) / win_max;
    AttnArgs p = a;
    p.q_win = (a.max_q_len + passes - 1) / passes;
    const int nb = (p.q_win * G + 15) / 16;   // row blocks of a pass's window
    if (a.auto_weight) p.unit_weight = nb >= 4 ? kUnitWeightDeep : kUnitWeight;
    p.team_blocks = nb > kChainRowBlocks ? attn_team_blocks(G) : 0;
    // (the costs per KV head are summed in 32 bits)
    p.plan_fits = a.batch <= kPlanMaxBatch &&
                  (uint64_t)a.batch * (((uint64_t)a.max_blocks + 1) / 2 * kMaxPairCost + kMaxOpenCost) < (1ull << 32);
    const size_t prefix_bytes = sizeof(int32_t) * ((size_t)a.batch + 1);
    const size_t lds = !p.plan_fits ? 0 : p.team_blocks ? 2 * prefix_bytes + sizeof(uint16_t) * a.batch : prefix_bytes;
    for (p.q_lo = 0; p.q_lo < a.max_q_len; p.q_lo += p.q_win) {
        if (!(a.reuse_plan && passes == 1)) {   // a stored plan describes one window only
            const dim3 grid((unsigned)a.batch * a.num_kv_heads);
            if (p.team_blocks && p.plan_fits)
                hipLaunchKernelGGL(attn_plan_kernel<true>, grid, dim3(256), lds, stream, p);
            else
                hipLaunchKernelGGL(attn_plan_kernel<false>, grid, dim3(256), lds, stream, p);
            SS_HIP_CHECK(hipGetLastError(), "launch attn_plan_kernel");
        }
        // the streaming and merge kernels of each grouping live in their own translation unit; a
        // profile's event pair goes to the first pass
        hipEvent_t e0 = p.q_lo ? nullptr : ev0, e1 = p.q_lo ? nullptr : ev1;
        int32_t rc;
        switch (G) {
        case 1: rc = attn_mfma_launch_g1(p, stream, e0, e1); break;
        case 2: rc = attn_mfma_launch_g2(p, stream, e0, e1); break;
        case 4: rc = attn_mfma_launch_g4(p, stream, e0, e1); break;
        default: rc = attn_mfma_launch_g8(p, stream, e0, e1); break;
        }
        if (rc != SS_OK) return rc;
    }
    return SS_OK;
}

}  // namespace ss
