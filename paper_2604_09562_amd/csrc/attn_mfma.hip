// Verify attention on the matrix cores (gfx950), head_dim 128, bf16 queries, bf16 or e4m3 cache.
//
// The work decomposition and the tile arithmetic are described in attn_mfma_kernels.h; here are the plan kernel,
// the workspace layout and the dispatch.
#include "common.h"
#include "span_cuts.h"

namespace ss {
namespace {

// ---------------------------------------------------------------------------------------------
// plan: workgroup (b, g) writes the flat list of tile pair addresses of its unit and the descriptors of the waves
// whose span starts inside it; (b, 0) / the last one publish the prefix and the partition count.
//
// Where the spans are cut.  A wave pays a fixed price for every unit it opens (query loads, a drained
// ring of pairs, the partial of the unit before: about the time of kUnitWeight pairs, of kUnitWeightDeep with four or five row
// blocks), so equal pair counts do not finish together: on a ragged batch the waves that cross ten short units were 10 % late.
// The cuts are therefore equal in a weighted coordinate in which every unit is `unit_weight` virtual
// pairs followed by its real ones; a cut that falls into a unit's virtual part becomes the unit's first
// pair.  The cuts depend on the batch's lengths only, so results do not vary from run to run.
// ---------------------------------------------------------------------------------------------
static_assert(kSpansPerWg == kWavesPerWg, "one span per wavefront");
constexpr int kPlanMaxBatch = 4096;   // requests whose pair prefix fits the plan kernel's LDS; beyond that the cuts are unweighted

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

__global__ __launch_bounds__(256) void attn_plan_kernel(AttnArgs a)
{
    __shared__ int32_t prefix[kPlanMaxBatch + 1];
    __shared__ int sh[4];
    const int b = blockIdx.x / a.num_kv_heads, g = blockIdx.x % a.num_kv_heads;
    const int tid = threadIdx.x;
    const bool weighted = a.batch <= kPlanMaxBatch && a.unit_weight > 0;

    // exclusive prefix of the pair counts of all requests (every workgroup builds its own copy), or,
    // for a batch too large for that, just the sums in front of and from request b on
    int pre = 0, longest = 0;   // (pairs of the longest unit)
    long long total = 0;
    __shared__ int longest_sh[4];
    auto note_longest = [&](int n) {
        n = wave_scan_int(n, [](int x, int y) { return max(x, y); });
        if ((tid & 63) == 63) longest_sh[tid >> 6] = n;
    };
    if (a.batch <= kPlanMaxBatch) {
        int carry = 0;
        for (int base = 0; base < a.batch; base += 256) {
            const int i = base + tid;
            const int t = i < a.batch ? window_pairs(a.kv_len[i], a.q_indptr[i + 1] - a.q_indptr[i], a.q_lo) : 0;
            longest = max(longest, t);
            const int incl = wave_scan_int(t, [](int x, int y) { return x + y; });
            if ((tid & 63) == 63) sh[tid >> 6] = incl;
            __syncthreads();
            int before = carry;
            for (int wv = 0; wv < (tid >> 6); ++wv) before += sh[wv];
            if (i < a.batch) prefix[i] = before + incl - t;
            const int chunk_total = sh[0] + sh[1] + sh[2] + sh[3];
            __syncthreads();
            carry += chunk_total;
        }
        if (tid == 0) prefix[a.batch] = carry;
        note_longest(longest);
        __syncthreads();
        pre = prefix[b];
        total = (long long)__builtin_amdgcn_readfirstlane(prefix[a.batch]) * a.num_kv_heads;   // (uniform: scalar arithmetic below)
    } else {
        int before = 0, rest = 0;
        for (int i = tid; i < a.batch; i += 256) {
            const int t = window_pairs(a.kv_len[i], a.q_indptr[i + 1] - a.q_indptr[i], a.q_lo);
            longest = max(longest, t);
            if (i < b) before += t; else rest += t;
        }
        for (int off = 32; off; off >>= 1) {
            before += __shfl_xor(before, off);
            rest += __shfl_xor(rest, off);
        }
        note_longest(longest);
        __shared__ int sh2[8];
        if ((tid & 63) == 0) {
            sh2[tid >> 6] = before;
            sh2[4 + (tid >> 6)] = rest;
        }
        __syncthreads();
        pre = sh2[0] + sh2[1] + sh2[2] + sh2[3];
        total = (long long)(pre + sh2[4] + sh2[5] + sh2[6] + sh2[7]) * a.num_kv_heads;
    }
    longest = __builtin_amdgcn_readfirstlane(max(max(longest_sh[0], longest_sh[1]), max(longest_sh[2], longest_sh[3])));
    const bool can_chain = (a.q_win * (a.num_q_heads / a.num_kv_heads) + 15) / 16 <= kChainRowBlocks;
    const SpanCount count = count_spans(total, longest, a.launch_waves, can_chain);
    const long long nw = count.spans;
    const int chain = count.chain;
    const int weight = weighted ? a.unit_weight : 0;
    const long long total_w = total + (long long)weight * a.batch * a.num_kv_heads;

    const int n = window_pairs(a.kv_len[b], a.q_indptr[b + 1] - a.q_indptr[b], a.q_lo);
    const long long off = (long long)pre * a.num_kv_heads + (long long)g * n;   // this unit's place in the flat list
    const int32_t *bt = a.block_table + (long long)b * a.max_blocks;
    const int blocks = (a.kv_len[b] + kTile - 1) / kTile;
    // (a pair whose second tile lies past the cache's end repeats the first; its slots are never visible)
    auto pair_at = [](const int32_t *table, int t, int nblk, int hkv, int gg) {
        const int b0 = table[2 * t], b1 = 2 * t + 1 < nblk ? table[2 * t + 1] : b0;
        return make_int2(b0 * hkv + gg, b1 * hkv + gg);
    };
    int2 *dst = a.pair_addr + off;
    for (int t = tid; t < n; t += 256) dst[t] = pair_at(bt, t, blocks, a.num_kv_heads, g);

    // waves whose cut falls into this unit's stretch [ya, ya + weight + n) of the weighted coordinate
    SpanCuts cuts;
    cuts.prefix = prefix;   // (only read when weight > 0, i.e. when the prefix was built)
    cuts.batch = a.batch;
    cuts.hkv = a.num_kv_heads;
    cuts.weight = weight;
    cuts.total = total;
    cuts.total_w = total_w;
    cuts.nw = nw;
    const long long ya = off + (long long)weight * ((long long)b * a.num_kv_heads + g);
    const long long w_lo = cuts.first_cut_at_or_after(ya);                // first w with w*total_w/nw >= ya
    const long long w_hi = cuts.first_cut_at_or_after(ya + weight + n);   // first w at or past the unit's end
    // Descriptor: {request, kv head, first pair, pairs of the unit, span begin, span end, kv_len,
    // first query row, end query row, addresses of the span's first kDescPairs tile pairs}: everything
    // the wave's first loads depend on, so that they go out after a single read.
    for (long long w = w_lo + tid; w < w_hi && w < nw; w += 256) {
        const int t0 = cuts.first_pair(cuts.cut(w), ya);
        const long long x0 = off + t0;
        const long long x1 = cuts.span_end(w);
        int32_t *d = a.wave_desc + w * kDescInts;
        d[0] = b; d[1] = g; d[2] = t0; d[3] = n;
        d[4] = (int)x0; d[5] = (int)x1;
        d[15] = chain;
        d[6] = a.kv_len[b]; d[7] = a.q_indptr[b]; d[8] = a.q_indptr[b + 1];
        // walk forward from (b, g, pair) over unit boundaries; past the last unit repeat the last pair
        int bb = b, gg = g, tt = t0, nn = n, nblk = blocks;
        int2 last = make_int2(0, 0);
        const int32_t *tb = bt;
        for (int j = 0; j < kDescPairs; ++j) {
            while (bb < a.batch && tt >= nn) {
                tt -= nn;
                if (++gg == a.num_kv_heads) {
                    gg = 0;
                    if (++bb < a.batch) {
                        nn = window_pairs(a.kv_len[bb], a.q_indptr[bb + 1] - a.q_indptr[bb], a.q_lo);
                        nblk = (a.kv_len[bb] + kTile - 1) / kTile;
                        tb = a.block_table + (long long)bb * a.max_blocks;
                    }
                }
            }
            if (bb < a.batch) last = pair_at(tb, tt, nblk, a.num_kv_heads, gg);
            d[9 + 2 * j] = last.x;
            d[10 + 2 * j] = last.y;
            ++tt;
        }
    }
    if (blockIdx.x == 0) {   // launched waves beyond the partition count get an empty span
        for (long long w = nw + tid; w < a.launch_waves; w += 256) {
            int32_t *d = a.wave_desc + w * kDescInts;
            d[4] = 0;
            d[5] = 0;
        }
    }
    if (g == 0 && tid == 0) {
        a.pair_prefix[b] = pre;
        if (b == a.batch - 1) {
            a.pair_prefix[a.batch] = pre + n;
            a.plan->total_pairs = (int)total;
            a.plan->num_waves = (int)nw;
            a.plan->unit_weight = weight;
            a.plan->chain = chain;
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
    n += align_up(sizeof(int32_t) * ((size_t)batch + 1), 256);
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
    if (p.unit_weight < 0) p.unit_weight = (p.q_win * G + 15) / 16 >= 4 ? kUnitWeightDeep : kUnitWeight;
    for (p.q_lo = 0; p.q_lo < a.max_q_len; p.q_lo += p.q_win) {
        if (!(a.reuse_plan && passes == 1)) {   // a stored plan describes one window only
            hipLaunchKernelGGL(attn_plan_kernel, dim3((unsigned)a.batch * a.num_kv_heads), dim3(256), 0, stream, p);
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
