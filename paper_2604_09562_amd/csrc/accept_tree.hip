// Sampled acceptance over draft trees (the chain rule and the greedy tree walk are in accept.hip).
#include "accept_common.h"

#include <algorithm>
#include <type_traits>

namespace ss {
namespace {

// ---- sampled acceptance over a draft tree ------------------------------------------------------------------
// The walk of a request is a chain of dependent steps, but only its rejections need the whole vocabulary:
// while the running distribution r is still a node's own target distribution a child is judged from two
// gathered logits and the row statistics of the first pass.  So the work is laid out in launches over all
// requests at once (the stream orders them, no kernel waits for another workgroup):
//   prep   one workgroup per request: merges the row statistics, evaluates q(x) and p(x) of every node, and
//          walks from the root until a child is rejected (-> a pass is due) or none is left (-> the draw)
//   round  begins by adopting the residual of the round before and walking on (each workgroup for itself: a few loads, cheaper
//          than a launch), then one pass over the vocabulary.  After a rejection: the sum of the rejected child's proposal, and
//          the sums of r and of the proposal over the entries whose residual r - q is positive; for a draw from a node's own
//          target distribution the sum of its exponentials, which are its block masses
//   pick   scan of the block masses, search inside one block
// A request needs a round per rejection, and one more if its last step accepted a child: at most k in all.
//
// One pass per rejection.  The sign of r - q depends on the proposal's normaliser Zq, which the same pass adds up.  As in the chain
// rule it is decided from the normaliser of the row statistics (good to 2e-5), and entries within 1e-4 of the boundary are set aside,
// each wavefront's in a run of its own; the next kernel adds them with the exact normaliser.  A block with more of them than its
// runs hold (rows that nearly coincide, or statistics that are no number) is evaluated entry by entry there.
//
// Where r comes from.  The residual of m rejections at a node is R_m = max(0, R_(m-1) / N_(m-1) - q_m), N_m its sum, R_0 the
// exponentials of the node's target row.  The pass of the first rejection reads two rows of logits, that of the second three (R_1 again from its
// logits).  From there on a pass reads R_(m-2) from memory, and R_(m-1) is written for the next one as long as a sibling is left: two fp64
// vocabulary vectors per request in turn.  At single tokens r is carried along in the nodes' records.
// All reductions have a fixed order.
//
// Bound by the fp64 exponentials of the rounds that have most requests pending and by the chain of a round: list, scalars and block sums,
// gathers, walk, rows, 6 us before the first exponential.  64 requests of 128256 entries, depth 4: 240 us with a walk kernel of dependent
// reads in every round, 2-byte loads, serial sums over the blocks and a pass that wrote r out for every draw; 129 us with two passes per
// rejection (the proposal's sum, then the residual, written out and read back); 96 us this way (rounds of 18, 20, 11 and 7 us).
struct TreeScalars {
    int32_t cur, n, next, phase;
    int32_t level, degenerate, which, rej;   // rejections at the current node that r has taken in; which: the buffer with R_(level-1), from
                                             // level 2 on; rej: the child just rejected
    int32_t rej_prev, more, copy, pad;       // the one taken in last; siblings after rej; the copy of the block sums that the last pass wrote
    float mp, mq, mq_prev, pad_f;      // exact maxima of the current node's target row and of the rejected children's draft rows
    double zp_stat, zq_stat;           // normalisers of the target row and of the rejected child's row as the row statistics have them
    double zp, zq_prev;                // exact ones, of the target row (from level 1 on) and of the child taken in last
    double norm, norm_prev;            // N_level, N_(level-1)
};
struct alignas(16) TreeNode {          // what the walk needs to know of a node, in one place: every further hop is a trip to memory
    double qx, px;                     // its token's probability under its own proposal / its parent's target row
    double zp, zq;                     // normalisers of its target row and its draft row from the row statistics
    float mp, mq;                      // exact maxima of the same
    int32_t par, x;                    // parent, token
    float u;
};
struct TreeState {
    TreeScalars s[2];                  // a round reads one copy while one of its workgroups writes the next
    double rx[2][SS_MAX_DEPTH + 1];    // R_level at the tokens of the current node's children, likewise
    TreeNode node_of[SS_MAX_DEPTH + 1];
    int32_t at;                        // the copy written last
    int32_t tok[SS_OUT_WIDTH];         // accepted tokens and nodes so far: written in place
    int32_t node[SS_MAX_DEPTH];
};
struct alignas(64) TreePending {       // how many requests a round has (those with a rejection in the round before)
    int32_t count;
};

// TS_WALK: not decided; TS_RESIDUAL: a child was rejected, its pass is this round's; TS_DRAW: from the current node's target row;
// TS_LAST: from the residual of the last pass (the scalars are those of the pass)
enum { TS_WALK = 0, TS_RESIDUAL = 1, TS_DRAW = 2, TS_LAST = 3 };

constexpr int kWaves = kThreads / 64;
constexpr int kRun = 64;               // boundary entries that a wavefront of a block can set aside

struct alignas(16) ZonePair {
    double r, q;                       // r (unnormalised at level 0) and the proposal's exponential
};
struct alignas(128) TreeBlock {        // what a pass leaves of a block
    double sum[4];                     // over all entries: R_0 (level 0), proposal; over the certainly positive: r, proposal
    uint64_t cnt;                      // entries that its wavefronts set aside, 16 bits each; more than kRun: evaluate the block entry by entry
    double mass;                       // of such a block, for the draw
    ZonePair head[kWaves];             // the first of each run (most runs are no longer), the others are in TreeMem::zone
};

struct TreeMem {
    TreeState *st;       // [batch]
    double *arr;         // [batch][2][vocab]
    TreeBlock *blocks;   // [batch][2][nsub]
    TreePending *pending;   // [SS_MAX_DEPTH], by round
    int32_t *list;       // [SS_MAX_DEPTH][batch] and which they are
    ZonePair *zone;      // [batch][2][nsub][kWaves][kRun], the first of a run unused
    __device__ __forceinline__ TreeBlock *block(int b, int copy, int nsub) const { return blocks + ((int64_t)b * 2 + copy) * nsub; }
    __device__ __forceinline__ ZonePair *runs(int b, int copy, int nsub) const
    {
        return zone + ((int64_t)b * 2 + copy) * nsub * (kWaves * kRun);
    }
};

// A lane's value in all lanes: c is the same in all of them.
__device__ __forceinline__ float lane_value(float x, int c)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), c));
}

// Offers children until one is rejected or none is left: one wavefront, lane c holding node c (1..k).  `r`: R_level at the lane's
// token (level > 0).  `write`: this workgroup records what happens.
__device__ __forceinline__ void tree_walk(const AcceptArgs &a, const TreeNode &nd, TreeState *st, TreeScalars &s, double r, int d0, bool write)
{
    const int lane = threadIdx.x & 63;
    const double u = (double)nd.u;
    double rx = nd.px;
    if (s.level > 0 && nd.par == s.cur && lane >= s.next) rx = r / s.norm;
    const unsigned long long pure_ok = __ballot(u * nd.qx < nd.px);
    unsigned long long offered = 0, ok = __ballot(u * nd.qx < rx);   // (level 0: the same)
    for (;;) {   // at most k steps: every step moves to a higher-numbered node
        const unsigned long long kids = __ballot(nd.par == s.cur && lane >= s.next);
        if (!kids) {
            s.phase = TS_DRAW;
            break;
        }
        const int c = __ffsll((long long)kids) - 1;
        offered |= 1ull << c;
        s.next = c + 1;
        if (!((ok >> c) & 1)) {
            s.phase = TS_RESIDUAL;
            s.rej = c;
            s.more = (kids & (kids - 1)) != 0;
            s.mq = lane_value(nd.mq, c);
            s.zq_stat = lane_value(nd.zq, c);
            break;
        }
        if (write && lane == c) {
            st->tok[s.n] = nd.x;
            st->node[s.n] = c;
        }
        // children of the node walked from were judged by its r; from here on r is the accepted node's own row
        if (write && lane == c && a.ratio_out) a.ratio_out[d0 + c - 1] = (float)(rx / nd.qx);
        offered &= ~(1ull << c);
        ++s.n;
        s.cur = c;
        s.level = 0;
        s.degenerate = 0;
        s.mp = lane_value(nd.mp, c);
        s.zp_stat = lane_value(nd.zp, c);
        ok = pure_ok;
        rx = nd.px;
    }
    if (write && a.ratio_out && ((offered >> lane) & 1)) a.ratio_out[d0 + lane - 1] = (float)(rx / nd.qx);
}

__global__ __launch_bounds__(kThreads) void tree_prep_kernel(AcceptArgs a, Workspace w, TreeMem mem)
{
    __shared__ float row_m[kMaxRows];
    __shared__ double row_z[kMaxRows];
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = a.q_indptr[b], k = min(a.q_indptr[b + 1] - t0 - 1, SS_MAX_DEPTH), d0 = t0 - b;
    const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
    const double inv_t = 1.0 / (double)T;
    // (gathers that depend on nothing the merge produces are requested first)
    int par = 0;
    float lq = 0.f, lp = 0.f;
    const bool is = wave == 0 && lane >= 1 && lane <= k;
    int parent = -2, token = 0;   // (-2: no node's child)
    float u = 0.f;
    if (is) {
        // (a node without a parent in front of it is never offered; the clamps keep its reads inside the batch)
        parent = a.tree_parent[t0 + lane];
        token = a.draft_tokens[d0 + lane - 1];
        u = a.u_accept[d0 + lane - 1];
        par = min(max(parent, 0), lane - 1);
        const int x = min(max(token, 0), a.vocab - 1);
        lq = load_logit(a.draft, d0 + lane - 1, a.row_stride, a.logit_dtype, x);
        lp = load_logit(a.target, t0 + par, a.row_stride, a.logit_dtype, x);
        if (a.ratio_out) a.ratio_out[d0 + lane - 1] = __builtin_nanf("");
    }
    merge_row_stats(w, t0, (int64_t)a.total_rows + d0, k, inv_t, row_m, row_z);
    __syncthreads();
    if (wave != 0) return;
    TreeState *st = &mem.st[b];
    const bool node = lane <= k;
    const float mp = node ? row_m[lane] : 0.f, mq = is ? row_m[k + lane] : 0.f;
    const double zp = node ? row_z[lane] : 1.0, zq = is ? row_z[k + lane] : 1.0;
    const double qx = is ? exp(((double)lq - (double)mq) * inv_t) / zq : 0.0;
    const double px = is ? exp(((double)lp - (double)row_m[par]) * inv_t) / row_z[par] : 0.0;
    const TreeNode nd = {qx, px, zp, zq, mp, mq, parent, token, u};
    if (node) st->node_of[lane] = nd;
    TreeScalars s = {};
    s.next = 1;
    s.phase = TS_WALK;
    s.mp = row_m[0];
    s.zp_stat = row_z[0];
    s.norm = 1.0;
    tree_walk(a, nd, st, s, 0.0, d0, true);
    if (lane == 0) {
        st->s[0] = s;
        st->at = 0;
    }
    if (b == 0 && lane < SS_MAX_DEPTH) mem.pending[lane].count = 0;
}

// A lane's eight logits of a 2048-entry block as four pairs, 512 entries apart: passes that move r move eight bytes per
// entry against two or four of logits, so their lanes stand next to each other in r (16 bytes each) rather than in the
// logits (eight consecutive entries per lane, 64 bytes apart in r: 25.1 us against 21.8 for 64 requests of 128256
// entries with one exponential of each row and r written).
template <int DT>
struct Raw2x4 {
    std::conditional_t<DT == SS_BF16, uint32_t, uint2> w[4];
    __device__ __forceinline__ void load(const void *row, int vocab, int i)
    {
        using W = std::remove_reference_t<decltype(w[0])>;
        using E = std::conditional_t<DT == SS_BF16, uint16_t, uint32_t>;
        const E *p = static_cast<const E *>(row);
        if ((i | (kSub - 1)) < vocab) {   // (the same for all lanes: the whole block lies inside the vocabulary)
#pragma unroll
            for (int t = 0; t < 4; ++t) w[t] = *reinterpret_cast<const W *>(p + i + t * 2 * kThreads);
            return;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {   // past the vocabulary: -inf
            const int v = i + t * 2 * kThreads;
            if constexpr (DT == SS_BF16)
                w[t] = (v < vocab ? p[v] : 0xff80u) | (v + 1 < vocab ? p[v + 1] : 0xff80u) << 16;
            else
                w[t] = make_uint2(v < vocab ? p[v] : 0xff800000u, v + 1 < vocab ? p[v + 1] : 0xff800000u);
        }
    }
    __device__ __forceinline__ bool equals(const Raw2x4 &o) const   // bit by bit
    {
        uint32_t d = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (DT == SS_BF16)
                d |= w[t] ^ o.w[t];
            else
                d |= (w[t].x ^ o.w[t].x) | (w[t].y ^ o.w[t].y);
        }
        return d == 0;
    }
    __device__ __forceinline__ void unpack(float (&x)[8]) const
    {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (DT == SS_BF16) {
                x[2 * t] = __uint_as_float(w[t] << 16);
                x[2 * t + 1] = __uint_as_float(w[t] & 0xffff0000u);
            } else {
                x[2 * t] = __uint_as_float(w[t].x);
                x[2 * t + 1] = __uint_as_float(w[t].y);
            }
        }
    }
};

// The residual of a pass with the exact normalisers, entry by entry: for the draw, and for blocks with too many boundary entries.
template <int DT>
struct TreeResidual {
    const void *prow, *qprow, *qrow;
    const double *src;   // R_(level) if the pass wrote it, R_(level-1) if it is to be formed from there, or null
    double inv_src, inv_prev, inv_norm, inv_q;
    RowArg ap, aqp, aq;
    bool form;           // a subtraction of the child taken in last lies between the source and r
    __device__ __forceinline__ TreeResidual(const AcceptArgs &a, const TreeMem &mem, const TreeScalars &s, int b, int t0, int d0, double inv_t,
                                            double zp, double zq)
        : ap(inv_t, s.mp), aqp(inv_t, s.mq_prev), aq(inv_t, s.mq)
    {
        prow = row_ptr(a.target, t0 + s.cur, a.row_stride, DT);
        qrow = row_ptr(a.draft, d0 + s.rej - 1, a.row_stride, DT);
        qprow = s.level ? row_ptr(a.draft, d0 + s.rej_prev - 1, a.row_stride, DT) : qrow;
        const bool stored = s.level >= 1 && s.more;
        src = stored || s.level >= 2 ? mem.arr + ((int64_t)b * 2 + (stored ? s.which ^ 1 : s.which)) * a.vocab : nullptr;
        form = s.level >= 1 && !stored;
        inv_src = stored ? 1.0 : 1.0 / (s.level >= 2 ? s.norm_prev : zp);
        inv_prev = s.level ? 1.0 / s.zq_prev : 0.0;
        inv_norm = s.level ? 1.0 / s.norm : 1.0;
        inv_q = 1.0 / zq;
    }
    // entries i .. i + 7
    __device__ __forceinline__ void operator()(const ExpTable &ex, int vocab, int i, double (&r)[8]) const
    {
        Raw8<DT> raw;
        float x[8];
        double q[8];
        if (src) {
#pragma unroll
            for (int t = 0; t < 8; ++t) r[t] = i + t < vocab ? src[i + t] : 0.0;
        } else {
            load8<DT>(prow, vocab, i, raw);
            unpack8<DT>(raw, x);
            exp8(ex, ap, x, r);
        }
        if (form) {
            load8<DT>(qprow, vocab, i, raw);
            unpack8<DT>(raw, x);
            exp8(ex, aqp, x, q);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            r[t] *= inv_src;
            if (form) r[t] = residual_of(r[t], q[t] * inv_prev);
            r[t] *= inv_norm;
        }
        load8<DT>(qrow, vocab, i, raw);
        unpack8<DT>(raw, x);
        exp8(ex, aq, x, q);
#pragma unroll
        for (int t = 0; t < 8; ++t) r[t] = residual_of(r[t], q[t] * inv_q);
    }
};

__device__ __forceinline__ int run_length(uint64_t cnt, int wave) { return (int)(cnt >> (16 * wave)) & 0xffff; }
__device__ __forceinline__ bool too_many(uint64_t cnt)
{
    static_assert(kRun < 0x7fff && kSub / kWaves < 0x7fff, "a count over the limit sets its top bit");
    return ((cnt + (0x7fffull - kRun) * 0x0001000100010001ull) & 0x8000800080008000ull) != 0;
}

// What is left of a block's sums, and of an entry that was set aside: scale_r is the exact 1 / Zp at level 0, else 1.
__device__ __forceinline__ double clipped(double r, double q, double scale_r, double inv_q) { return residual_of(r * scale_r, q * inv_q); }

// What a block's entries that were set aside add to its mass, in their stored order.
__device__ __forceinline__ double boundary_mass(const TreeBlock &v, const ZonePair *run, double scale_r, double inv_q)
{
    if (!v.cnt) return 0.0;
    double m = 0.0;
    bool more = false;
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) {
        const int n = run_length(v.cnt, wv);
        if (n > 0) m += clipped(v.head[wv].r, v.head[wv].q, scale_r, inv_q);
        more |= n > 1;
    }
    for (int e = 1; more; ++e) {
        more = false;
#pragma unroll
        for (int wv = 0; wv < kWaves; ++wv) {
            const int n = run_length(v.cnt, wv);
            if (e < n) m += clipped(run[wv * kRun + e].r, run[wv * kRun + e].q, scale_r, inv_q);
            more |= e + 1 < n;
        }
    }
    return m;
}

// The exact normalisers of the last pass of a request and the sum of its residual, the same bits in every workgroup that asks.  One
// wavefront adds them up, its lanes a block each (with all four at it, a run of boundary entries each, every workgroup of a round spent
// the fp64 instructions of the scans and divisions four times); all help with blocks that have too many boundary entries.
struct TreeTotals {
    double zp, zq, norm;
    int listed;   // no block has too many boundary entries
};
template <int DT>
__device__ __forceinline__ TreeTotals tree_totals(const AcceptArgs &a, const Workspace &w, const TreeMem &mem, const TreeScalars &s, int copy,
                                                  const ExpTable &ex, int b, int t0, int d0, double inv_t, TreeTotals &sh, double (&sum_sh)[kWaves])
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const TreeBlock *blk = mem.block(b, copy, w.nsub);
    if (wave == 0) {
        const ZonePair *run = mem.runs(b, copy, w.nsub);
        // (the lane's first block, usually its only one, is read once)
        const TreeBlock v = blk[min(lane, w.nsub - 1)];
        double zp = lane < w.nsub ? v.sum[0] : 0.0, zq = lane < w.nsub ? v.sum[1] : 0.0;
        for (int c = lane + 64; c < w.nsub; c += 64) {
            zp += blk[c].sum[0];
            zq += blk[c].sum[1];
        }
        TreeTotals t;
        t.zp = s.level ? s.zp : lane_value(wave_scan(zp), 63);
        t.zq = lane_value(wave_scan(zq), 63);
        const double scale_r = s.level ? 1.0 : 1.0 / t.zp, inv_q = 1.0 / t.zq;
        double sum = 0.0;
        bool listed = true;
        const auto add = [&](const TreeBlock &v, int c) __attribute__((always_inline)) {
            if (too_many(v.cnt)) {
                listed = false;
                return;
            }
            sum += clipped(v.sum[2], v.sum[3], scale_r, inv_q);
            sum += boundary_mass(v, run + (int64_t)c * kWaves * kRun, scale_r, inv_q);
        };
        if (lane < w.nsub) add(v, lane);
        for (int c = lane + 64; c < w.nsub; c += 64) add(blk[c], c);
        t.norm = lane_value(wave_scan(sum), 63);
        t.listed = !__any(!listed);
        if (lane == 0) sh = t;
    }
    __syncthreads();
    TreeTotals t = sh;
    if (!t.listed) {
        const TreeResidual<DT> residual(a, mem, s, b, t0, d0, inv_t, t.zp, t.zq);
        double sum = 0.0;
        for (int c = 0; c < w.nsub; ++c) {
            if (!too_many(blk[c].cnt)) continue;
            double r[8];
            residual(ex, a.vocab, c * kSub + threadIdx.x * 8, r);
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += r[i];
        }
        t.norm += block_sum<double>(sum, sum_sh);
    }
    return t;
}

// A round's requests are those with a rejection in the round before, and its workgroups share them evenly: as many to a request as
// there are workgroups for it, each with a run of its blocks.  With a fixed share of every request's blocks, workgroups of requests that
// were done took places of the others for the 3 us that each needs to find out.  FIRST: round 0, all requests, whose walk the prep kernel
// has done; without one in front a workgroup may be as small as a block, and the small ones even out requests with one row to read and
// with two.
constexpr int kMaxBpw = 8;   // blocks of a workgroup; the grid has enough of them for it
template <int DT, bool FIRST>
__global__ __launch_bounds__(kThreads, DT == SS_BF16 ? 4 : 3) void tree_round_kernel(AcceptArgs a, Workspace w, TreeMem mem, int round)
{
    __shared__ ExpTable ex;
    __shared__ TreeScalars s_sh;
    __shared__ double sum_sh[FIRST ? 1 : kMaxBpw][4][kWaves], norm_sh[kWaves];
    __shared__ TreeTotals tot_sh;
    __shared__ int cnt_sh[FIRST ? 1 : kMaxBpw][kWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b, part, bpw = 1;
    if constexpr (FIRST) {
        b = blockIdx.x / w.nsub;
        part = blockIdx.x % w.nsub;
    } else {
        const int32_t *list = mem.list + (int64_t)round * a.batch;
        const int listed = mem.pending[round].count, near_ones = list[min(lane, a.batch - 1)];
        if (listed == 0) return;
        const int share = max((int)gridDim.x / listed, 1);   // workgroups of a request, if its blocks are as many
        bpw = min((w.nsub + share - 1) / share, kMaxBpw);
        const int parts = (w.nsub + bpw - 1) / bpw, place = blockIdx.x / parts;
        if (place >= listed) return;
        part = blockIdx.x % parts;
        b = place < 64 ? __builtin_amdgcn_readlane(near_ones, place) : list[place];
    }
    TreeState *st = &mem.st[b];
    TreeScalars s = st->s[FIRST ? 0 : (round - 1) & 1];
    TreeNode nd = st->node_of[min(lane, SS_MAX_DEPTH)];   // (read with the scalars, for the lanes that hold a node)
    const int V = a.vocab, t0 = a.q_indptr[b], k = min(a.q_indptr[b + 1] - t0 - 1, SS_MAX_DEPTH), d0 = t0 - b;
    const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
    const double inv_t = 1.0 / (double)T;
    if constexpr (!FIRST) {
        if (lane == 0 || lane > k) nd.par = -2;
        const bool waits = wave == 0 && nd.par == s.cur && lane >= s.next;   // a child that has not been offered yet
        const int x_in = min(max(nd.x, 0), V - 1);   // inside the row, as the prep kernel's gathers
        float lp = 0.f, lq = 0.f;
        double r = 0.0;
        if (waits) {
            lq = load_logit(a.draft, d0 + s.rej - 1, a.row_stride, DT, x_in);
            if (s.level)
                r = st->rx[(round - 1) & 1][lane];
            else
                lp = load_logit(a.target, t0 + s.cur, a.row_stride, DT, x_in);
        }
        ex.init();
        const TreeTotals t = tree_totals<DT>(a, w, mem, s, (round - 1) & 1, ex, b, t0, d0, inv_t, tot_sh, norm_sh);
        if (wave == 0) {
            const TreeScalars before = s;
            if (t.norm > 0.0) {   // r takes the rejected child in
                // (by reciprocals, as in the passes: what vanishes there vanishes here)
                const double from = s.level ? r * (1.0 / s.norm) : ex(RowArg(inv_t, s.mp)(lp)) * (1.0 / t.zp);
                r = residual_of(from, ex(RowArg(inv_t, s.mq)(lq)) * (1.0 / t.zq));
                if (s.level && s.more) s.which ^= 1;
                ++s.level;
                s.degenerate = 0;
                s.zp = t.zp;
                s.zq_prev = t.zq;
                s.mq_prev = s.mq;
                s.rej_prev = s.rej;
                s.norm_prev = s.norm;
                s.norm = t.norm;
            } else {
                s.degenerate = 1;   // no mass is left: r stays as it is
            }
            s.phase = TS_WALK;
            tree_walk(a, nd, st, s, r, d0, part == 0);
            if (s.phase == TS_DRAW && s.level) {
                const int degenerate = s.degenerate;
                s = before;   // nothing was accepted since: the draw is from the pass's residual
                s.phase = TS_LAST;
                s.degenerate = degenerate;
            } else {
                s.copy = round & 1;
            }
            if (part == 0) {
                if (lane <= k) st->rx[round & 1][lane] = r;
                if (lane == 0) {
                    st->s[round & 1] = s;
                    st->at = round & 1;
                }
            }
            if (lane == 0) s_sh = s;
        }
        __syncthreads();
        s = s_sh;
    } else {
        ex.init();
    }
    const bool rejected = s.phase == TS_RESIDUAL;
    if (rejected && part == 0 && tid == 0 && round + 1 < SS_MAX_DEPTH)   // (the order of the list has no influence on any result)
        mem.list[(int64_t)(round + 1) * a.batch + atomicAdd(&mem.pending[round + 1].count, 1)] = b;
    if (!rejected && (s.phase != TS_DRAW || s.degenerate)) return;
    const RowArg ap(inv_t, s.mp), aq(inv_t, s.mq);
    const void *prow = row_ptr(a.target, t0 + s.cur, a.row_stride, DT);
    const void *qrow = rejected ? row_ptr(a.draft, d0 + s.rej - 1, a.row_stride, DT) : prow;
    const int sub0 = part * bpw, count = min(bpw, w.nsub - sub0);
    TreeBlock *const out = mem.block(b, round & 1, w.nsub) + sub0;
    ZonePair *const runs = mem.runs(b, round & 1, w.nsub) + (int64_t)sub0 * kWaves * kRun + wave * kRun;
    // A wavefront's sums of block j, and the entries that it sets aside if `close` says that a lane has one (near(t): the lane's entry t is
    // one; t ascending first in the run, lanes in order: their later additions have a fixed order).
    auto leave = [&](int j, double z0, double z1, double rr, double qq, unsigned long long close, const double (&r)[8], const double (&q)[8],
                     auto near) __attribute__((always_inline)) {
        const double sum = wave_sum4(z0, z1, rr, qq);
        if ((lane & 15) == 15) sum_sh[j][sum4_index(lane)][wave] = sum;
        int n = 0;
        if (close) {
            ZonePair *run = runs + (int64_t)j * kWaves * kRun, *head = &out[j].head[wave];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const bool mine = near(t) && r[t] > 0.0;
                const unsigned long long who = __ballot(mine);
                const int at = n + __popcll(who & ((1ull << lane) - 1));
                if (mine && at < kRun) *(at ? run + at : head) = ZonePair{r[t], q[t]};
                n += __popcll(who);
            }
        }
        if (lane == 0) cnt_sh[j][wave] = n;
    };
    if (FIRST || !rejected || s.level == 0) {
        // The target row, and the rejected child's row: where r - q is positive the difference of their logits says (accept_common.h).
        const double ln_ratio = (double)logf((float)(s.zp_stat / s.zq_stat));
        const float theta = (float)((double)T * ln_ratio + ((double)s.mp - (double)s.mq));
        const float width = (float)(kAmbEps * (double)T) + 4.0e-7f * fabsf(theta);
        const float above = theta + width, below = theta - width;
        const int i0 = sub0 * kSub + tid * 8;
        Raw8<DT> rp, rq;
        load8<DT>(prow, V, i0, rp);
        if (rejected) load8<DT>(qrow, V, i0, rq);
#pragma unroll 1
        for (int j = 0; j < count; ++j) {   // (the next block's logits are requested before this one's are used)
            float xp[8], xq[8];
            double e[8], q[8];
            unpack8<DT>(rp, xp);
            if (j + 1 < count) load8<DT>(prow, V, i0 + (j + 1) * kSub, rp);
            if (rejected) {
                unpack8<DT>(rq, xq);
                if (j + 1 < count) load8<DT>(qrow, V, i0 + (j + 1) * kSub, rq);
            }
            exp8(ex, ap, xp, e);
            double z0 = 0.0, z1 = 0.0, rr = 0.0, qq = 0.0;
            unsigned long long close = 0;
            if (rejected) {
                exp8(ex, aq, xq, q);
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float d = xp[t] - xq[t];
                    const bool up = d > above;
                    const double sure = up ? 1.0 : 0.0;
                    z0 += e[t];
                    z1 += q[t];
                    rr = fma(e[t], sure, rr);
                    qq = fma(q[t], sure, qq);
                    close |= __ballot(!(d < below)) ^ __ballot(up);   // (also if the statistics are no number)
                }
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t) z0 += e[t];
            }
            leave(j, z0, z1, rr, qq, close, e, q, [&](int t) __attribute__((always_inline)) {
                const float d = xp[t] - xq[t];
                return !(d < below) && !(d > above);
            });
        }
    } else {
        const bool logits = s.level == 1;   // R_0 is formed from its logits, otherwise R_(level-1) is in memory
        const RowArg aqp(inv_t, s.mq_prev);
        const void *qprow = row_ptr(a.draft, d0 + s.rej_prev - 1, a.row_stride, DT);
        const double *src = mem.arr + ((int64_t)b * 2 + s.which) * V;
        double *dst = mem.arr + ((int64_t)b * 2 + (s.which ^ 1)) * V;
        const double inv_src = 1.0 / (logits ? s.zp : s.norm_prev), inv_prev = 1.0 / s.zq_prev, inv_norm = 1.0 / s.norm, zq_stat = s.zq_stat;
        const int i0 = sub0 * kSub + tid * 2;
        Raw2x4<DT> rp, rqp, rq;
        if (logits) rp.load(prow, V, i0);
        rqp.load(qprow, V, i0);
        rq.load(qrow, V, i0);
#pragma unroll 1
        for (int j = 0; j < count; ++j) {
            const int i = i0 + j * kSub;
            const bool whole = (sub0 + j + 1) * kSub <= V;
            float x[8];
            double e[8], q[8];
            if (logits) {
                rp.unpack(x);
                if (j + 1 < count) rp.load(prow, V, i + kSub);
                exp8(ex, ap, x, e);
            } else {
                if (whole) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) __builtin_memcpy(&e[2 * t], src + i + t * 2 * kThreads, 16);   // (rows start 8-byte aligned)
                } else {
#pragma unroll
                    for (int t = 0; t < 8; ++t) e[t] = i + (t >> 1) * 2 * kThreads + (t & 1) < V ? src[i + (t >> 1) * 2 * kThreads + (t & 1)] : 0.0;
                }
            }
            rqp.unpack(x);
            const bool same = s.mq == s.mq_prev && !__any(!rq.equals(rqp));
            if (j + 1 < count) rqp.load(qprow, V, i + kSub);
            exp8(ex, aqp, x, q);
#pragma unroll
            for (int t = 0; t < 8; ++t) e[t] = residual_of(e[t] * inv_src, q[t] * inv_prev);
            if (s.more && whole) {
#pragma unroll
                for (int t = 0; t < 4; ++t) __builtin_memcpy(dst + i + t * 2 * kThreads, &e[2 * t], 16);
            } else if (s.more) {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (i + (t >> 1) * 2 * kThreads + (t & 1) < V) dst[i + (t >> 1) * 2 * kThreads + (t & 1)] = e[t];
            }
            if (!same) {   // (siblings drawn from one proposal carry equal rows, whose exponentials serve twice: 2 us of the second round)
                rq.unpack(x);
                exp8(ex, aq, x, q);
            }
            if (j + 1 < count) rq.load(qrow, V, i + kSub);
            double z1 = 0.0, rr = 0.0, qq = 0.0;
            unsigned long long close = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                e[t] *= inv_norm;
                const double d = fma(e[t], zq_stat, -q[t]), edge = kAmbEps * q[t];
                const bool up = d > edge;
                const double sure = up ? 1.0 : 0.0;
                z1 += q[t];
                rr = fma(e[t], sure, rr);
                qq = fma(q[t], sure, qq);
                close |= __ballot(!(d < -edge)) ^ __ballot(up);
            }
            leave(j, 0.0, z1, rr, qq, close, e, q, [&](int t) __attribute__((always_inline)) {
                const double d = fma(e[t], zq_stat, -q[t]), edge = kAmbEps * q[t];
                return !(d < -edge) && !(d > edge);
            });
        }
    }
    __syncthreads();
    if (tid < 4 * count) {
        const double *v = sum_sh[tid >> 2][tid & 3];
        out[tid >> 2].sum[tid & 3] = (v[0] + v[1]) + (v[2] + v[3]);
        const int *n = cnt_sh[tid >> 2];
        if ((tid & 3) == 0) out[tid >> 2].cnt = n[0] | n[1] << 16 | (uint64_t)(n[2] | n[3] << 16) << 32;
    }
}

// The draw.  Masses are unnormalised: the block sums and the exponentials of the current node's target row, or those of
// the last pass's residual.  grid: batch.
template <int DT>
__global__ __launch_bounds__(kThreads) void tree_pick_kernel(AcceptArgs a, Workspace w, TreeMem mem)
{
    __shared__ ExpTable ex;
    __shared__ DrawShared sh;
    __shared__ double norm_sh[kWaves];
    __shared__ TreeTotals tot_sh;
    const int b = blockIdx.x, tid = threadIdx.x;
    TreeState *st = &mem.st[b];
    const TreeScalars s0 = st->s[0], s1 = st->s[1], s = st->at ? s1 : s0;   // (both read at once)
    const int V = a.vocab, t0 = a.q_indptr[b], d0 = t0 - b;
    const bool residual = s.phase != TS_DRAW;   // (a child was rejected in the last round, and no other is left; or TS_LAST)
    const float u = a.u_sample[b];
    int y = -1;
    bool none = s.degenerate && s.phase != TS_RESIDUAL;
    if (!none) {
        ex.init();
        const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
        const double inv_t = 1.0 / (double)T;
        const TreeBlock *blk = mem.block(b, s.copy, w.nsub);
        if (residual) {
            const TreeTotals t = tree_totals<DT>(a, w, mem, s, s.copy, ex, b, t0, d0, inv_t, tot_sh, norm_sh);
            none = !(t.norm > 0.0);
            if (!none) {
                const TreeResidual<DT> entry(a, mem, s, b, t0, d0, inv_t, t.zp, t.zq);
                const ZonePair *runs = mem.runs(b, s.copy, w.nsub);
                const double scale_r = s.level ? 1.0 : 1.0 / t.zp, inv_q = 1.0 / t.zq;
                // blocks without a list first, by all lanes: their masses take the place of the sums
                for (int c = 0; !t.listed && c < w.nsub; ++c) {
                    if (!too_many(blk[c].cnt)) continue;
                    double r[8], m = 0.0;
                    entry(ex, V, c * kSub + tid * 8, r);
#pragma unroll
                    for (int i = 0; i < 8; ++i) m += r[i];
                    m = block_sum<double>(m, norm_sh);
                    if (tid == 0) mem.block(b, s.copy, w.nsub)[c].mass = m;
                }
                __syncthreads();
                auto mass_of = [&](int c) __attribute__((always_inline)) {
                    const TreeBlock &v = blk[c];
                    if (too_many(v.cnt)) return v.mass;
                    return clipped(v.sum[2], v.sum[3], scale_r, inv_q) + boundary_mass(v, runs + (int64_t)c * kWaves * kRun, scale_r, inv_q);
                };
                auto entries = [&](int cstar, double (&r)[kSubPer]) __attribute__((always_inline)) {
                    entry(ex, V, cstar * kSub + tid * kSubPer, r);
                };
                y = draw_token(w.nsub, u, sh, mass_of, entries);
            }
        } else {
            const RowArg ap(inv_t, s.mp);
            const void *prow = row_ptr(a.target, t0 + s.cur, a.row_stride, DT);
            auto mass_of = [&](int c) __attribute__((always_inline)) { return blk[c].sum[0]; };
            auto entries = [&](int cstar, double (&r)[kSubPer]) __attribute__((always_inline)) {
                Raw8<DT> raw;
                float x[8];
                load8<DT>(prow, V, cstar * kSub + tid * kSubPer, raw);
                unpack8<DT>(raw, x);
                exp8(ex, ap, x, r);
            };
            y = draw_token(w.nsub, u, sh, mass_of, entries);
        }
    }
    if (y < 0) {
        // the residual vanished, or there is no mass at all (an infinite logit): lowest-index maximum of the current node's
        // target row, as in the chain rule
        y = lowest_index_of(a.target, t0 + s.cur, a.row_stride, DT, V, s.mp, sh);
        if (!none && y >= V) y = 0;   // (a row of NaN)
    }
    if (tid < SS_OUT_WIDTH)
        a.out_tokens[(int64_t)b * SS_OUT_WIDTH + tid] = tid < s.n ? st->tok[tid] : (tid == s.n ? y : -1);
    if (tid < SS_MAX_DEPTH) a.accepted_nodes[(int64_t)b * SS_MAX_DEPTH + tid] = tid < s.n ? st->node[tid] : -1;
    if (tid == 0) a.accepted_len[b] = s.n;
}

}  // namespace

// The part of the workspace behind the chain rule's: states, residuals, block sums, boundary entries.
static size_t carve_tree(char *p, int batch, int vocab, TreeMem *mem)
{
    const size_t blocks = 2 * (size_t)batch * num_sub(vocab);
    size_t at = 0;
    const auto take = [&](size_t bytes) {
        char *q = p + at;
        at += align_up(bytes, 256);
        return q;
    };
    mem->st = reinterpret_cast<TreeState *>(take(sizeof(TreeState) * (size_t)batch));
    mem->arr = reinterpret_cast<double *>(take(sizeof(double) * 2 * (size_t)batch * vocab));
    mem->pending = reinterpret_cast<TreePending *>(take(sizeof(TreePending) * SS_MAX_DEPTH));
    mem->list = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * SS_MAX_DEPTH * (size_t)batch));
    mem->blocks = reinterpret_cast<TreeBlock *>(take(sizeof(TreeBlock) * blocks));
    mem->zone = reinterpret_cast<ZonePair *>(take(sizeof(ZonePair) * blocks * kWaves * kRun));
    return at;
}

size_t accept_tree_workspace_bytes(int batch, int total_rows, int vocab)
{
    TreeMem mem;
    return accept_workspace_bytes(batch, total_rows, vocab) + carve_tree(nullptr, batch, vocab, &mem);
}

template <int DT>
static int32_t tree_sample_rounds(const AcceptArgs &a, const Workspace &w, const TreeMem &mem, hipStream_t stream)
{
    // Four workgroups to a compute unit, all there at once, and more only if a round of all requests needs them.
    const long long least = (long long)a.batch * ((w.nsub + kMaxBpw - 1) / kMaxBpw), blocks = (long long)a.batch * w.nsub;
    const dim3 per_request((unsigned)a.batch), grid((unsigned)std::max(least, std::min(blocks, 1024ll)));
    hipLaunchKernelGGL(tree_prep_kernel, per_request, dim3(kThreads), 0, stream, a, w, mem);
    // A request has at most max_q_len - 1 children to offer.  Each takes a round if it is rejected, and a draw from a target row takes one
    // after the last accepted child, or without any.
    const int rounds = a.max_q_len > 1 ? a.max_q_len - 1 : 1;
    hipLaunchKernelGGL((tree_round_kernel<DT, true>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, a, w, mem, 0);
    for (int round = 1; round < rounds; ++round)
        hipLaunchKernelGGL((tree_round_kernel<DT, false>), grid, dim3(kThreads), 0, stream, a, w, mem, round);
    hipLaunchKernelGGL(tree_pick_kernel<DT>, per_request, dim3(kThreads), 0, stream, a, w, mem);
    SS_HIP_CHECK(hipGetLastError(), "launch of the sampled tree walk");
    return SS_OK;
}

int32_t accept_tree_sample_launch(const AcceptArgs &a, hipStream_t stream)
{
    const Workspace w = carve(a.workspace, a.batch, a.total_rows, a.vocab);
    TreeMem mem;
    carve_tree(static_cast<char *>(a.workspace) + accept_workspace_bytes(a.batch, a.total_rows, a.vocab), a.batch, a.vocab, &mem);
    if ((unsigned long long)a.batch * w.nsub > 0x7fffffffull) return fail(SS_ERR_UNSUPPORTED, "batch * vocab too large for one launch");
    const int32_t rc = accept_rowstats_launch(a, stream);
    if (rc != SS_OK) return rc;
    if (a.logit_dtype == SS_BF16) return tree_sample_rounds<SS_BF16>(a, w, mem, stream);
    return tree_sample_rounds<SS_F32>(a, w, mem, stream);
}

}  // namespace ss
