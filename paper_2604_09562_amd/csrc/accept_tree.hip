// Sampled acceptance over draft trees (the chain rule and the greedy tree walk are in accept.hip).
#include "accept_common.h"

#include <type_traits>

namespace ss {
namespace {

// ---- sampled acceptance over a draft tree ------------------------------------------------------------------
// The walk of a request is a chain of dependent steps, but only its rejections need the whole vocabulary:
// while the running distribution r is still a node's own target distribution a child is judged from two
// gathered logits and the row statistics of the first pass.  So the work is laid out in launches over all
// requests at once (the stream orders them, no kernel waits for another workgroup):
//   prep   one workgroup per request: merges the row statistics, evaluates q(x) and p(x) of every node, and
//          walks from the root until a child is rejected (-> a residual is due) or none is left (-> the draw)
//   sums   per 2048-entry block, exact fp64 sums of the rejected child's proposal's exponentials, and of the
//          target row's if r has not been written out yet; for a draw from a node's own target distribution
//          the target row's, which are its block masses
//   resid  the residual max(0, r - q) with the exact normalisers, written to the request's other buffer, and its
//          sum per block (its normaliser once added up, and the block masses of a draw from it)
//   pick   scan of the block masses, search inside one block
// A request needs a (sums, resid) round per rejection, at most k; the sums kernel of every later round begins by
// walking on (each of its workgroups for itself: a few loads of a record per node, cheaper than a launch), and a
// last sums kernel ends every walk.  r lives unnormalised in device memory, two fp64 vocabulary vectors per
// request.  All reductions have a fixed order.
//
// Bound by the fp64 exponentials of the rounds that have most requests pending and by the length of the launch
// chain.  64 requests of 128256 entries, depth 4: 240 us with a walk kernel of dependent reads in every round, 2-byte
// loads, serial sums over the blocks and a pass that wrote r out for every draw; 125 to 132 us this way.
struct TreeScalars {
    int32_t cur, n, next, phase;       // phase: 0 walking, 1 residual due, 2 draw due
    int32_t pure, degenerate, which, rej;   // which: the buffer that holds r; rej: the child just rejected
    float mp, mq;                      // exact maxima of the current node's target row / the rejected child's draft row
    double pad;
    double norm;                       // exact normaliser of the buffer that holds r
};
struct TreeState {
    TreeScalars s;                     // copied to registers by the kernels
    int32_t tok[SS_OUT_WIDTH];         // accepted tokens and nodes so far: written in place
    int32_t node[SS_MAX_DEPTH];
};
struct TreeNode {                      // what the walk needs to know of a node
    double qx, px;                     // its token's probability under its own proposal / its parent's target row
    float mp, mq;                      // exact maxima of its target row / its draft row
};

enum { TS_WALK = 0, TS_RESIDUAL = 1, TS_DRAW = 2 };

// The walk reads one copy of a request's scalars while one of its workgroups writes the next: two copies in turn, in
// arrays of the chain rule's workspace that the tree walk has no other use for (as are the node records).
struct TreeMem {
    TreeState *st;
    double *arr;   // [batch][2][vocab]
    __device__ __forceinline__ TreeScalars *scalars(const Workspace &w, int b, int copy) const
    {
        return copy ? reinterpret_cast<TreeScalars *>(w.amb_eq + (int64_t)b * kAmbCap) : &st[b].s;
    }
    __device__ __forceinline__ TreeNode *nodes(const Workspace &w, int b) const
    {
        return reinterpret_cast<TreeNode *>(w.amb_ep + (int64_t)b * kAmbCap);
    }
};
static_assert(sizeof(TreeNode) * (SS_MAX_DEPTH + 1) <= sizeof(double) * kAmbCap, "node records fit the list");

// Offers children until one is rejected or none is left: one wavefront, lane c holding node c (1..k).  `write`: this
// workgroup records what happens.
__device__ __forceinline__ void tree_walk(const AcceptArgs &a, const TreeNode *nodes, TreeState *st, const double *arr_b, TreeScalars &s,
                                          int t0, int d0, int k, bool write)
{
    const int lane = threadIdx.x & 63;
    const bool is = lane >= 1 && lane <= k;
    const int par = is ? a.tree_parent[t0 + lane] : -2;
    const int x = is ? a.draft_tokens[d0 + lane - 1] : 0;
    const int x_in = min(max(x, 0), a.vocab - 1);   // where r is read: inside the request's buffer, as the prep kernel's gathers
    const double u = is ? (double)a.u_accept[d0 + lane - 1] : 0.0;
    const double qx = is ? nodes[lane].qx : 0.0, px = is ? nodes[lane].px : 0.0;
    const float mp = lane <= k ? nodes[lane].mp : 0.f, mq = is ? nodes[lane].mq : 0.f;
    double rx = px;
    if (!s.pure && par == s.cur && lane >= s.next) rx = arr_b[(int64_t)s.which * a.vocab + x_in] / s.norm;
    const unsigned long long pure_ok = __ballot(is && u * qx < px);
    const unsigned long long here_ok = __ballot(is && u * qx < rx);   // (s.pure: the same)
    unsigned long long offered = 0, ok = here_ok;
    for (;;) {   // at most k steps: every step moves to a higher-numbered node
        const unsigned long long kids = __ballot(par == s.cur && lane >= s.next);
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
            s.mq = __shfl(mq, c);
            break;
        }
        if (write && lane == c) {
            st->tok[s.n] = x;
            st->node[s.n] = c;
        }
        // children of the node walked from were judged by its r; from here on r is the accepted node's own row
        if (write && lane == c && a.ratio_out) a.ratio_out[d0 + c - 1] = (float)(rx / qx);
        offered &= ~(1ull << c);
        ++s.n;
        s.cur = c;
        s.pure = 1;
        s.degenerate = 0;
        s.mp = __shfl(mp, c);
        ok = pure_ok;
        rx = px;
    }
    if (write && a.ratio_out && ((offered >> lane) & 1)) a.ratio_out[d0 + lane - 1] = (float)(rx / qx);
}

__global__ __launch_bounds__(kThreads) void tree_prep_kernel(AcceptArgs a, Workspace w, TreeMem mem)
{
    __shared__ float row_m[kMaxRows];
    __shared__ double row_z[kMaxRows];
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = a.q_indptr[b], k = a.q_indptr[b + 1] - t0 - 1, d0 = t0 - b;
    const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
    const double inv_t = 1.0 / (double)T;
    // (gathers that depend on nothing the merge produces are requested first)
    int par = 0;
    float lq = 0.f, lp = 0.f;
    const bool is = wave == 0 && lane >= 1 && lane <= k;
    if (is) {
        // (a node without a parent in front of it is never offered; the clamps keep its reads inside the batch)
        par = min(max(a.tree_parent[t0 + lane], 0), lane - 1);
        const int x = min(max(a.draft_tokens[d0 + lane - 1], 0), a.vocab - 1);
        lq = load_logit(a.draft, d0 + lane - 1, a.row_stride, a.logit_dtype, x);
        lp = load_logit(a.target, t0 + par, a.row_stride, a.logit_dtype, x);
        if (a.ratio_out) a.ratio_out[d0 + lane - 1] = __builtin_nanf("");
    }
    merge_row_stats(w, t0, (int64_t)a.total_rows + d0, k, inv_t, row_m, row_z);
    __syncthreads();
    if (wave != 0) return;
    TreeNode *nodes = mem.nodes(w, b);
    if (lane <= k) {
        TreeNode nd;
        nd.mp = row_m[lane];
        nd.mq = is ? row_m[k + lane] : 0.f;
        nd.qx = is ? exp(((double)lq - (double)nd.mq) * inv_t) / row_z[k + lane] : 0.0;
        nd.px = is ? exp(((double)lp - (double)row_m[par]) * inv_t) / row_z[par] : 0.0;
        nodes[lane] = nd;
    }
    TreeScalars s;
    s.cur = 0; s.n = 0; s.next = 1; s.phase = TS_WALK; s.pure = 1; s.degenerate = 0; s.which = 0; s.rej = 0;
    s.mp = row_m[0]; s.mq = 0.f; s.pad = 0.0; s.norm = 1.0;
    tree_walk(a, nodes, &mem.st[b], mem.arr, s, t0, d0, k, true);
    if (lane == 0) *mem.scalars(w, b, 0) = s;
}

// Total of a request's block sums, the same bits in every lane of every wavefront that asks.
__device__ __forceinline__ double blocks_total(const double *v, int nsub)
{
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    for (int c = lane; c < nsub; c += 64) s += v[c];
    return lane_value(wave_scan(s), 63);
}

// A workgroup handles `bpw` blocks of one request; round 0 finds the walk done by the prep kernel, a later round adopts
// the residual that the round before wrote and walks on first.  grid: batch * ceil(nsub / bpw).
constexpr int kMaxBpw = 8;
template <int DT>
__global__ __launch_bounds__(kThreads) void tree_sums_kernel(AcceptArgs a, Workspace w, TreeMem mem, int round, int bpw)
{
    __shared__ ExpTable ex;
    __shared__ TreeScalars s_sh;
    __shared__ double sum_sh[kMaxBpw][2][4];
    const int parts = (w.nsub + bpw - 1) / bpw;
    const int part = blockIdx.x % parts, b = blockIdx.x / parts, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t ob = (int64_t)b * w.nsub;
    TreeScalars s = *mem.scalars(w, b, round ? (round - 1) & 1 : 0);
    const int t0 = a.q_indptr[b], k = a.q_indptr[b + 1] - t0 - 1, d0 = t0 - b;
    if (round) {
        if (s.phase == TS_DRAW) {   // (its block masses are there already)
            if (part == 0 && tid == 0) *mem.scalars(w, b, round & 1) = s;
            return;
        }
        if (wave == 0) {
            // the residual of the last rejection is in the other buffer: adopt it
            const double S = blocks_total(w.sc + ob, w.nsub);
            s.degenerate = !(S > 0.0);
            if (!s.degenerate) {
                s.which ^= 1;
                s.norm = S;
                s.pure = 0;
            }
            s.phase = TS_WALK;
            tree_walk(a, mem.nodes(w, b), &mem.st[b], mem.arr + (int64_t)b * 2 * a.vocab, s, t0, d0, k, part == 0);
            if (lane == 0) {
                s_sh = s;
                if (part == 0) *mem.scalars(w, b, round & 1) = s;
            }
        }
        __syncthreads();
        s = s_sh;
    }
    const bool want_q = s.phase == TS_RESIDUAL;
    const bool want_p = s.pure && (want_q || !s.degenerate);
    if (!want_q && !want_p) return;
    ex.init();
    const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
    const double inv_t = 1.0 / (double)T;
    const RowArg ap(inv_t, s.mp), aq(inv_t, s.mq);
    const void *prow = row_ptr(a.target, t0 + s.cur, a.row_stride, DT);
    const void *qrow = want_q ? row_ptr(a.draft, d0 + s.rej - 1, a.row_stride, DT) : prow;
    const int sub0 = part * bpw, count = min(bpw, w.nsub - sub0);
    const int i0 = sub0 * kSub + tid * 8;
    Raw8<DT> rp, rq;
    if (want_p) load8<DT>(prow, a.vocab, i0, rp);
    if (want_q) load8<DT>(qrow, a.vocab, i0, rq);
#pragma unroll 1
    for (int j = 0; j < count; ++j) {   // (the next block's logits are requested before this one's are used)
        float x[8];
        double e[8];
        if (want_p) {
            unpack8<DT>(rp, x);
            if (j + 1 < count) load8<DT>(prow, a.vocab, i0 + (j + 1) * kSub, rp);
            exp8(ex, ap, x, e);
            double z = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) z += e[i];
            z = wave_scan(z);
            if (lane == 63) sum_sh[j][0][wave] = z;
        }
        if (want_q) {
            unpack8<DT>(rq, x);
            if (j + 1 < count) load8<DT>(qrow, a.vocab, i0 + (j + 1) * kSub, rq);
            exp8(ex, aq, x, e);
            double z = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) z += e[i];
            z = wave_scan(z);
            if (lane == 63) sum_sh[j][1][wave] = z;
        }
    }
    __syncthreads();
    if (tid < 2 * count) {
        const int j = tid >> 1, which = tid & 1;
        if (which ? want_q : want_p) {
            const double *v = sum_sh[j][which];
            (which ? w.zq : w.zp)[ob + sub0 + j] = (v[0] + v[1]) + (v[2] + v[3]);
        }
    }
}

// A lane's eight logits of a 2048-entry block as four pairs, 512 entries apart: the residual pass moves eight bytes per
// entry against two or four of logits, so its lanes stand next to each other in r (16 bytes each) rather than in the
// logits (eight consecutive entries per lane, 64 bytes apart in r: 25.1 us for the first round of 64 requests of 128256
// entries, this way 21.8 us).
template <int DT>
struct Raw2x4 {
    typename std::conditional<DT == SS_BF16, uint32_t, uint2>::type w[4];
    __device__ __forceinline__ void load(const void *row, int vocab, int i)
    {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int v = i + t * 2 * kThreads;
            if constexpr (DT == SS_BF16) {
                const uint16_t *p = static_cast<const uint16_t *>(row);
                if (v + 2 <= vocab)
                    w[t] = *reinterpret_cast<const uint32_t *>(p + v);
                else
                    w[t] = (v < vocab ? p[v] : 0xff80u) | 0xff800000u;   // past the vocabulary: -inf
            } else {
                const uint32_t *p = static_cast<const uint32_t *>(row);
                if (v + 2 <= vocab)
                    w[t] = *reinterpret_cast<const uint2 *>(p + v);
                else
                    w[t] = make_uint2(v < vocab ? p[v] : 0xff800000u, 0xff800000u);
            }
        }
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

// Residual due: other buffer <- max(0, r - q), its block sums.  grid: batch * ceil(nsub / bpw).
template <int DT>
__global__ __launch_bounds__(kThreads) void tree_resid_kernel(AcceptArgs a, Workspace w, TreeMem mem, int round, int bpw)
{
    __shared__ ExpTable ex;
    __shared__ double sum_sh[kMaxBpw][4];
    const int parts = (w.nsub + bpw - 1) / bpw;
    const int part = blockIdx.x % parts, b = blockIdx.x / parts, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t ob = (int64_t)b * w.nsub;
    const TreeScalars s = *mem.scalars(w, b, round & 1);
    if (s.phase != TS_RESIDUAL) return;
    const int V = a.vocab;
    const int t0 = a.q_indptr[b], d0 = t0 - b;
    const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
    const double inv_t = 1.0 / (double)T;
    const RowArg ap(inv_t, s.mp), aq(inv_t, s.mq);
    const void *prow = row_ptr(a.target, t0 + s.cur, a.row_stride, DT);
    const void *qrow = row_ptr(a.draft, d0 + s.rej - 1, a.row_stride, DT);
    const double *cur_arr = mem.arr + ((int64_t)b * 2 + s.which) * V;
    double *alt = mem.arr + ((int64_t)b * 2 + (s.which ^ 1)) * V;
    const int sub0 = part * bpw, count = min(bpw, w.nsub - sub0);
    const int i0 = sub0 * kSub + tid * 2;
    Raw2x4<DT> rp, rq;
    rq.load(qrow, V, i0);
    if (s.pure) rp.load(prow, V, i0);
    ex.init();
    const double zq = blocks_total(w.zq + ob, w.nsub);
    const double norm = s.pure ? blocks_total(w.zp + ob, w.nsub) : s.norm;
    const double inv_norm = 1.0 / norm, inv_zq = 1.0 / zq;
#pragma unroll 1
    for (int j = 0; j < count; ++j) {
        const int i = i0 + j * kSub;
        float x[8];
        double e[8], q[8];
        rq.unpack(x);
        if (j + 1 < count) rq.load(qrow, V, i + kSub);
        if (!s.pure) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {   // (rows of the buffers start 8-byte aligned)
                const int v = i + t * 2 * kThreads;
                if (v + 2 <= V) {
                    __builtin_memcpy(&e[2 * t], cur_arr + v, 16);
                } else {
                    e[2 * t] = v < V ? cur_arr[v] : 0.0;
                    e[2 * t + 1] = 0.0;
                }
            }
        }
        exp8(ex, aq, x, q);
        if (s.pure) {
            rp.unpack(x);
            if (j + 1 < count) rp.load(prow, V, i + kSub);
            exp8(ex, ap, x, e);
        }
        double sum = 0.0;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const double rt = e[t] * inv_norm, qt = q[t] * inv_zq;
            e[t] = rt > qt ? rt - qt : 0.0;
            sum += e[t];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int v = i + t * 2 * kThreads;
            if (v + 2 <= V)
                __builtin_memcpy(alt + v, &e[2 * t], 16);
            else if (v < V)
                alt[v] = e[2 * t];
        }
        sum = wave_scan(sum);
        if (lane == 63) sum_sh[j][wave] = sum;
    }
    __syncthreads();
    if (tid < count) w.sc[ob + sub0 + tid] = (sum_sh[tid][0] + sum_sh[tid][1]) + (sum_sh[tid][2] + sum_sh[tid][3]);
}

// The draw.  Masses are unnormalised: the block sums and the exponentials of the current node's target row, or those of
// the last residual.  grid: batch.
template <int DT>
__global__ __launch_bounds__(kThreads) void tree_pick_kernel(AcceptArgs a, Workspace w, TreeMem mem, int copy)
{
    __shared__ ExpTable ex;
    __shared__ DrawShared sh;
    const int b = blockIdx.x, tid = threadIdx.x;
    const TreeScalars s = *mem.scalars(w, b, copy);
    const int V = a.vocab, t0 = a.q_indptr[b];
    const int64_t ob = (int64_t)b * w.nsub;
    int y;
    if (s.degenerate) {   // the residual vanished: lowest-index maximum of the current node's target row
        y = lowest_index_of(a.target, t0 + s.cur, a.row_stride, DT, V, s.mp, sh);
    } else {
        ex.init();
        const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
        const RowArg ap(1.0 / (double)T, s.mp);
        const void *prow = row_ptr(a.target, t0 + s.cur, a.row_stride, DT);
        const double *r_arr = mem.arr + ((int64_t)b * 2 + s.which) * V;
        const double *blocks = (s.pure ? w.zp : w.sc) + ob;
        auto mass_of = [&](int c) __attribute__((always_inline)) { return blocks[c]; };
        auto entries = [&](int cstar, double (&r)[kSubPer]) __attribute__((always_inline)) {
            const int i = cstar * kSub + tid * kSubPer;
            if (s.pure) {
                Raw8<DT> raw;
                float x[8];
                load8<DT>(prow, V, i, raw);
                unpack8<DT>(raw, x);
                exp8(ex, ap, x, r);
            } else {
#pragma unroll
                for (int t = 0; t < kSubPer; ++t) r[t] = i + t < V ? r_arr[i + t] : 0.0;
            }
        };
        y = draw_token(w.nsub, a.u_sample[b], sh, mass_of, entries);
        if (y < 0) {   // no mass at all, as with an infinite logit: the arg-maximum, as in the chain rule
            y = lowest_index_of(a.target, t0 + s.cur, a.row_stride, DT, V, s.mp, sh);
            if (y >= V) y = 0;   // (a row of NaN)
        }
    }
    if (tid < SS_OUT_WIDTH)
        a.out_tokens[(int64_t)b * SS_OUT_WIDTH + tid] = tid < s.n ? mem.st[b].tok[tid] : (tid == s.n ? y : -1);
    if (tid < SS_MAX_DEPTH) a.accepted_nodes[(int64_t)b * SS_MAX_DEPTH + tid] = tid < s.n ? mem.st[b].node[tid] : -1;
    if (tid == 0) a.accepted_len[b] = s.n;
}

}  // namespace

size_t accept_tree_workspace_bytes(int batch, int total_rows, int vocab)
{
    return accept_workspace_bytes(batch, total_rows, vocab) + align_up(sizeof(TreeState) * (size_t)batch, 256) +
           align_up(sizeof(double) * 2 * (size_t)batch * vocab, 256);
}

template <int DT>
static int32_t tree_sample_rounds(const AcceptArgs &a, const Workspace &w, const TreeMem &mem, hipStream_t stream)
{
    // Blocks per workgroup: one as long as that leaves no more than four wavefronts for each of the chip's 1024 SIMDs,
    // then as many as keep it there, so that a large batch pays the walk and the totals once for several blocks and an
    // idle round stays a small launch.
    const long long blocks = (long long)a.batch * w.nsub;
    const int bpw = (int)(blocks <= 1024 ? 1 : blocks >= 1024 * kMaxBpw ? kMaxBpw : (blocks + 1023) / 1024);
    const dim3 per_request((unsigned)a.batch), per_part((unsigned)a.batch * ((w.nsub + bpw - 1) / bpw));
    hipLaunchKernelGGL(tree_prep_kernel, per_request, dim3(kThreads), 0, stream, a, w, mem);
    // a request has at most max_q_len - 1 rejections; the last sums kernel only walks on and prepares draws
    const int rounds = a.max_q_len - 1;
    for (int round = 0; round <= rounds; ++round) {
        hipLaunchKernelGGL(tree_sums_kernel<DT>, per_part, dim3(kThreads), 0, stream, a, w, mem, round, bpw);
        if (round < rounds) hipLaunchKernelGGL(tree_resid_kernel<DT>, per_part, dim3(kThreads), 0, stream, a, w, mem, round, bpw);
    }
    hipLaunchKernelGGL(tree_pick_kernel<DT>, per_request, dim3(kThreads), 0, stream, a, w, mem, rounds & 1);
    SS_HIP_CHECK(hipGetLastError(), "launch of the sampled tree walk");
    return SS_OK;
}

int32_t accept_tree_sample_launch(const AcceptArgs &a, hipStream_t stream)
{
    const Workspace w = carve(a.workspace, a.batch, a.total_rows, a.vocab);
    char *p = static_cast<char *>(a.workspace) + accept_workspace_bytes(a.batch, a.total_rows, a.vocab);
    TreeMem mem;
    mem.st = reinterpret_cast<TreeState *>(p);
    mem.arr = reinterpret_cast<double *>(p + align_up(sizeof(TreeState) * (size_t)a.batch, 256));
    if ((unsigned long long)a.batch * w.nsub > 0x7fffffffull) return fail(SS_ERR_UNSUPPORTED, "batch * vocab too large for one launch");
    const int32_t rc = accept_rowstats_launch(a, stream);
    if (rc != SS_OK) return rc;
    if (a.logit_dtype == SS_BF16) return tree_sample_rounds<SS_BF16>(a, w, mem, stream);
    return tree_sample_rounds<SS_F32>(a, w, mem, stream);
}

}  // namespace ss
