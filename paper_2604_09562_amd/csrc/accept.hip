// spec_accept: acceptance walk and resampling over full-vocabulary logits.
//
// Pass 1 (rowstats) streams every target and draft row once (the HBM-bound part): per
// 8192-entry chunk it leaves the chunk maximum and the sum of exp2((x - max) * log2e/T) in fp32
// (greedy mode: maximum and lowest-index argmax of target rows only).
// decide      one workgroup per request merges the chunk statistics of all its rows in parallel,
//             evaluates u < p/q for every draft in fp64 and fixes the accepted length and the
//             row(s) the new token is drawn from; in greedy mode it compares arg-maxima instead,
//             along the chain or, given parent pointers, down a draft tree.
// Passes 2a-2b touch only those one or two rows per request and work in fp64, so that the drawn
// token can be reproduced by an fp64 reference.  2a leaves, per 2048-entry block, the sums of the
// unnormalised exponentials of both rows (the exact normalisers Zp, Zq once added up) and the same
// sums restricted to the entries whose residual p - q is positive; which entries those are follows
// from Zp/Zq as known from pass 1, except for entries within 1e-4 of the boundary, which are set
// aside in a list (each block's entries contiguous).  2b turns the sums into block masses
// P/Zp - Q/Zq, adds the listed entries with the exact normalisers, and does the inverse-CDF search
// inside the block that holds u * mass.
// All reductions have a fixed order (no atomics): results are run-to-run identical.
#include "common.h"
#include "accept_common.h"

namespace ss {
namespace {

// ---- pass 1 ---------------------------------------------------------------------------------
// grid: batch * rows_max * ceil(nchunks / 2), rows_max from the caller's bound of k+1; workgroup (b, j, group): its wavefronts
// stream chunks 2 * group and 2 * group + 1 of request b's row j (j <= k: target row j; k < j <= 2k: draft row j-k-1; larger j:
// nothing to do), two wavefronts to a chunk.  A wavefront's 16-byte loads all go out first, then the
// values are folded vector by vector into a per-lane running (max, sum) and reduced across the wave
// with shuffles; the two halves of a chunk meet in LDS at the end.  Bound by memory: 147.7 MB (64 requests, depth 4,
// 128256 entries) take 28 us, 182 MB of target rows 31 us.  With a wavefront per chunk (twice the registers, five
// instead of eight wavefronts on a SIMD, a coarser tail) 30 and 33 us, 8.0 against 6.3 us for 8 requests of 32000; four
// wavefronts per chunk are level with two.
constexpr int kRowWaves = 2;   // wavefronts per chunk

// Every logit is read exactly once by this pass: non-temporal loads keep the stream from displacing the one or
// two rows per request that the later passes read again.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream_load16(const char *p)
{
    const u32x4 r = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(r.x, r.y, r.z, r.w);
}

template <int DT>
__global__ __launch_bounds__(kThreads) void accept_rowstats_kernel(AcceptArgs a, Workspace w)
{
    constexpr int vec = DT == SS_BF16 ? 8 : 4;       // logits per 16-byte load
    constexpr int WPC = kRowWaves;                   // wavefronts per chunk
    constexpr int PART = kChunk / WPC, CPG = 4 / WPC;   // entries of a wavefront, chunks of a workgroup
    constexpr int NV = PART / (64 * vec);            // loads per lane
    constexpr int STEP = 4;                          // vectors folded per update of the running maximum
    __shared__ float part_m[4], part_z[4];
    __shared__ int part_arg[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int groups = (w.nchunks + CPG - 1) / CPG;
    const int chunk = (blockIdx.x % groups) * CPG + wv / WPC;
    const int rows_max = a.greedy ? a.max_q_len : 2 * a.max_q_len - 1;   // rows a request can have
    const int bj = blockIdx.x / groups, b = bj / rows_max, j = bj % rows_max;
    const int t0 = a.q_indptr[b], k = a.q_indptr[b + 1] - t0 - 1;
    if (j > (a.greedy ? k : 2 * k)) return;   // (the whole workgroup)
    const bool is_draft = j > k;
    const int r = is_draft ? t0 - b + (j - k - 1) : t0 + j;
    const int64_t ry = is_draft ? (int64_t)a.total_rows + r : r;
    const void *row = row_ptr(is_draft ? a.draft : a.target, r, a.row_stride, DT);
    const int base = chunk * kChunk + (wv % WPC) * PART;
    const int64_t o = ry * w.nchunks + chunk;
    const float T = a.greedy ? 1.f : (a.temperature ? a.temperature[b] : a.temperature_scalar);
    const float sc = 1.4426950408889634f / T;

    // vector v of this lane starts at vocabulary id base + v * (64 * vec) + lane * vec
    uint4 raw[NV];
    const bool full = base + PART <= a.vocab;         // uniform: the part lies inside the vocabulary
    const int last_full = a.vocab >= vec ? (a.vocab - vec) / vec * vec : -1;
    if (full) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int i0 = base + v * (64 * vec) + lane * vec;
            raw[v] = stream_load16(static_cast<const char *>(row) + (int64_t)i0 * (DT == SS_BF16 ? 2 : 4));
        }
    } else {
        // the chunk that holds the end of the vocabulary: loads from a clamped, in-bounds address
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int i0 = base + v * (64 * vec) + lane * vec;
            const int ic = i0 < last_full ? i0 : last_full;
            raw[v] = make_uint4(0, 0, 0, 0);
            if (last_full >= 0)
                raw[v] = *reinterpret_cast<const uint4 *>(static_cast<const char *>(row) + (int64_t)ic * (DT == SS_BF16 ? 2 : 4));
        }
    }

    float m = -INFINITY, z = 0.f;
    int best = 0x7fffffff;
#pragma unroll
    for (int s0 = 0; s0 < NV; s0 += STEP) {
        float x[STEP][vec];
#pragma unroll
        for (int v = 0; v < STEP; ++v) {
            unpack<DT>(raw[s0 + v], x[v]);
            if (!full) {
                const int i0 = base + (s0 + v) * (64 * vec) + lane * vec;
                if (i0 + vec > a.vocab) {   // past the end, or the one vector that straddles it
#pragma unroll
                    for (int e = 0; e < vec; ++e) {
                        float val = -INFINITY;
                        if (i0 + e < a.vocab) {
                            if constexpr (DT == SS_BF16)
                                val = __uint_as_float((uint32_t) static_cast<const uint16_t *>(row)[i0 + e] << 16);
                            else
                                val = static_cast<const float *>(row)[i0 + e];
                        }
                        x[v][e] = val;
                    }
                }
            }
        }
        float mx = x[0][0];
#pragma unroll
        for (int v = 0; v < STEP; ++v)
#pragma unroll
            for (int e = 0; e < vec; ++e) mx = fmaxf(mx, x[v][e]);
        if (a.greedy) {
            if (mx > m) {   // a new maximum: its first position within this step, ids ascend with (v, e)
                m = mx;
                best = 0x7fffffff;
#pragma unroll
                for (int v = STEP - 1; v >= 0; --v)
#pragma unroll
                    for (int e = vec - 1; e >= 0; --e)
                        if (x[v][e] == mx) best = base + (s0 + v) * (64 * vec) + lane * vec + e;
            }
        } else {
            const float m_new = fmaxf(m, mx);
            if (m_new != -INFINITY) {
                float acc = 0.f;
#pragma unroll
                for (int v = 0; v < STEP; ++v)
#pragma unroll
                    for (int e = 0; e < vec; ++e) acc += __builtin_amdgcn_exp2f((x[v][e] - m_new) * sc);
                z = z * __builtin_amdgcn_exp2f((m - m_new) * sc) + acc;   // m == -inf: z is 0 and the factor 0
                m = m_new;
            }
        }
    }
    // across the wave, then across the chunk's wavefronts
    float cm = m;
    for (int off = 32; off; off >>= 1) cm = fmaxf(cm, __shfl_xor(cm, off));
    if (a.greedy) {
        int arg = m == cm ? best : 0x7fffffff;   // lowest vocabulary id holding the part's maximum
        for (int off = 32; off; off >>= 1) arg = min(arg, __shfl_xor(arg, off));
        if (lane == 0) {
            part_m[wv] = cm;
            part_arg[wv] = arg;
        }
        __syncthreads();
        if (lane == 0 && wv % WPC == 0 && chunk < w.nchunks) {
#pragma unroll
            for (int i = 1; i < WPC; ++i)   // (ids ascend with the wavefront: the first holder of the maximum wins)
                if (part_m[wv + i] > cm) {
                    cm = part_m[wv + i];
                    arg = part_arg[wv + i];
                }
            w.cmax[o] = cm;
            w.carg[o] = arg;
        }
        return;
    }
    if (m != -INFINITY) z *= __builtin_amdgcn_exp2f((m - cm) * sc);
    for (int off = 32; off; off >>= 1) z += __shfl_xor(z, off);
    if (lane == 0) {
        part_m[wv] = cm;
        part_z[wv] = z;
    }
    __syncthreads();
    if (lane == 0 && wv % WPC == 0 && chunk < w.nchunks) {
        float all = cm;
#pragma unroll
        for (int i = 1; i < WPC; ++i) all = fmaxf(all, part_m[wv + i]);
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < WPC; ++i)
            if (part_m[wv + i] != -INFINITY) sum += part_z[wv + i] * __builtin_amdgcn_exp2f((part_m[wv + i] - all) * sc);
        w.cmax[o] = all;
        w.csum[o] = sum;
    }
}

// ---- decide ---------------------------------------------------------------------------------
// One 256-lane workgroup per request.  Each quarter of a wavefront merges the chunk statistics of one row
// (16 lanes over the chunks; 16 rows per trip), then lanes 0..k-1 of wave 0 evaluate their draft and a
// ballot finds the first rejection.
__global__ __launch_bounds__(kThreads) void accept_decide_kernel(AcceptArgs a, Workspace w)
{
    __shared__ float row_m[kMaxRows];
    __shared__ double row_z[kMaxRows];
    __shared__ int row_arg[kMaxRows];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = a.q_indptr[b], k = a.q_indptr[b + 1] - t0 - 1, d0 = t0 - b;
    const float T = a.temperature ? a.temperature[b] : a.temperature_scalar;
    const double inv_t = a.greedy ? 1.0 : 1.0 / (double)T;

    // Wave 0's gathers (draft token, then its two logits) depend on nothing the row merge below
    // produces: they are requested first so that their latency runs under it.
    int x_early = -1;
    float lp_early = 0.f, lq_early = 0.f, u_early = 0.f;
    if (wave == 0 && lane < k && !a.tree_parent) {
        x_early = a.draft_tokens[d0 + lane];
        if (!a.greedy) {
            lp_early = load_logit(a.target, t0 + lane, a.row_stride, a.logit_dtype, x_early);
            lq_early = load_logit(a.draft, d0 + lane, a.row_stride, a.logit_dtype, x_early);
            u_early = a.u_accept[d0 + lane];
        }
    }

    if (a.greedy) {
        // Sixteen rows at a time: every quarter of a wavefront (16 lanes over the chunks) merges one row, so the
        // rows of an ordinary request are done in one trip.
        const int quarter = lane >> 4, ql = lane & 15;
        for (int j0 = 0; j0 <= k; j0 += 16) {
            const int j = j0 + wave * 4 + quarter;
            const bool live = j <= k;
            const int64_t ry = live ? t0 + j : 0;
            float m = -INFINITY;
            if (live)
                for (int c = ql; c < w.nchunks; c += 16) m = fmaxf(m, w.cmax[ry * w.nchunks + c]);
            for (int off = 8; off; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));   // (stays inside the quarter)
            int best = 0x7fffffff;
            if (live)
                for (int c = ql; c < w.nchunks; c += 16)
                    if (w.cmax[ry * w.nchunks + c] == m) best = min(best, w.carg[ry * w.nchunks + c]);
            for (int off = 8; off; off >>= 1) best = min(best, __shfl_xor(best, off));
            if (live && ql == 0) row_arg[j] = best;
        }
    } else {
        merge_row_stats(w, t0, (int64_t)a.total_rows + d0, k, inv_t, row_m, row_z);
    }
    __syncthreads();
    if (wave != 0) return;

    if (a.tree_parent) {
        // Greedy walk over a draft tree: lane i holds node i (1..k) with its parent and token; each
        // step a ballot finds the lowest-numbered child of the current node that carries the token
        // greedy decoding emits there.
        const int par = (lane >= 1 && lane <= k) ? a.tree_parent[t0 + lane] : -2;
        const int x = (lane >= 1 && lane <= k) ? a.draft_tokens[d0 + lane - 1] : -1;
        int cur = 0, n = 0, my_tok = -1, my_node = -1;
        for (;;) {   // at most k steps: every step moves to a higher-numbered node
            const int t = row_arg[cur];
            const unsigned long long hit = __ballot(par == cur && x == t);
            if (!hit) break;
            cur = __ffsll((long long)hit) - 1;
            if (lane == n) {
                my_tok = t;
                my_node = cur;
            }
            ++n;
        }
        if (lane == n) my_tok = row_arg[cur];
        if (lane < SS_OUT_WIDTH) a.out_tokens[(int64_t)b * SS_OUT_WIDTH + lane] = my_tok;
        if (lane < SS_MAX_DEPTH) a.accepted_nodes[(int64_t)b * SS_MAX_DEPTH + lane] = my_node;
        if (lane == 0) a.accepted_len[b] = n;
        return;
    }

    // every draft in parallel: lane i judges draft i
    bool reject = false;
    int x = -1;
    if (lane < k) {
        x = x_early;
        if (a.greedy) {
            reject = row_arg[lane] != x;
        } else {
            const double lp = lp_early, lq = lq_early;
            // p(x)/q(x) = exp((lp-mp)/T - (lq-mq)/T) * Zq/Zp
            const double e = (lp - (double)row_m[lane]) * inv_t - (lq - (double)row_m[k + 1 + lane]) * inv_t;
            const double rho = exp(e) * (row_z[k + 1 + lane] / row_z[lane]);
            if (a.ratio_out) a.ratio_out[d0 + lane] = (float)rho;
            reject = !((double)u_early < rho);
        }
    }
    const unsigned long long rej = __ballot(reject);
    const int n = rej ? __ffsll((long long)rej) - 1 : k;   // first rejection, k if none
    if (lane < SS_OUT_WIDTH) {
        int tok = lane < n ? x : -1;
        if (a.greedy && lane == n) tok = row_arg[n];
        a.out_tokens[(int64_t)b * SS_OUT_WIDTH + lane] = tok;   // slot n is filled by pass 2b when sampling
    }
    if (lane == 0) {
        a.accepted_len[b] = n;
        if (!a.greedy) {
            RowPick pk;
            pk.p_row = t0 + n;
            pk.q_row = n < k ? d0 + n : -1;
            pk.m_p = row_m[n];
            pk.m_q = n < k ? row_m[k + 1 + n] : 0.f;
            pk.temperature = T;
            pk.n = n;
            // kAmbEps wide in e_p / e_q is kAmbEps * T in the difference; rounding moves a difference by 2^-24 of it and of theta
            // (near the boundary it is about theta)
            pk.theta = n < k ? (float)((double)T * (double)logf((float)(row_z[n] / row_z[k + 1 + n])) + ((double)pk.m_p - (double)pk.m_q)) : 0.f;
            pk.width = (float)(kAmbEps * (double)T) + 4.0e-7f * fabsf(pk.theta);
            w.pick[b] = pk;
            w.amb_cnt[b] = 0;
            w.done[b] = 0;
        }
    }
}

// ---- pass 2a: fp64 sums per block -------------------------------------------------------------
// One 256-lane workgroup per 2048-entry block, eight entries of each row per lane.  The instructions of an entry (25 fp64 ones and 14
// others per pair) are 8 to 11 of the 17.5 us below at 4 to 5.5 cycles each; the rest is not issue: each workgroup waits for its request's record, then
// its rows and the table, before it computes.  The four sums cross the lanes together and by data-parallel moves, the power of two goes into
// the table's exponent, and which lanes are near the boundary stays in scalar registers.  Measured for 64 requests of 128256 entries: 22.7 us with
// shuffles through LDS and ldexp, 20.3 with data-parallel moves and 32 fp64 instructions per pair, 19.2 with 26 of them, a scan per sum and
// the boundary test in vector registers, 17.5 this way (the call 56.8 -> 55.3); two wavefronts per block 22.3, one 21.5 (and 6.8, 11.5
// against 4.9 us for 8 requests of 32000: a wavefront that walks a block alone is a long chain); all 32 entries of a lane as
// straight-line code 27 us (instruction fetch).  Exponentials of bf16 logits by a table of all values in LDS (64 KB, 1024-lane workgroups)
// saved 2 us of the 19; not kept for its size.
template <int DT>
__global__ __launch_bounds__(kThreads) void accept_norm_kernel(AcceptArgs a, Workspace w)
{
    __shared__ ExpTable ex;
    __shared__ double sum_sh[4][4];
    __shared__ int cnt_sh[4], base_sh;
    constexpr int WPB = kThreads / 64;
    static_assert(kSub == kThreads * 8, "eight entries per lane");
    const int b = blockIdx.x / w.nsub, sub = blockIdx.x % w.nsub, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const RowPick pk = w.pick[b];
    const bool residual = pk.q_row >= 0;
    const void *prow = row_ptr(a.target, pk.p_row, a.row_stride, DT);
    const void *qrow = residual ? row_ptr(a.draft, pk.q_row, a.row_stride, DT) : prow;
    const int i0 = sub * kSub + threadIdx.x * 8;   // vocabulary id of this lane's first entry
    Raw8<DT> rp, rq;
    load8<DT>(prow, a.vocab, i0, rp);
    if (residual) load8<DT>(qrow, a.vocab, i0, rq);
    ex.init();
    const double inv_t = 1.0 / (double)pk.temperature;
    const RowArg ap(inv_t, pk.m_p), aq(inv_t, pk.m_q);
    const int64_t o = (int64_t)b * w.nsub + sub;
    // exponentials of all entries (zp, zq) and of those whose residual p - q is positive for certain (pp, qq): the difference of an
    // entry's logits decides that in 32 bits (before, two fp64 instructions and two fp64 comparisons did)
    double zp = 0.0, zq = 0.0, pp = 0.0, qq = 0.0;
    // clearly above or below the boundary, and else too close to call before Zp/Zq are exact
    const float above = pk.theta + pk.width, below = pk.theta - pk.width;
    unsigned long long close = 0;   // lanes with such an entry
    auto pair = [&](double ep, double eq, float d) __attribute__((always_inline)) {
        zp += ep;
        zq += eq;
        const bool up = d > above;
        const double sure = up ? 1.0 : 0.0;   // (a factor costs fewer instructions than two selects of doubles)
        pp = fma(ep, sure, pp);
        qq = fma(eq, sure, qq);
        close |= __ballot(d >= below) ^ __ballot(up);
    };
    float xp[8], xq[8];
    unpack8<DT>(rp, xp);
    if (residual) unpack8<DT>(rq, xq);
    // whether all of the wavefront's exponentials are normal numbers (masked logits are not) is one test
    float low_p = xp[0], low_q = residual ? xq[0] : 0.f;
#pragma unroll
    for (int s = 1; s < 8; ++s) {
        low_p = min_or_nan(low_p, xp[s]);
        if (residual) low_q = min_or_nan(low_q, xq[s]);
    }
    const bool normal = ap.fused && (!residual || aq.fused) &&
                        !__any(!(ap.fma_form(low_p) >= kExpNormal) || (residual && !(aq.fma_form(low_q) >= kExpNormal)));
    if (!residual) {   // bonus distribution: only the normaliser of the target row is needed
        if (normal) {
#pragma unroll
            for (int s = 0; s < 8; ++s) zp += ex.normal(ap.fma_form(xp[s]));
        } else {
#pragma unroll
            for (int s = 0; s < 8; ++s) zp += ex(ap(xp[s]));
        }
    } else if (normal) {
#pragma unroll
        for (int s = 0; s < 8; ++s) pair(ex.normal(ap.fma_form(xp[s])), ex.normal(aq.fma_form(xq[s])), xp[s] - xq[s]);
    } else {
#pragma unroll
        for (int s = 0; s < 8; ++s) pair(ex(ap(xp[s])), ex(aq(xq[s])), xp[s] - xq[s]);
    }
    const double sum = wave_sum4(zp, zq, pp, qq);
    if ((lane & 15) == 15) sum_sh[wave][sum4_index(lane)] = sum;
    unsigned near = 0;   // entries of this lane that go to the list (one without mass is not worth a place)
    if (close) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const float d = xp[s] - xq[s];
            if (d >= below && d <= above && ap(xp[s]) >= kExpMass) near |= 1u << s;
        }
    }
    // The boundary entries of a block go to the request's list as one contiguous run, in wavefront, lane and entry
    // order (so their later additions have a fixed order); one counter update per block.
    int incl = __popc(near);
    const int mine = incl;
    const bool any = __any(near != 0);
    if (any) {
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(incl, off);
            if (lane >= off) incl += t;
        }
    }
    const int in_wave = __builtin_amdgcn_readlane(incl, 63);
    int total = 0, before = 0, run_base = 0;
    if (lane == 0) cnt_sh[wave] = in_wave;
    __syncthreads();
    for (int wv = 0; wv < WPB; ++wv) {
        if (wv < wave) before += cnt_sh[wv];
        total += cnt_sh[wv];
    }
    if (total > 0) {   // (the same in all of the workgroup's wavefronts)
        if (threadIdx.x == 0) base_sh = atomicAdd(&w.amb_cnt[b], total);
        __syncthreads();
        run_base = base_sh;
    }
    if (near && run_base + total <= kAmbCap) {
        int64_t l = (int64_t)b * kAmbCap + run_base + before + (incl - mine);
        for (unsigned left = near; left; left &= left - 1) {
            // read and evaluated again (the same bits) rather than kept through the loop above
            const int v = i0 + __ffs(left) - 1;
            w.amb_ep[l] = ex(ap(load_logit(prow, 0, 0, DT, v)));
            w.amb_eq[l] = ex(aq(load_logit(qrow, 0, 0, DT, v)));
            ++l;
        }
    }
    if (threadIdx.x == 0) {
        double v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = 0.0;
#pragma unroll
            for (int wv = 0; wv < WPB; ++wv) v[i] += sum_sh[wv][i];
        }
        w.zp[o] = v[0];
        if (residual) {
            w.zq[o] = v[1];
            w.pp[o] = v[2];
            w.qq[o] = v[3];
            w.blk_cnt[o] = total;
            if (total > 0) w.blk_base[o] = run_base;
        }
    }
}

// ---- pass 2b: block masses and inverse-CDF search ------------------------------------------------------------
// A chain of dependent steps: two sums over the blocks, the running sum of the block masses, and the search inside one
// block, each a wavefront scan plus one exchange between the four wavefronts.  Lane t owns a contiguous run of
// blocks (one, up to vocabularies of 512k entries), so one scan of the lanes' sums serves any number of blocks.
// 64 requests of 128256 entries: 13.4 us with shuffles through LDS and two scans, this way 7.4 us.
template <int DT>
__global__ __launch_bounds__(kThreads) void accept_pick_kernel(AcceptArgs a, Workspace w)
{
    __shared__ double tot_sh[4][2], scan_sh[4];
    __shared__ DrawShared draw_sh;
    __shared__ float sh_f[4];
    __shared__ ExpTable ex;
    const int b = blockIdx.x / kPickWgs, part = blockIdx.x % kPickWgs;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t ob = (int64_t)b * w.nsub;
    const int per = blocks_per_lane(w.nsub);
    const int c0 = tid * per, c1 = min(c0 + per, w.nsub);
    // everything that does not depend on anything else is requested up front (what a bonus request has no values for
    // is read and not used)
    const RowPick pk = w.pick[b];
    const int amb = w.amb_cnt[b];
    const float u_s = a.u_sample[b];
    const int64_t o0 = ob + min(c0, w.nsub - 1);
    const double zp0 = w.zp[o0], zq0 = w.zq[o0], pp0 = w.pp[o0], qq0 = w.qq[o0];
    const int cnt0 = w.blk_cnt[o0], base0 = w.blk_base[o0];
    const bool residual = pk.q_row >= 0;
    const int namb = residual ? amb : 0;
    const bool listed = namb <= kAmbCap;
    if (listed && part != 0) return;   // one workgroup does the whole request unless the list overflowed
    int32_t *dst = a.out_tokens + (int64_t)b * SS_OUT_WIDTH + pk.n;
    ex.init();

    // exact normalisers
    double zp = c0 < c1 ? zp0 : 0.0, zq = c0 < c1 && residual ? zq0 : 0.0;
    for (int c = c0 + 1; c < c1; ++c) {
        zp += w.zp[ob + c];
        if (residual) zq += w.zq[ob + c];
    }
    zp = wave_scan(zp);
    zq = wave_scan(zq);
    if (lane == 63) {
        tot_sh[wave][0] = zp;
        tot_sh[wave][1] = zq;
    }
    __syncthreads();
    zp = (tot_sh[0][0] + tot_sh[1][0]) + (tot_sh[2][0] + tot_sh[3][0]);
    zq = residual ? (tot_sh[0][1] + tot_sh[1][1]) + (tot_sh[2][1] + tot_sh[3][1]) : 1.0;
    const double inv_t = 1.0 / (double)pk.temperature, inv_zp = 1.0 / zp, inv_zq = 1.0 / zq;
    const RowArg ap(inv_t, pk.m_p), aq(inv_t, pk.m_q);
    // residual (or bonus) mass of one vocabulary entry
    auto entry_mass = [&](float lp, float lq) __attribute__((always_inline)) {
        const double p = ex(ap(lp)) * inv_zp;
        if (!residual) return p;
        const double q = ex(aq(lq)) * inv_zq;
        return p > q ? p - q : 0.0;
    };
    if (!listed) {
        // Too many entries near p == q to list (rows that nearly coincide, or many equal logit pairs on
        // the boundary): the request's workgroups share the blocks and compute every mass entry by
        // entry; the last one to deliver (a counter in device memory) goes on to draw the token.
        for (int c = part; c < w.nsub; c += kPickWgs) {
            float yp[kSubPer], yq[kSubPer];
            load_slots<DT, kSubPer, false>(row_ptr(a.target, pk.p_row, a.row_stride, DT), a.vocab, c * kSub, tid, yp);
            load_slots<DT, kSubPer, false>(row_ptr(a.draft, pk.q_row, a.row_stride, DT), a.vocab, c * kSub, tid, yq);
            double m = 0.0;
#pragma unroll
            for (int i = 0; i < kSubPer; ++i) m += entry_mass(yp[i], yq[i]);
            m = block_sum<double>(m, scan_sh);
            if (tid == 0) w.sc[ob + c] = m;
        }
        __shared__ int ticket_sh;
        __threadfence();   // the masses are out before the counter moves
        __syncthreads();
        if (tid == 0) ticket_sh = atomicAdd(&w.done[b], 1);
        __syncthreads();
        if (ticket_sh != kPickWgs - 1) return;
        __threadfence();   // and the other workgroups' masses are read from memory, not from a stale cache line
    }
    // mass of block c, given its sums and its listed run (the boundary entries, now that Zp and Zq are exact, in
    // their stored order)
    auto block_mass = [&](double zpc, double ppc, double qqc, int cnt, int base) __attribute__((always_inline)) {
        if (!residual) return zpc / zp;
        double m = ppc * inv_zp - qqc * inv_zq;
        m = m > 0.0 ? m : 0.0;
        if (namb > 0 && cnt > 0) {
            const int64_t l0 = (int64_t)b * kAmbCap + base;
            double add = 0.0;
            for (int e = 0; e < cnt; ++e) {
                const double r = w.amb_ep[l0 + e] * inv_zp - w.amb_eq[l0 + e] * inv_zq;
                add += r > 0.0 ? r : 0.0;
            }
            m += add;
        }
        return m;
    };
    auto mass_of = [&](int c) __attribute__((always_inline)) {
        if (!listed) return w.sc[ob + c];
        if (c == c0) return block_mass(zp0, pp0, qq0, cnt0, base0);
        return block_mass(w.zp[ob + c], w.pp[ob + c], w.qq[ob + c], w.blk_cnt[ob + c], w.blk_base[ob + c]);
    };

    auto entries = [&](int cstar, double (&r)[kSubPer]) __attribute__((always_inline)) {
        float xp[kSubPer], xq[kSubPer];
        load_slots<DT, kSubPer, true>(row_ptr(a.target, pk.p_row, a.row_stride, DT), a.vocab, cstar * kSub, tid, xp);
        if (residual)
            load_slots<DT, kSubPer, true>(row_ptr(a.draft, pk.q_row, a.row_stride, DT), a.vocab, cstar * kSub, tid, xq);
        else {
#pragma unroll
            for (int i = 0; i < kSubPer; ++i) xq[i] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < kSubPer; ++i) r[i] = entry_mass(xp[i], xq[i]);
    };
    int tok = draw_token(w.nsub, u_s, draw_sh, mass_of, entries);
    if (tok < 0) {
        // p_n == q_n exactly: no residual mass; fall back to the lowest-index argmax of the target row
        float best = -INFINITY;
        for (int v = tid; v < a.vocab; v += kThreads)
            best = fmaxf(best, load_logit(a.target, pk.p_row, a.row_stride, DT, v));
        best = block_max(best, sh_f);
        tok = lowest_index_of(a.target, pk.p_row, a.row_stride, DT, a.vocab, best, draw_sh);
    }
    if (tid == 0) *dst = tok;
}

}  // namespace

size_t accept_workspace_bytes(int batch, int total_rows, int vocab)
{
    const size_t nch = num_chunks(vocab), nsub = num_sub(vocab);
    const size_t rows = 2 * (size_t)total_rows - batch;
    size_t n = 3 * align_up(sizeof(float) * rows * nch, 256);
    n += align_up(sizeof(RowPick) * (size_t)batch, 256);
    n += 5 * align_up(sizeof(double) * (size_t)batch * nsub, 256);
    n += 2 * align_up(sizeof(double) * (size_t)batch * kAmbCap, 256);
    n += 2 * align_up(sizeof(int32_t) * (size_t)batch * nsub, 256);
    n += 2 * align_up(sizeof(int32_t) * (size_t)batch, 256);
    return n + 256;
}

// The first pass over the whole batch.  A grid has fewer than 2^32 work items (beyond that the runtime drops workgroups
// without an error), and the bound of the rows, 41 per request if the caller gives none, counts for every request: a larger
// batch goes out in several launches over runs of requests.
template <int DT>
static int32_t rowstats_launch_dt(const AcceptArgs &args, const Workspace &w, hipStream_t stream)
{
    constexpr long long kMaxGrid = 1 << 23;   // workgroups of 256 work items
    const long long per_request = (long long)(args.greedy ? args.max_q_len : 2 * args.max_q_len - 1) * ((w.nchunks * kRowWaves + 3) / 4);
    if (per_request > kMaxGrid) return fail(SS_ERR_UNSUPPORTED, "vocab too large for one launch");
    const int run = (int)(kMaxGrid / per_request);
    AcceptArgs a = args;
    for (int first = 0; first < args.batch; first += run) {
        a.batch = args.batch - first < run ? args.batch - first : run;
        a.q_indptr = args.q_indptr + first;   // (target rows are numbered over the whole batch)
        if (args.temperature) a.temperature = args.temperature + first;
        // A request's draft rows start at its first target row less its number, which counts from `first` here.
        if (args.draft) a.draft = static_cast<const char *>(args.draft) - first * args.row_stride * (DT == SS_BF16 ? 2 : 4);
        a.total_rows = args.total_rows - first;
        hipLaunchKernelGGL(accept_rowstats_kernel<DT>, dim3((unsigned)(a.batch * per_request)), dim3(kThreads), 0, stream, a, w);
        SS_HIP_CHECK(hipGetLastError(), "launch accept_rowstats_kernel");
        if (args.batch - first <= run) break;
    }
    return SS_OK;
}

template <int DT>
static int32_t accept_launch_dt(const AcceptArgs &a, const Workspace &w, hipStream_t stream)
{
    const int32_t rc = rowstats_launch_dt<DT>(a, w, stream);
    if (rc != SS_OK) return rc;
    hipLaunchKernelGGL(accept_decide_kernel, dim3(a.batch), dim3(kThreads), 0, stream, a, w);
    SS_HIP_CHECK(hipGetLastError(), "launch accept_decide_kernel");
    if (a.greedy) return SS_OK;
    hipLaunchKernelGGL(accept_norm_kernel<DT>, dim3((unsigned)a.batch * w.nsub), dim3(kThreads), 0, stream, a, w);
    SS_HIP_CHECK(hipGetLastError(), "launch accept_norm_kernel");
    hipLaunchKernelGGL(accept_pick_kernel<DT>, dim3((unsigned)a.batch * kPickWgs), dim3(kThreads), 0, stream, a, w);
    SS_HIP_CHECK(hipGetLastError(), "launch accept_pick_kernel");
    return SS_OK;
}

int32_t accept_launch(const AcceptArgs &a, hipStream_t stream)
{
    const Workspace w = carve(a.workspace, a.batch, a.total_rows, a.vocab);
    if ((unsigned long long)a.batch * w.nsub > 0x7fffffffull)
        return fail(SS_ERR_UNSUPPORTED, "batch * vocab too large for one launch");
    if (a.logit_dtype == SS_BF16) return accept_launch_dt<SS_BF16>(a, w, stream);
    return accept_launch_dt<SS_F32>(a, w, stream);
}

int32_t accept_rowstats_launch(const AcceptArgs &a, hipStream_t stream)
{
    const Workspace w = carve(a.workspace, a.batch, a.total_rows, a.vocab);
    if (a.logit_dtype == SS_BF16) return rowstats_launch_dt<SS_BF16>(a, w, stream);
    return rowstats_launch_dt<SS_F32>(a, w, stream);
}

}  // namespace ss
