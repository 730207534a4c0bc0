// Verify attention on the matrix cores (gfx950), head_dim 128, bf16 queries, bf16 or e4m3 cache.
//
// The work decomposition and the tile arithmetic are described in attn_mfma_kernels.h; here are the plan kernel,
// the workspace layout and the dispatch.
#include "attn_plan.h"

namespace ss {
namespace {

// The layout of a batch beyond kPlanLanes (kPlanLanesClasses with classes): one workgroup, each wavefront a run of the requests.  One
// pass counts the classes, the other finds the places (stable, class by class) and writes the records.
constexpr int kLayoutWaves = 16;
__global__ __launch_bounds__(64 * kLayoutWaves) void attn_layout_kernel(AttnArgs a)
{
    __shared__ int count_sh[kLayoutWaves][kMaxClasses], pairs_sh[kLayoutWaves][kMaxClasses], longest_sh[kLayoutWaves];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int classes = max(a.team_blocks, 1);
    const int per = (a.batch + kLayoutWaves * 64 - 1) / (kLayoutWaves * 64) * 64;
    const int lo = min(a.batch, wave * per), hi = min(a.batch, lo + per);

    int count[kMaxClasses] = {0, 0, 0, 0, 0}, pairs[kMaxClasses] = {0, 0, 0, 0, 0}, longest = 0;
    for (int base = lo; base < hi; base += 64) {
        const int i = base + lane;
        int n = 0, c = kMaxClasses;
        if (i < hi) plan_request(a, a.kv_len[i], a.q_indptr[i + 1] - a.q_indptr[i], n, c);
        longest = max(longest, n);
#pragma unroll
        for (int k = 0; k < kMaxClasses; ++k) {
            if (k < classes) {
                count[k] += __popcll(__ballot(c == k));
                pairs[k] += c == k ? n : 0;
            }
        }
    }
    longest = wave_total(longest, Max());
#pragma unroll
    for (int k = 0; k < kMaxClasses; ++k) {
        const int x = wave_total(pairs[k], Add());
        if (lane == 0) {
            count_sh[wave][k] = count[k];
            pairs_sh[wave][k] = x;
        }
    }
    if (lane == 0) longest_sh[wave] = longest;
    __syncthreads();
    Cut cut;
    int place0[kMaxClasses], pre0[kMaxClasses];   // the next free place of each class, and the pairs in front of it, for this wavefront
    int end = 0, x = 0;
#pragma unroll
    for (int k = 0; k < kMaxClasses; ++k) {
        const int c_w = lane < kLayoutWaves ? count_sh[lane & (kLayoutWaves - 1)][k] : 0, x_w = lane < kLayoutWaves ? pairs_sh[lane & (kLayoutWaves - 1)][k] : 0;
        place0[k] = end + wave_total(lane < wave ? c_w : 0, Add());
        pre0[k] = x + wave_total(lane < wave ? x_w : 0, Add());
        end += wave_total(c_w, Add());
        x += wave_total(x_w, Add());
        cut.classes.end[k] = end;
        cut.classes.x[k] = x;
    }
    cut.choose(a, wave_total(lane < kLayoutWaves ? longest_sh[lane & (kLayoutWaves - 1)] : 0, Max()));
    if (threadIdx.x == 0) cut.publish(a);

    for (int base = lo; base < hi; base += 64) {
        const int i = base + lane;
        AttnReq r = {};
        r.cls = kMaxClasses;
        if (i < hi) {
            r.b = i;
            r.L = a.kv_len[i];
            r.q0 = a.q_indptr[i];
            r.q1 = a.q_indptr[i + 1];
            plan_request(a, r.L, r.q1 - r.q0, r.n, r.cls);
        }
        int place = 0;
#pragma unroll
        for (int k = 0; k < kMaxClasses; ++k) {
            if (k < classes) {
                const unsigned long long m = __ballot(r.cls == k);
                const int n_k = r.cls == k ? r.n : 0, incl = wave_scan_int(n_k, Add());
                if (r.cls == k) {
                    place = place0[k] + __popcll(m & ((1ull << lane) - 1));
                    r.pre = pre0[k] + incl - n_k;
                }
                place0[k] += __popcll(m);
                pre0[k] += __builtin_amdgcn_readlane(incl, 63);
            }
        }
        if (i < hi) {
            r.cpre = cut.classes.start(place, r.pre, r.cls);
            a.req[place] = r;
        }
    }
}

template <int SLOTS>
__global__ __launch_bounds__(256) void attn_plan_kernel(AttnArgs a, int heads)
{
    __shared__ Place places[SLOTS ? SLOTS * 64 : 1];
    plan_block<SLOTS>(a, heads, blockIdx.x, places);
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
    n += align_up(sizeof(int32_t) * kDescInts * ((size_t)launch_waves + 1), 256);
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
    if (a.auto_weight) p.unit_weight = kUnitWeight;
    p.team_blocks = nb > kChainRowBlocks ? attn_team_blocks(G) : 0;
    const AttnUnitChoice unit = attn_unit_choose(p);
    if (unit.splits) return attn_unit_launch(p, unit, stream, ev0, ev1);
    for (p.q_lo = 0; p.q_lo < a.max_q_len; p.q_lo += p.q_win) {
        if (!(a.reuse_plan && passes == 1)) {   // a stored plan describes one window only
            const int heads = plan_heads(p);
            const dim3 grid((unsigned)(a.batch * (a.num_kv_heads / heads)));
            if (plan_laid_out(p)) {
                hipLaunchKernelGGL(attn_layout_kernel, dim3(1), dim3(64 * kLayoutWaves), 0, stream, p);
                SS_HIP_CHECK(hipGetLastError(), "launch attn_layout_kernel");
                hipLaunchKernelGGL(attn_plan_kernel<0>, grid, dim3(256), 0, stream, p, heads);
            } else if (a.batch <= 64) {
                hipLaunchKernelGGL(attn_plan_kernel<1>, grid, dim3(256), 0, stream, p, heads);
            } else if (a.batch <= 128) {
                hipLaunchKernelGGL(attn_plan_kernel<2>, grid, dim3(256), 0, stream, p, heads);
            } else if (a.batch <= 256) {
                hipLaunchKernelGGL(attn_plan_kernel<4>, grid, dim3(256), 0, stream, p, heads);
            } else {
                hipLaunchKernelGGL(attn_plan_kernel<8>, grid, dim3(256), 0, stream, p, heads);
            }
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
