// fp32 verify attention: the path for fp32 caches or queries, head_dim 64 and any head grouping the bf16
// matrix-core kernel is not built for.  All arithmetic is fp32 (fp32 matrix instructions, fp32 probabilities).
//
// One workgroup per (request, KV head, block of 16 query rows); its wavefronts take the request's 16-token cache
// blocks in turn and are merged through LDS by their log-sum-exp.  A wavefront works on one block at a time:
//   S^T[token][row] = K[token][:] . Q[row][:]    v_mfma_f32_16x16x4_f32, a lane holds a quarter of a token's d
//   O^T[d][row]    += V[token][d] * P[row][token] the same shape; step i contracts tokens {4 jq + i}, so that P is
//                                                taken straight from the S^T accumulators
// What bounds it: short calls are a chain of dependent reads (offsets, block table, keys, values) and the merge, so
// many wavefronts per workgroup with the next block's tile in flight; long ones the fp32 matrix rate (D/2
// instructions of 32 cycles per block and 16 rows) where there are workgroups enough to fill the chip.  The cache of a
// request is not split over workgroups: one request of 65536 tokens, 32 heads of 64 over 8, is 8 to 24 workgroups at depth
// 0 to 8 and takes 0.65 ms at any of them (4.0 to 8.6 ms with one workgroup per (row, head) and one token per lane); its
// bytes alone would take about 0.04 ms.  4 requests of 64..512 tokens, 8 heads of 64, depth 4: 57 us with that form, 10.5 us
// with this one (12.2 with each lane's quarter of a key in one piece, the block ids read behind the lengths, and the weights of the
// wavefronts' parts worked out by every lane for itself); 64 requests of 1000 tokens, 56 heads over 8, e4m3, depth 4: 174 us (190).
#include "common.h"

namespace ss {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));

constexpr float kNoRef = -3.4028234663852886e38f;   // softmax reference before any visible score: no finite score lies below it

// Wavefronts per workgroup, as many as the registers of a compute unit hold (four on a SIMD at head_dim 64, two at 128).
template <int D>
constexpr int kGenericWaves = D == 64 ? 16 : 8;

template <int DT, int N>
__device__ __forceinline__ void load_run(const void *base, int64_t i, float (&x)[N])
{
    // N consecutive elements from index i (a multiple of N; every run starts on a multiple of its own size)
    if constexpr (DT == SS_F32) {
        const float4v *p = reinterpret_cast<const float4v *>(static_cast<const float *>(base) + i);
#pragma unroll
        for (int j = 0; j < N / 4; ++j) {
            const float4v v = p[j];
#pragma unroll
            for (int c = 0; c < 4; ++c) x[4 * j + c] = v[c];
        }
    } else if constexpr (DT == SS_BF16) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(static_cast<const uint16_t *>(base) + i);
        uint32_t w[N / 2];
        __builtin_memcpy(w, __builtin_assume_aligned(p, N >= 8 ? 16 : 2 * N), 2 * N);
#pragma unroll
        for (int j = 0; j < N / 2; ++j) {
            x[2 * j] = __uint_as_float(w[j] << 16);
            x[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
        }
    } else {
        const uint8_t *p = static_cast<const uint8_t *>(base) + i;
        uint32_t w[N / 4];
        __builtin_memcpy(w, __builtin_assume_aligned(p, N >= 16 ? 16 : N), N);
#pragma unroll
        for (int j = 0; j < N / 4; ++j) {   // e4m3fn bytes: the gfx950 converter implements the OCP format
            const float2v a = __builtin_amdgcn_cvt_pk_f32_fp8(w[j], false), b = __builtin_amdgcn_cvt_pk_f32_fp8(w[j], true);
            x[4 * j] = a.x; x[4 * j + 1] = a.y; x[4 * j + 2] = b.x; x[4 * j + 3] = b.y;
        }
    }
}

// A lane's quarter of a row for the score product: pieces of 16 bytes of the cache's type, those of the four lanes of a token side by side, so that
// a read takes 64 bytes of a row (with a quarter in one piece it takes 16 bytes of each of 64 places, and a compute unit gets 15 GB/s
// out of memory instead of 24).  The queries, of either type, are taken in the same order: base + piece * 4 * PIECE + jq * PIECE.
template <int DT, int D, int PIECE>
__device__ __forceinline__ void load_quarter(const void *base, int64_t row, int jq, float (&x)[D / 4])
{
#pragma unroll
    for (int j = 0; j < D / 4 / PIECE; ++j) {
        float part[PIECE];
        load_run<DT>(base, row * D + j * 4 * PIECE + jq * PIECE, part);
#pragma unroll
        for (int c = 0; c < PIECE; ++c) x[j * PIECE + c] = part[c];
    }
}

template <int D>
struct GenericTile {
    float k[D / 4];         // of the key of token (lane & 15), as load_quarter lays it out
    float v[4][D / 16];     // values of tokens 4 * (lane >> 4) + i at d = (lane & 15) * D/16 ..
    float ks, vs;
};

template <int D, int KV, int QDT>
__global__ __launch_bounds__(64 * kGenericWaves<D>) void attn_generic_kernel(AttnArgs a, int row_blocks, const int32_t *__restrict__ q_indptr, const int32_t *__restrict__ kv_len,
                                                                         const int32_t *__restrict__ block_table)
{
    // (the offsets come in as no-alias arguments of their own, so that they are scalar loads)
    constexpr int NW = kGenericWaves<D>, MB = D / 16;
    constexpr int PIECE = KV == SS_F32 ? 4 : KV == SS_BF16 ? 8 : 16;   // elements of 16 bytes
    __shared__ float part_o[NW][16][D + 4];
    __shared__ float part_m[NW][16], part_l[NW][16];

    const int rb = blockIdx.x % row_blocks, unit = blockIdx.x / row_blocks;
    const int b = unit / a.num_kv_heads, g = unit % a.num_kv_heads;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, jq = lane >> 4;
    const int G = a.num_q_heads / a.num_kv_heads;
    const int q0 = q_indptr[b], q_len = q_indptr[b + 1] - q0, rows = q_len * G;
    // This wavefront's tiles are wave, wave + NW, ..: their block ids are read 64 at a time, one per lane; the first ones together with the lengths
    // (inside the request's row of the table, whose entries past the cache's end may hold anything and are not used).
    const int32_t *bt = block_table + (int64_t)b * a.max_blocks;
    int ids = bt[min(wave + lane * NW, a.max_blocks - 1)];
    if (rb * 16 >= rows) return;
    const int L = kv_len[b], ctx = L - q_len;
    const int n = rb * 16 + n16, qi = min(n, rows - 1) / G, hh = n % G;   // this lane's query row (padding rows: the last one's mask)
    // Visible cache positions: everything before this step's new tokens, then the new tokens the
    // row's mask word names (its own node and its ancestors); for a chain those are tokens 0..i.
    const uint32_t newmask = a.tree_mask ? a.tree_mask[q0 + qi] : (2u << qi) - 1u;
    // one past the last position any row of the block sees
    const int qi_last = min(rb * 16 + 15, rows - 1) / G;
    const int end = a.tree_mask ? L : ctx + qi_last + 1;
    const int tiles = (end + kTile - 1) / kTile;

    float q[D / 4];   // B operand: the lane's quarter of its row, in the order of the keys
#pragma unroll
    for (int j = 0; j < D / 4; ++j) q[j] = 0.f;
    if (n < rows) load_quarter<QDT, D, PIECE>(a.q, (int64_t)(q0 + qi) * a.num_q_heads + g * G + hh, jq, q);

    float m = kNoRef, l = 0.f;
    float4v acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = float4v{0.f, 0.f, 0.f, 0.f};

    // The next tile's keys are requested once this tile's scores are formed and its values once they are used, so
    // that one tile's registers hold both and a read is always in flight under the arithmetic.
    GenericTile<D> t;
    auto load_k = [&](int phys) __attribute__((always_inline)) {
        const int64_t addr = (int64_t)phys * a.num_kv_heads + g;
        load_quarter<KV, D, PIECE>(a.k, addr * kTile + n16, jq, t.k);
        t.ks = KV == SS_FP8_E4M3 ? a.k_scale[addr] : 1.f;
    };
    auto load_v = [&](int phys) __attribute__((always_inline)) {
        const int64_t addr = (int64_t)phys * a.num_kv_heads + g;
#pragma unroll
        for (int i = 0; i < 4; ++i) load_run<KV>(a.v, (addr * kTile + 4 * jq + i) * D + n16 * MB, t.v[i]);
        t.vs = KV == SS_FP8_E4M3 ? a.v_scale[addr] : 1.f;
    };
    // tile ti, whose keys and values are in t; `next` is the block of the wavefront's next tile, or -1
    auto compute = [&](int ti, int next) __attribute__((always_inline)) {
        const int tok0 = ti * kTile + 4 * jq;   // first of this lane's four positions
        float4v chain[4];   // (four chains: the instruction's latency is long, and short sums round less)
#pragma unroll
        for (int c = 0; c < 4; ++c) chain[c] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < D / 4; ++j) chain[j & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[j], q[j], chain[j & 3], 0, 0, 0);
        const float4v s = (chain[0] + chain[1]) + (chain[2] + chain[3]);
        const float kscale = t.ks * a.sm_scale;
        if (next >= 0) load_k(next);
        const bool tail = ti * kTile + kTile > ctx;   // holds new tokens or slots past the end
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = s[i] * kscale;
            if (tail) {
                const int pos = tok0 + i - ctx;
                const bool see = pos < 0 || (pos < 32 && ((newmask >> pos) & 1u));
                p[i] = see ? p[i] : -INFINITY;
            }
        }
        float mx = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        if (__any(m_new > m)) {
            const float alpha = expf(m - m_new);
            l *= alpha;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb] *= alpha;
            m = m_new;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = expf(p[i] - m);
        l += (p[0] + p[1]) + (p[2] + p[3]);
        // Slots past the cache's end may hold anything; a new token some rows do not see may hold a non-finite
        // value, which must not reach those rows through 0 * value: such a tile (rare) is added entry by entry.
        bool odd = false;
        if (tail) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < MB; ++c) {
                    t.v[i][c] = tok0 + i < L ? t.v[i][c] : 0.f;
                    odd |= !(fabsf(t.v[i][c]) <= 3.4e38f);
                }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] *= t.vs;
        if (!__any(odd)) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.v[i][mb], p[i], acc[mb], 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                for (int tq = 0; tq < 4; ++tq) {   // token 4 * tq + i
                    const float pt = __shfl(p[i], tq * 16 + n16);
                    const bool see = __shfl(p[i] != 0.f || !(tok0 + i >= ctx), tq * 16 + n16);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb) {
                            const float vt = __shfl(t.v[i][mb], tq * 16 + 4 * jq + e);
                            acc[mb][e] = see ? fmaf(vt, pt, acc[mb][e]) : acc[mb][e];
                        }
                }
        }
    };

    for (int base = wave; base < tiles; base += 64 * NW) {
        if (base != wave) ids = bt[min(base + lane * NW, a.max_blocks - 1)];
        const int count = min(64, (tiles - base + NW - 1) / NW);
        int cur = __builtin_amdgcn_readlane(ids, 0);
        load_k(cur);
        load_v(cur);
        for (int i = 0; i < count; ++i) {
            const int next = i + 1 < count ? __builtin_amdgcn_readlane(ids, i + 1) : -1;
            compute(base + i * NW, next);
            if (next >= 0) load_v(next);
        }
    }

    // merge the wavefronts: accumulator row 4*jq+e of block mb is d = (4*jq+e) * MB + mb of row n16
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (jq == 0) {
        part_m[wave][n16] = m;
        part_l[wave][n16] = l;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) part_o[wave][n16][(4 * jq + e) * MB + mb] = acc[mb][e];
    __syncthreads();
    const int used = min(NW, tiles);
    for (int i = tid; i < 16 * D; i += 64 * NW) {
        const int r = __builtin_amdgcn_readfirstlane(i / D), d = i % D, nn = rb * 16 + r;   // (a wavefront's 64 elements are of one row)
        if (nn >= rows) continue;
        // lane w of every NW has what wavefront w's part weighs
        const int part = min(lane & (NW - 1), used - 1);
        const float pm = part_m[part][r], pl = part_l[part][r];
        float gm = pm;
#pragma unroll
        for (int x = 1; x < NW; x *= 2) gm = fmaxf(gm, __shfl_xor(gm, x));   // (every group of NW lanes holds all of them)
        const float sc = expf(pm - gm);
        float ls = 0.f, o = 0.f;
        float po[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) po[w] = part_o[w][r][d];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (w < used) {   // (the others had no tile)
                const float f = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sc), w));
                ls = fmaf(__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, pl), w)), f, ls);
                o = fmaf(po[w], f, o);
            }
        }
        const int64_t orow = (int64_t)(q0 + nn / G) * a.num_q_heads + g * G + nn % G;
        if (a.q_dtype == SS_F32)
            static_cast<float *>(a.out)[orow * D + d] = o / ls;
        else
            static_cast<__bf16 *>(a.out)[orow * D + d] = (__bf16)(o / ls);  // round to nearest even
        if (a.lse && d == 0) a.lse[orow] = gm + logf(ls);
    }
}

template <int D, int KV>
void launch_generic(const AttnArgs &a, int row_blocks, hipStream_t stream)
{
    const dim3 grid((unsigned)a.batch * a.num_kv_heads * row_blocks), wg(64 * kGenericWaves<D>);
    if (a.q_dtype == SS_F32)
        hipLaunchKernelGGL((attn_generic_kernel<D, KV, SS_F32>), grid, wg, 0, stream, a, row_blocks, a.q_indptr, a.kv_len, a.block_table);
    else
        hipLaunchKernelGGL((attn_generic_kernel<D, KV, SS_BF16>), grid, wg, 0, stream, a, row_blocks, a.q_indptr, a.kv_len, a.block_table);
}

template <int D>
void launch_generic_kv(const AttnArgs &a, int row_blocks, hipStream_t stream)
{
    switch (a.kv_dtype) {
    case SS_F32: launch_generic<D, SS_F32>(a, row_blocks, stream); break;
    case SS_BF16: launch_generic<D, SS_BF16>(a, row_blocks, stream); break;
    default: launch_generic<D, SS_FP8_E4M3>(a, row_blocks, stream);
    }
}

}  // namespace

int32_t attn_generic_launch(const AttnArgs &args, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1)
{
    AttnArgs a = args;
    const int row_blocks = (a.max_q_len * (a.num_q_heads / a.num_kv_heads) + 15) / 16;
    const long long per_request = (long long)a.num_kv_heads * row_blocks;   // workgroups
    // A grid has fewer than 2^32 work items (beyond that the runtime drops workgroups without an error): a larger batch goes out
    // in several launches over runs of requests.
    constexpr long long kMaxGrid = 1 << 21;   // workgroups of up to 1024 work items
    if (per_request > kMaxGrid) return fail(SS_ERR_UNSUPPORTED, "kv heads * rows too large for one launch");
    const int run = (int)(kMaxGrid / per_request);
    if (ev0) SS_HIP_CHECK(hipEventRecord(ev0, stream), "hipEventRecord");
    for (int first = 0; first < args.batch; first += run) {
        a.batch = args.batch - first < run ? args.batch - first : run;
        a.block_table = args.block_table + (int64_t)first * args.max_blocks;
        a.kv_len = args.kv_len + first;
        a.q_indptr = args.q_indptr + first;   // (rows are numbered over the whole batch)
        if (a.head_dim == 64)
            launch_generic_kv<64>(a, row_blocks, stream);
        else
            launch_generic_kv<128>(a, row_blocks, stream);
        SS_HIP_CHECK(hipGetLastError(), "launch attn_generic_kernel");
        if (args.batch - first <= run) break;
    }
    if (ev1) SS_HIP_CHECK(hipEventRecord(ev1, stream), "hipEventRecord");
    return SS_OK;
}

}  // namespace ss
