// Verify attention with a workgroup per unit (a request's rows of one KV head), or several to a unit and a small kernel that merges them: one launch
// or two where the streaming kernels take a plan, a stream and a merge, each a chain of dependent reads.
//
// Serves the calls of the matrix-core kernels (head_dim 128, bf16 queries, bf16 or e4m3 caches, groups of 1/2/4/8) in which no unit can be
// long; the rule stands in unit_rule.h.
//
// What bounds it: the chain of lengths, block ids, tiles, exchange and rows written (6 us for 64 tokens, launch included); beyond a few steps
// what a compute unit gets out of memory, about 60 GB/s while the chip is not full.
//
// Eight or four wavefronts of 256 registers, two to a SIMD: while one waits for a result, or for its loads to be accepted, the other issues.
// Wavefronts 2s and 2s + 1 are siblings.  A step takes a pair of tiles (32 tokens) to a wavefront, 256 or 128 tokens:
//   scores   S^T = K Q^T of the wavefront's own pair                                     (all row blocks)
//   softmax  P as bf16 into LDS
//   output   O^T += V^T P^T of both siblings' pairs, the sibling's P from LDS, for the wavefront's half of the head dimension
// so that a wavefront holds accumulators of half a row: with five row blocks 80 registers instead of 160, which is what lets two
// wavefronts share a SIMD.  No matrix or vector work is done twice for it; what it costs is 1 KB of LDS written and 2 KB read per row block and
// wavefront, and a barrier or two per step.
//
// The operands' lane layouts are those of attn_mfma_kernels.h: for S^T a K tile is the A operand, for O^T the contraction runs over
// the 32 tokens of a pair, lane group jq bringing tokens 4 jq .. 4 jq + 3 of either tile, so that P is taken straight from the
// accumulators of S^T; V is loaded as four consecutive d of a token per lane, the M-blocks being the four interleaved phases.
//
// The softmax reference is the largest score so far, not one that lags as in the streaming kernels: the largest probabilities stay exact in bf16
// (1.68e-3 to 1.74e-3 from 64 bits over the range, the streaming kernels 1.69e-3 to 2.0e-3; a reference that lags by up to 2^8 for a whole
// unit 1.9e-3 to 2.3e-3, and 5 % faster).
#include <type_traits>

#include <hip/hip_ext.h>

#include "attn_plan.h"
#include "tree_window.h"

namespace ss {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int D = kMfmaHeadDim;
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
constexpr float kNoMax = -1.0e30f;   // reference before any score was seen, as in attn_mfma_kernels.h
constexpr int kNonTemporal = 2;                     // tiles are read once
constexpr int kRowStride = 17;                      // 16-byte words from one bf16 row to the next in LDS (16 and one of padding)
constexpr int kHalfRow = 17;                        // float4 from one row of a staged half block to the next (16 and one of padding)

// (What is read at constant offsets stands first: an offset inside an LDS instruction ends at 64 KB.)
template <int TEAM>
struct UnitLds {
    u32x4 q[kMaxRowBlocks * 16 * kRowStride];            // the query rows
    float top[2][TEAM][kMaxRowBlocks * 16];             // by step parity: references, or row maxima of a step's pairs; at the end the references
    float sum[TEAM][kMaxRowBlocks * 16];
    union {
        uint4 p[2][TEAM][kMaxRowBlocks][64];            // P operands by step parity, wavefront, row block
        float4v o[2][TEAM][16 * kHalfRow];              // at the unit's end: one row block's halves of all wavefronts, two buffers
    };
};

__device__ __forceinline__ uint32_t pack_hi16(uint32_t lo_src, uint32_t hi_src) { return __builtin_amdgcn_perm(hi_src, lo_src, 0x07060302u); }
__device__ __forceinline__ uint32_t pack_lo16(uint32_t lo_src, uint32_t hi_src) { return __builtin_amdgcn_perm(hi_src, lo_src, 0x05040100u); }
template <bool HI>
__device__ __forceinline__ uint32_t fp8x2_to_bf16x2(uint32_t w)   // exact
{
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HI));
}
__device__ __forceinline__ uint32_t pack_bf16(float x, float y)
{
    const float2v v = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// The maximum over the four rows of 16 lanes.
__device__ __forceinline__ float max_over_rows(float x)
{
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
    const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
}
// Waits for this wavefront's LDS accesses only (not for the tiles in flight), then for the others.
__device__ __forceinline__ void team_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

struct Unit {
    int b, g, L, q0, q_len, rows, lane, wave;
    int group_log;             // log2 of the query heads per KV head
    int tile_lo, tiles;        // this workgroup's share of the cache's tiles: from tile_lo to before `tiles`
    int shares;                // workgroups of the unit that have one
    int slot;                  // of the partial, if there are more than this one
};

// NB: 16-row blocks of the request's query rows
// TEAM: wavefronts of the workgroup
template <int NB, int TEAM, bool FP8, bool TREE>
__device__ __forceinline__ void walk_unit(const AttnArgs &a, UnitLds<TEAM> &lds, const Unit &u, const int32_t *__restrict__ table,
                                          const float *__restrict__ k_scale, const float *__restrict__ v_scale)
{
    constexpr int kTeam = TEAM, kStepTiles = 2 * TEAM;
    constexpr bool QLDS = NB >= 3;
    // OWN: each sibling's pairs have a reference of their own, and accumulators too (the largest of 32 probabilities is exact, as in the
    // streaming kernels' first pairs: four requests of 64 tokens 1.73e-3 from 64 bits either way, with a reference of 64 tokens 1.78e-3).  From four
    // row blocks on there is room for one set of accumulators, and the siblings agree on a reference; with e4m3 caches a probability is
    // rounded with its tile's scale, and no reference makes it exact.
    constexpr bool OWN = NB <= 3 && !FP8;
    constexpr bool LATE = NB == 5 && !FP8;   // registers: the second pair's values are asked for after the scores
    constexpr int BYTES = kTile * D * (FP8 ? 1 : 2), ROW = D * (FP8 ? 1 : 2);
    const int lane = u.lane, wave = u.wave, half = wave & 1;
    const int r16 = lane & 15, jq = lane >> 4;
    const int ctx = u.L - u.q_len;
    const float sc2 = a.sm_scale * kLog2e;
    const int heads = a.num_kv_heads;

    // ---- queries: row n of the unit is head n % G of the group at new token n / G; rows the unit does not have read as zeros ----
    const long long q_row = (long long)a.num_q_heads * D * 2;
    const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(static_cast<const char *>(a.q)) + (u.q0 * q_row + ((long long)u.g << u.group_log) * (D * 2)), 0, (int)(u.q_len * q_row), 0x00020000);
    // Four whole rows to an instruction, shared out over the wavefronts; operands come from LDS.  (In operand order, 16 bytes of each of sixteen
    // rows in consecutive lanes, an instruction takes the memory pipeline four times as long.)
    constexpr int LINES = (NB * 4 + kTeam - 1) / kTeam;
    u32x4 qline[LINES];
#pragma unroll
    for (int i = 0; i < LINES; ++i) {
        const int n = (wave + i * kTeam) * 4 + jq;   // (of the last ones some are past the row blocks: not a row either)
        const int off = n < u.rows ? (n >> u.group_log) * (int)q_row + (n & ((1 << u.group_log) - 1)) * (D * 2) + r16 * 16 : 0x7fffff00;
        qline[i] = __builtin_amdgcn_raw_buffer_load_b128(qr, off, 0, 0);
    }
    bf16x8 qreg[QLDS ? 1 : NB][4];
    int lim[TREE ? 1 : NB];            // chain: the last position this lane's row sees
    uint32_t newmask[TREE ? NB : 1];   // tree: the new tokens it sees (padding rows: all of them)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = nb * 16 + r16, qi = n >> u.group_log;
        const bool ok = n < u.rows;
        if constexpr (TREE) {
            const uint32_t m = a.tree_mask[u.q0 + (ok ? qi : 0)];
            newmask[nb] = ok ? m : (2u << (u.q_len - 1)) - 1u;
        } else {
            lim[nb] = min(ok ? ctx + qi : u.L - 1, u.tiles * kTile - 1);
        }
    }

    // ---- tiles.  Buffer loads through a descriptor of exactly the tile, of no bytes (zeros) for one past the cache's end. ----
    u32x4 kr[2][FP8 ? 2 : 4];          // own pair, in the order of memory
    typedef typename std::conditional<FP8, uint32_t, u32x2>::type vword;
    vword vr[4][4];                    // both siblings' tiles: d = 64 half + 4 r16 .. + 3 of tokens 4 jq + e
    float kscale[2], vscale[2];
    auto tile_rsrc = [&](const void *base, int id, bool live) __attribute__((always_inline)) {
        const unsigned long long at = (unsigned long long)(uint32_t)(id * heads + u.g) * BYTES;   // (the product fits 31 bits)
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(static_cast<const char *>(base)) + at, 0, live ? BYTES : 0, 0x00020000);
    };
    auto load_keys = [&](int tile0, const int (&ids)[4]) __attribute__((always_inline)) {   // tile0: first of the siblings' four tiles
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int id = half ? ids[2 + h] : ids[h];
            const __amdgpu_buffer_rsrc_t r = tile_rsrc(a.k, id, tile0 + 2 * half + h < u.tiles);
#pragma unroll
            for (int i = 0; i < (FP8 ? 2 : 4); ++i) kr[h][i] = __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, i * 1024, kNonTemporal);
        }
    };
    auto load_scales = [&](int tile0, const int (&ids)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (FP8) {
                const int id = half ? ids[2 + h] : ids[h];
                const int at = id * heads + u.g;
                kscale[h] = k_scale[at] * sc2;
                vscale[h] = v_scale[at];
            } else {
                kscale[h] = sc2;
                vscale[h] = 1.f;
            }
        }
    };
    auto load_values = [&](int tile0, const int (&ids)[4], int t) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t r = tile_rsrc(a.v, ids[t], tile0 + t < u.tiles);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int off = 4 * jq * ROW + half * (ROW / 2) + r16 * (FP8 ? 4 : 8);
            if constexpr (FP8) vr[t][e] = __builtin_amdgcn_raw_buffer_load_b32(r, off, e * ROW, kNonTemporal);
            else vr[t][e] = __builtin_amdgcn_raw_buffer_load_b64(r, off, e * ROW, kNonTemporal);
        }
    };
    auto load_ids = [&](int tile0, int (&ids)[4]) __attribute__((always_inline)) {   // (inside the row: entries past the end may hold anything)
#pragma unroll
        for (int t = 0; t < 4; ++t) ids[t] = table[min(tile0 + t, u.tiles - 1)];
    };

    int tile0 = u.tile_lo + (wave >> 1) * 4;
    int ids[4];
    load_ids(tile0, ids);
    load_keys(tile0, ids);
    load_scales(tile0, ids);
#pragma unroll
    for (int t = 0; t < (LATE ? 2 : 4); ++t) load_values(tile0, ids, t);

    float m_run[NB], l_run[NB];         // of the wavefront's own pairs
    float m_pair[2][OWN ? NB : 1];      // what the accumulators are relative to
    float4v acc[OWN ? 2 : 1][4][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        m_run[nb] = kNoMax;
        l_run[nb] = 0.f;
#pragma unroll
        for (int c = 0; c < (OWN ? 2 : 1); ++c) {
            if constexpr (OWN) m_pair[c][nb] = kNoMax;
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) acc[c][mb][nb] = float4v{0.f, 0.f, 0.f, 0.f};
        }
    }
    // operand of k-step ks and row block nb: row 16 nb + r16, 16-byte word 4 ks + jq (e4m3: 8 (ks / 2) + 2 jq + ks % 2, as its keys come)
    const u32x4 *const qs = lds.q + r16 * kRowStride + (FP8 ? 2 : 1) * jq;
    auto q_at = [](int nb, int ks) __attribute__((always_inline)) { return nb * 16 * kRowStride + (FP8 ? (ks >> 1) * 8 + (ks & 1) : ks * 4); };
#pragma unroll
    for (int i = 0; i < LINES; ++i)
        if (wave + i * kTeam < NB * 4) lds.q[((wave + i * kTeam) * 4 + jq) * kRowStride + r16] = qline[i];
    team_barrier();
    if constexpr (!QLDS) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) qreg[nb][ks] = __builtin_bit_cast(bf16x8, qs[q_at(nb, ks)]);
    }

    const int steps = (u.tiles - u.tile_lo + kStepTiles - 1) / kStepTiles;
    for (int step = 0;; ++step) {
        const bool more = step + 1 < steps;
        const int par = step & 1;
        int next[4];
        load_ids(tile0 + kStepTiles, next);   // (clamped to the cache's last block: also past the end)

        // scores
        float4v s[NB][2];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) s[nb][0] = s[nb][1] = float4v{0.f, 0.f, 0.f, 0.f};
        {
            // Keys as operands: read in the order of memory and turned through LDS, a tile at a time, in this wavefront's place for P of this
            // step (its sibling is done with what stood there two steps ago).  Rows stand one 16-byte word further apart than they are long.
            constexpr int KSEG = FP8 ? 8 : 16, KROW = KSEG + 1;
            static_assert(16 * KROW <= kMaxRowBlocks * 64, "a tile fits the place of P");
            u32x4 *const to = reinterpret_cast<u32x4 *>(&lds.p[par][wave][0][0]) + lane / KSEG * KROW + lane % KSEG;
            const u32x4 *const from = reinterpret_cast<const u32x4 *>(&lds.p[par][wave][0][0]) + r16 * KROW + jq;
            bf16x8 kop[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < (FP8 ? 2 : 4); ++i) to[i * (64 / KSEG) * KROW] = kr[h][i];
                __builtin_amdgcn_wave_barrier();   // (LDS serves a wavefront's requests in order; this keeps the compiler to it)
                u32x4 kw[FP8 ? 2 : 4];
#pragma unroll
                for (int i = 0; i < (FP8 ? 2 : 4); ++i) kw[i] = from[i * 4];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    if constexpr (FP8) {
                        const uint32_t w0 = kw[ks >> 1][(ks & 1) * 2], w1 = kw[ks >> 1][(ks & 1) * 2 + 1];
                        kop[h][ks] = __builtin_bit_cast(bf16x8, make_uint4(fp8x2_to_bf16x2<false>(w0), fp8x2_to_bf16x2<true>(w0),
                                                                           fp8x2_to_bf16x2<false>(w1), fp8x2_to_bf16x2<true>(w1)));
                    } else {
                        kop[h][ks] = __builtin_bit_cast(bf16x8, kw[ks]);
                    }
                }
            }
            constexpr int NOPS = 4 * NB, AHEAD = QLDS ? 4 : 1;   // query operands from LDS are requested ahead of their use
            u32x4 qb[AHEAD];
            if constexpr (QLDS) {
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) qb[i] = qs[q_at(i % NB, i / NB)];
            }
#pragma unroll
            for (int i = 0; i < NOPS; ++i) {
                const int ks = i / NB, nb = i % NB;
                bf16x8 qop;
                if constexpr (QLDS) {
                    qop = __builtin_bit_cast(bf16x8, qb[i % AHEAD]);
                    if (i + AHEAD < NOPS) qb[i % AHEAD] = qs[q_at((i + AHEAD) % NB, (i + AHEAD) / NB)];
                } else {
                    qop = qreg[nb][ks];
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) s[nb][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[h][ks], qop, s[nb][h], 0, 0, 0);
                if constexpr (QLDS) __builtin_amdgcn_sched_barrier(0);
            }
        }
        // the keys' registers are free: the next step's go out under softmax and output
        const float ks_now[2] = {kscale[0], kscale[1]}, vs_now[2] = {vscale[0], vscale[1]};
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LATE) {
            load_values(tile0, ids, 2);
            load_values(tile0, ids, 3);
        }
        load_keys(tile0 + kStepTiles, next);   // (past the end: nothing)
        load_scales(tile0 + kStepTiles, next);
        __builtin_amdgcn_sched_barrier(0);

        // softmax.  The scores are formed once (times the scale, in units of log2); masked only in pairs that reach into the new tokens or past
        // this workgroup's share.
        const int tok0 = (tile0 + 2 * half) * kTile + jq * 4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[nb][h][e] *= ks_now[h];
        if ((tile0 + 2 * half + 2) * kTile > min(ctx, u.tiles * kTile)) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int p0 = tok0 + h * kTile;
                    if constexpr (TREE) {
                        const uint32_t vis = p0 < u.tiles * kTile ? tree_visible4(newmask[nb], p0 - ctx) : 0;   // (nothing past this share)
#pragma unroll
                        for (int e = 0; e < 4; ++e) s[nb][h][e] = ((vis >> e) & 1u) ? s[nb][h][e] : -INFINITY;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) s[nb][h][e] = p0 + e > lim[nb] ? -INFINITY : s[nb][h][e];
                    }
                }
        }
        auto top8 = [&](int nb) __attribute__((always_inline)) {
            return fmaxf(fmaxf(fmaxf(s[nb][0][0], s[nb][0][1]), fmaxf(s[nb][0][2], s[nb][0][3])),
                         fmaxf(fmaxf(s[nb][1][0], s[nb][1][1]), fmaxf(s[nb][1][2], s[nb][1][3])));
        };
        auto probabilities = [&](int nb) __attribute__((always_inline)) {
            uint32_t w[4];
            float sum = 0.f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(s[nb][h][e] - m_run[nb]);
                sum += (p[0] + p[1]) + (p[2] + p[3]);
                w[2 * h] = pack_bf16(p[0] * vs_now[h], p[1] * vs_now[h]);
                w[2 * h + 1] = pack_bf16(p[2] * vs_now[h], p[3] * vs_now[h]);
            }
            l_run[nb] += sum;
            asm volatile("" : "+v"(l_run[nb]));   // (here: put off past the barrier, the eight summands stay in registers)
            lds.p[par][wave][nb][lane] = make_uint4(w[0], w[1], w[2], w[3]);
        };
        // The reference is the largest score so far, of the wavefront's own pairs or of both siblings'.
        auto move_to = [&](int nb, float m_new) __attribute__((always_inline)) {
            const float alpha = __builtin_amdgcn_exp2f(m_run[nb] - m_new);
            m_run[nb] = m_new;
            l_run[nb] *= alpha;
            return alpha;
        };
        float m_next[2][OWN ? NB : 1];
        if constexpr (OWN) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                move_to(nb, fmaxf(m_run[nb], max_over_rows(top8(nb))));
                if (jq == 0) lds.top[par][wave][nb * 16 + r16] = m_run[nb];
                probabilities(nb);
            }
            team_barrier();
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) m_next[c][nb] = lds.top[par][(wave & ~1) + c][nb * 16 + r16];
        } else {
            float mine[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                mine[nb] = max_over_rows(top8(nb));
                if (jq == 0) lds.top[0][wave][nb * 16 + r16] = mine[nb];
            }
            team_barrier();
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const float m_new = fmaxf(m_run[nb], fmaxf(mine[nb], lds.top[0][wave ^ 1][nb * 16 + r16]));
                if (__any(m_new != m_run[nb])) {
                    const float alpha = move_to(nb, m_new);
#pragma unroll
                    for (int mb = 0; mb < 4; ++mb) acc[0][mb][nb] *= alpha;
                }
                probabilities(nb);
                __builtin_amdgcn_sched_barrier(0);   // (registers: a block at a time)
            }
            team_barrier();
        }

        // output
        // one sibling's pair after the other: its values' operands (vop[mb]: phase mb of the pair's 32 tokens), the next step's loads into
        // the registers that are free, its part of the product
#pragma unroll
        for (int sib = 0; sib < 2; ++sib) {
            uint32_t vop[4][4];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {   // word h of a token's four values holds phases 2h and 2h + 1
                    uint32_t w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (FP8) w[e] = h ? fp8x2_to_bf16x2<true>(vr[2 * sib + t][e]) : fp8x2_to_bf16x2<false>(vr[2 * sib + t][e]);
                        else w[e] = vr[2 * sib + t][e][h];
                    }
                    vop[2 * h][2 * t] = pack_lo16(w[0], w[1]);
                    vop[2 * h][2 * t + 1] = pack_lo16(w[2], w[3]);
                    vop[2 * h + 1][2 * t] = pack_hi16(w[0], w[1]);
                    vop[2 * h + 1][2 * t + 1] = pack_hi16(w[2], w[3]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!LATE || sib == 0) {
                load_values(tile0 + kStepTiles, next, 2 * sib);
                load_values(tile0 + kStepTiles, next, 2 * sib + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            // slots at or past kv_len may hold anything: cleared, so that 0 * garbage cannot occur
            if ((tile0 + 2 * sib + 2) * kTile > u.L) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int p0 = (tile0 + 2 * sib + t) * kTile + jq * 4;
                    const uint32_t m01 = (p0 + 0 < u.L ? 0x0000ffffu : 0u) | (p0 + 1 < u.L ? 0xffff0000u : 0u);
                    const uint32_t m23 = (p0 + 2 < u.L ? 0x0000ffffu : 0u) | (p0 + 3 < u.L ? 0xffff0000u : 0u);
#pragma unroll
                    for (int mb = 0; mb < 4; ++mb) {
                        vop[mb][2 * t] &= m01;
                        vop[mb][2 * t + 1] &= m23;
                    }
                }
            }
            if constexpr (OWN) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    if (__any(m_next[sib][nb] != m_pair[sib][nb])) {
                        const float alpha = __builtin_amdgcn_exp2f(m_pair[sib][nb] - m_next[sib][nb]);
                        m_pair[sib][nb] = m_next[sib][nb];
#pragma unroll
                        for (int mb = 0; mb < 4; ++mb) acc[sib][mb][nb] *= alpha;
                    }
            }
            const uint4 (&pair)[kMaxRowBlocks][64] = lds.p[par][(wave & ~1) + sib];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const bf16x8 pop = __builtin_bit_cast(bf16x8, pair[nb][lane]);
#pragma unroll
                for (int mb = 0; mb < 4; ++mb)
                    acc[OWN ? sib : 0][mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, make_uint4(vop[mb][0], vop[mb][1], vop[mb][2], vop[mb][3])), pop, acc[OWN ? sib : 0][mb][nb], 0, 0, 0);
            }
        }
        tile0 += kStepTiles;
        if (!more) break;
#pragma unroll
        for (int t = 0; t < 4; ++t) ids[t] = next[t];
    }

    // ---- the unit's end: brought to one reference, the siblings' results are added through LDS, block by block ----
    float weight[OWN ? 2 : 1][NB];   // of the accumulators against the unit's reference
    team_barrier();   // (the references of the last step have been read, and P, whose place the blocks take)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
        if (jq == 0) lds.top[0][wave][nb * 16 + r16] = m_run[nb];
    team_barrier();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float m = m_run[nb];
#pragma unroll
        for (int w = 0; w < kTeam; ++w) m = fmaxf(m, lds.top[0][w][nb * 16 + r16]);
        float l = l_run[nb] * __builtin_amdgcn_exp2f(m_run[nb] - m);   // (who saw nothing: 0 times sums of 0)
#pragma unroll
        for (int c = 0; c < (OWN ? 2 : 1); ++c) weight[c][nb] = __builtin_amdgcn_exp2f((OWN ? m_pair[c][OWN ? nb : 0] : m_run[nb]) - m);
        m_run[nb] = m;
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (jq == 0) lds.sum[wave][nb * 16 + r16] = l;
    }
    const int d4 = lane & 31;   // four values of a row to a lane
    const long long first_row = (long long)u.q0 * a.num_q_heads + ((long long)u.g << u.group_log);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float4v *o = lds.o[nb & 1][wave];
#pragma unroll
        for (int e = 0; e < 4; ++e)   // accumulator row 4 jq + e of phase mb is d = 64 half + 4 (4 jq + e) + mb
        {
            float4v x = float4v{acc[0][0][nb][e], acc[0][1][nb][e], acc[0][2][nb][e], acc[0][3][nb][e]} * weight[0][nb];
            if constexpr (OWN) x += float4v{acc[1][0][nb][e], acc[1][1][nb][e], acc[1][2][nb][e], acc[1][3][nb][e]} * weight[1][nb];
            o[r16 * kHalfRow + jq * 4 + e] = x;
        }
        team_barrier();   // (two buffers: who writes block nb + 2 has passed the barrier of nb + 1, which follows the others' reads of nb)
#pragma unroll
        for (int it = 0; it < 16 / (2 * kTeam); ++it) {
            const int r = (it * kTeam + wave) * 2 + (lane >> 5), nn = nb * 16 + r;   // of the block, written by this lane
            const float m = __shfl(m_run[nb], r);
            if (nn < u.rows) {
                float4v v = float4v{0.f, 0.f, 0.f, 0.f};
                float l = 0.f;
#pragma unroll
                for (int w = 0; w < kTeam / 2; ++w) v += lds.o[nb & 1][2 * w + (d4 >> 4)][r * kHalfRow + (d4 & 15)];
#pragma unroll
                for (int w = 0; w < kTeam; ++w) l += lds.sum[w][nn];
                if (u.shares == 1) {
                    const float inv = 1.f / l;
                    const long long row = first_row + (nn >> u.group_log) * a.num_q_heads + (nn & ((1 << u.group_log) - 1));
                    *reinterpret_cast<uint2 *>(static_cast<__bf16 *>(a.out) + row * D + d4 * 4) = make_uint2(pack_bf16(v[0] * inv, v[1] * inv), pack_bf16(v[2] * inv, v[3] * inv));
                    if (a.lse && d4 == 0) a.lse[row] = (m + log2f(l)) * kLn2;
                } else {
                    const long long row = (long long)u.slot * a.rows_pad + nn;
                    *reinterpret_cast<float4v *>(a.part_o + row * D + d4 * 4) = v;
                    if (d4 == 0) *reinterpret_cast<float2 *>(a.part_ml + row * 2) = make_float2(m, l);
                }
            }
        }
    }
}

// How a unit's tiles are shared out: `per` tiles (whole pairs) to a workgroup, from the first one on; a short unit leaves the last ones without.
struct Shares {
    int per, count;
};
__device__ __forceinline__ Shares unit_shares(int tiles, int splits)
{
    Shares s;
    s.per = max(((tiles + splits - 1) / splits + 1) & ~1, 2);
    s.count = (tiles + s.per - 1) / s.per;
    return s;
}

template <int TEAM, bool FP8, bool TREE>
__global__ __launch_bounds__(64 * TEAM, 2) void attn_unit_kernel(AttnArgs a, int group_log, int splits, int heads, const int32_t *__restrict__ block_table,
                                                               const int32_t *__restrict__ kv_len, const int32_t *__restrict__ q_indptr,
                                                               const float *__restrict__ k_scale, const float *__restrict__ v_scale)
{
    // (what is read wave-uniformly comes in as no-alias arguments of its own, so that the reads are scalar loads)
    __shared__ UnitLds<TEAM> lds;
    Unit u;
    if ((int)blockIdx.x >= a.batch * a.num_kv_heads * splits) {
        // The workgroups behind the units' leave the plan in the workspace, as every call does that does not reuse one.  (A call that reuses it has
        // the same sizes, so it takes this path again and does not read it.)  They run beside the others (4 requests of 64 tokens 6.1 us, 64 of
        // 8..64 12.8, and 9.4 without).
        if (threadIdx.x >= 256) return;
        const int block = blockIdx.x - a.batch * a.num_kv_heads * splits;
        Place *places = reinterpret_cast<Place *>(&lds.p[0][0][0][0]);
        if (a.batch <= 64) plan_block<1>(a, heads, block, places);
        else if (a.batch <= 128) plan_block<2>(a, heads, block, places);
        else if (a.batch <= 256) plan_block<4>(a, heads, block, places);
        else plan_block<8>(a, heads, block, places);
        return;
    }
    const int unit = blockIdx.x / splits, share = blockIdx.x % splits;
    u.b = unit / a.num_kv_heads;
    u.g = unit % a.num_kv_heads;
    u.lane = threadIdx.x & 63;
    u.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u.group_log = group_log;
    const int32_t *table = block_table + (long long)u.b * a.max_blocks;
    u.L = kv_len[u.b];
    u.q0 = q_indptr[u.b];
    u.q_len = q_indptr[u.b + 1] - u.q0;
    const int tiles = (u.L + kTile - 1) / kTile;
    const Shares s = unit_shares(tiles, splits);
    u.shares = s.count;
    u.tile_lo = share * s.per;
    u.tiles = min(u.tile_lo + s.per, tiles);
    u.slot = blockIdx.x;
    u.rows = min(u.q_len, a.max_q_len) << group_log;   // (rows past the caller's bound are not computed)
    if ((u.tile_lo >= tiles) | (u.rows <= 0)) return;
    const int blocks = (u.rows + 15) >> 4;
    if (blocks <= 1) walk_unit<1, TEAM, FP8, TREE>(a, lds, u, table, k_scale, v_scale);
    else if (blocks == 2) walk_unit<2, TEAM, FP8, TREE>(a, lds, u, table, k_scale, v_scale);
    else if (blocks == 3) walk_unit<3, TEAM, FP8, TREE>(a, lds, u, table, k_scale, v_scale);
    else if (blocks == 4) walk_unit<4, TEAM, FP8, TREE>(a, lds, u, table, k_scale, v_scale);
    else walk_unit<5, TEAM, FP8, TREE>(a, lds, u, table, k_scale, v_scale);
}

// Workgroup (unit, slab of eight rows): adds the shares' partials in their order, 32 lanes to a row.
__global__ __launch_bounds__(256) void attn_unit_merge_kernel(AttnArgs a, int group_log, int splits)
{
    const int slabs = a.rows_pad / 8;
    const int unit = blockIdx.x / slabs, b = unit / a.num_kv_heads, g = unit % a.num_kv_heads;
    const int n = blockIdx.x % slabs * 8 + (threadIdx.x >> 5), d4 = threadIdx.x & 31;
    const int L = a.kv_len[b], q0 = a.q_indptr[b], q1 = a.q_indptr[b + 1];
    const Shares s = unit_shares((L + kTile - 1) / kTile, splits);
    if ((s.count == 1) | (n >= min(q1 - q0, a.max_q_len) << group_log)) return;
    const long long first = (long long)unit * splits * a.rows_pad + n;
    float2 ml[kMaxShares];
    constexpr int CHUNK = 8;
    float4v o[CHUNK];
    auto load = [&](int c) __attribute__((always_inline)) {   // (past the last share the first one's again)
#pragma unroll
        for (int i = 0; i < CHUNK; ++i)
            o[i] = *reinterpret_cast<const float4v *>(a.part_o + (first + (long long)(c + i < s.count ? c + i : 0) * a.rows_pad) * D + d4 * 4);
    };
#pragma unroll
    for (int i = 0; i < kMaxShares; ++i)
        ml[i] = *reinterpret_cast<const float2 *>(a.part_ml + (first + (long long)(i < s.count ? i : 0) * a.rows_pad) * 2);
    load(0);   // (all on their way at once)
    float m = ml[0].x;
#pragma unroll
    for (int i = 1; i < kMaxShares; ++i) m = fmaxf(m, ml[i].x);
    float l = 0.f;
    float4v v = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < kMaxShares; c += CHUNK) {
        if (c) {
            if (c >= s.count) break;
            load(c);
        }
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            const float w = c + i < s.count ? __builtin_amdgcn_exp2f(ml[c + i].x - m) : 0.f;   // a share without visible tokens has l = 0
            l += ml[c + i].y * w;
            v += o[i] * w;
        }
    }
    const float inv = 1.f / l;
    const long long row = (long long)q0 * a.num_q_heads + ((long long)g << group_log) + (n >> group_log) * a.num_q_heads + (n & ((1 << group_log) - 1));
    *reinterpret_cast<uint2 *>(static_cast<__bf16 *>(a.out) + row * D + d4 * 4) = make_uint2(pack_bf16(v[0] * inv, v[1] * inv), pack_bf16(v[2] * inv, v[3] * inv));
    if (a.lse && d4 == 0) a.lse[row] = (m + log2f(l)) * kLn2;
}

template <int TEAM>
void launch(const AttnArgs &a, int group_log, int splits, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1)
{
    const bool fp8 = a.kv_dtype == SS_FP8_E4M3, tree = a.tree_mask != nullptr;
    const auto kernel = fp8 ? (tree ? attn_unit_kernel<TEAM, true, true> : attn_unit_kernel<TEAM, true, false>)
                            : (tree ? attn_unit_kernel<TEAM, false, true> : attn_unit_kernel<TEAM, false, false>);
    const int heads = plan_heads(a), plan_groups = a.reuse_plan ? 0 : a.batch * (a.num_kv_heads / heads);
    hipExtLaunchKernelGGL(kernel, dim3((unsigned)(a.batch * a.num_kv_heads * splits + plan_groups)), dim3(64 * TEAM), 0, stream, ev0, ev1, 0, a, group_log,
                          splits, heads, a.block_table, a.kv_len, a.q_indptr, a.k_scale, a.v_scale);
}

}  // namespace

// Batches whose plan takes a kernel in front are left to the streaming kernels; the rule itself is in unit_rule.h.
AttnUnitChoice attn_unit_choose(const AttnArgs &a)
{
    const long long units = (long long)a.batch * a.num_kv_heads;
    const int cus = a.launch_waves / kWavesPerWg, rows = a.max_q_len * (a.num_q_heads / a.num_kv_heads);
    if (!a.default_waves || rows > 16 * kMaxRowBlocks || plan_laid_out(a) || units > kUnitsPerCu * cus) return {0, 0};
    return attn_unit_rule(units, a.max_blocks, rows, a.kv_dtype == SS_FP8_E4M3, cus);
}

int32_t attn_unit_launch(const AttnArgs &a, const AttnUnitChoice &choice, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1)
{
    const int splits = choice.splits;
    int group_log = 0;
    while (a.num_kv_heads << group_log < a.num_q_heads) ++group_log;
    if (choice.team == 8) launch<8>(a, group_log, splits, stream, ev0, ev1);
    else launch<4>(a, group_log, splits, stream, ev0, ev1);
    SS_HIP_CHECK(hipGetLastError(), "launch attn_unit_kernel");
    if (splits > 1) {
        hipLaunchKernelGGL(attn_unit_merge_kernel, dim3((unsigned)(a.batch * a.num_kv_heads * (a.rows_pad / 8))), dim3(256), 0, stream, a, group_log, splits);
        SS_HIP_CHECK(hipGetLastError(), "launch attn_unit_merge_kernel");
    }
    return SS_OK;
}

}  // namespace ss
