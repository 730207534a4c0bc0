// Streaming and merge kernels of the matrix-core verify attention, and their launchers, as templates.
// Included by one translation unit per head grouping (attn_mfma_g1.hip ...), so that the many
// instances compile in parallel; attn_mfma.hip holds the plan kernel and the dispatch.
//
// Work decomposition.  The KV cache of one (request, KV head) pair ("unit") is a run of
// 16-token tiles, one per cache block, taken two at a time ("pair").  All pairs of all units form one flat
// sequence (unit major).  A plan kernel writes that sequence out as a flat list of tile addresses (physical
// block * kv heads + kv head) and cuts it into contiguous spans of equal cost (opening a unit costs as much as
// some pairs), so the load is balanced whatever the mix of context lengths, and the load side of the
// kernel is a plain linear walk that never stops at a unit boundary.  A span may cover the tail
// of one unit, several whole units and the head of another; for every unit it touches there is
// one partial result (softmax reference, sum, unnormalised output).
//
// Whose a span is (choose_spans says, from the batch's lengths):
//
// A wavefront's, handed over: units of one or two row blocks on a full chip, or many of them.  The four wavefronts of a workgroup, whose
// spans are consecutive, hand the partials of a shared unit from right to left through LDS and combine them by their log-sum-exp; a unit that
// lies inside one workgroup's spans is normalised, rounded and written by that workgroup.
//
// A workgroup's, whose wavefronts are a team and take its pairs in turn (every fourth), so that they reach the
// end of a unit together and add their results block by block through LDS.  One partial per workgroup instead of four: with five row
// blocks a partial is 40 KB (52 MB of them and as much read again by the merge for 281 MB of keys and values, 32 requests of 256..4096
// with trees of 8..16 nodes; the call 76.5 us with a span per wavefront, 69 with teams).  On a chip that is not full the team ends
// sooner than a chain of hand-overs (one request of 8000 tokens 28.9 us and 23.9).
//
// A wavefront's by itself: many units of three row blocks and more, where opening and ending each of them with all four wavefronts would
// be most of a team's time (256 requests of 48 tokens over 8 KV heads, five row blocks, e4m3: 95 us and 55).
//
// In the kernels for three row blocks and more the requests are laid out by row blocks, and each run of units is walked by the code for
// its own number of them (see the plan kernel).
//
// What is left (a unit that crosses spans that are not combined) goes to device memory as a partial in slot
// `workgroup + unit` (`wavefront + unit` for wavefronts by themselves; unique along the sequence), and a last
// kernel merges those partials in span order and writes the rounded output.
//
// Per pair, with rows = (k+1) * (query heads per KV head) padded to a multiple of 16:
//   S^T[token][row] = K[token][:] . Q[row][:]   v_mfma_f32_16x16x32_bf16, each K tile as A operand
//   online softmax on S^T in registers (a row's 16 scores of a tile sit in 4 lanes x 4 registers)
//   O^T[d][row]    += V[token][d] * P[row][token]   v_mfma_f32_16x16x32_bf16 over both tiles' tokens, V as A
//                     operand.  Which token stands at which place of the contraction is free as long as both operands
//                     agree: lane group jq brings tokens 4 jq .. 4 jq + 3 of the first tile and of the second, so that P
//                     is taken straight from the two S^T accumulators.
// Both K and V are read from HBM directly in operand layout with 16-byte loads: for K a lane
// holds 8 consecutive d of one token; for V a lane holds d = 8*i .. 8*i+7 of four tokens of each tile and
// the eight M-blocks of O^T are the eight interleaved d-phases, so no transpose through LDS is
// needed (only a 16-bit pack per operand register).
//
// Why pairs: contracting over 32 tokens the output product runs at the full matrix rate (the 16-token shape takes the
// same 16 cycles for half of the work), and matrix and vector instructions of a wavefront hardly overlap on this
// chip (16 cycles and 5 cycles take 18.9 together), so every matrix instruction less is time.
//
// Why the code is written to be small (one copy of a unit's beginning and end outside the ring, which is rotated in
// registers instead): the instances took up to 150 KB of code with those inlined into every step of an unrolled ring and its
// epilogue, more than the 64 KB instruction cache that two compute units share; now 14 to 28 KB per number of row blocks.
//
// Measured, a whole call: 96 requests of 512..8192 tokens, e4m3, 64 heads over 8, depth 2..8: 305 us as single tiles with 16-token output
// products, 247 as pairs, 221 in teams by classes; 32 requests of 256..4096, trees of 8..16 nodes, 32 heads over 8: 98 / 76.5 / 69;
// 128 requests of 128..16384, depth 0..8, 32 heads over 8: 292 / 291 / 278; 64 requests of 256..4096 at depth 4 (bound by memory): 108.4 /
// 107.2 / 106.1; four requests of 40..600: 26.0 / 20.8 / 18.4.
#pragma once

#include <type_traits>

#include <hip/hip_ext.h>

#include "common.h"
#include "span_cuts.h"
#include "tree_window.h"

namespace ss {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));

constexpr int D = kMfmaHeadDim;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kSlack = 8.0f;       // log2 headroom of the lagging softmax reference
constexpr float kNoMax = -1.0e30f;   // reference before any score was seen (finite, so that -inf - ref stays -inf)
constexpr int kMaxFlagPolls = 1 << 23;   // polls of a neighbour's deposit flag before giving up (each at least 128 cycles)
constexpr int kPartRowStride = 33;   // float4 per staged partial row in LDS (32 of data + 1 of padding)
constexpr int kBlockStride = 16 * kPartRowStride;   // float4 from one staged 16-row block to the next (more than a pair of e4m3 key tiles takes)
template <int NB>
constexpr bool kQueriesInLds = NB >= 4;        // for many row blocks the registers are needed for the accumulators

// ---------------------------------------------------------------------------------------------
// streaming kernel
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t pack_hi16(uint32_t lo_src, uint32_t hi_src)
{
    // (hi_src & 0xffff0000) | (lo_src >> 16): upper halves of two words
    return __builtin_amdgcn_perm(hi_src, lo_src, 0x07060302u);
}
__device__ __forceinline__ uint32_t pack_lo16(uint32_t lo_src, uint32_t hi_src)
{
    return __builtin_amdgcn_perm(hi_src, lo_src, 0x05040100u);
}

// Two e4m3 bytes (the lower or upper half of a word) -> two bf16 (exact: e4m3 has 4 significant bits; the scale is 1)
template <bool HI>
__device__ __forceinline__ uint32_t fp8x2_to_bf16x2(uint32_t w)
{
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HI));
}
__device__ __forceinline__ uint4 fp8x8_to_bf16x8(uint32_t w0, uint32_t w1)
{
    return make_uint4(fp8x2_to_bf16x2<false>(w0), fp8x2_to_bf16x2<true>(w0), fp8x2_to_bf16x2<false>(w1), fp8x2_to_bf16x2<true>(w1));
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Output accumulators live in the accumulator registers (the matrix instructions are selected in that form
// once a kernel needs more than 256 registers).  A value that ordinary vector arithmetic produced -- the zero
// of a new unit, a rescaled or merged accumulator -- is handed over through this empty statement, so that
// every value flowing into the tile loop comes from an accumulator register; otherwise the compiler keeps the
// loop-carried accumulators in vector registers and moves all of them to the accumulator file and back on
// every tile.
__device__ __forceinline__ void to_accumulator_file(float4v &c) { asm volatile("" : "+a"(c)); }
// The opposite direction for the rare rescale: the move is written out, so that it stays inside the rarely taken
// branch (left to the compiler, the moves of all accumulators to vector registers can end up in front of the
// branch, on every tile).  The compiler does not look into the statement: the caller leaves the wait states
// between the last matrix instruction that wrote the register and this read (accumulator_read_guard).
__device__ __forceinline__ float from_accumulator_file(float x)
{
    float r;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(x));
    return r;
}
__device__ __forceinline__ void accumulator_read_guard() { asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory"); }

template <bool FP8>
struct TileRegs {
    // bf16: k[ks] = 8 bf16 of token (lane&15) at d = 32*ks + 8*(lane>>4)
    // fp8 : k[kk] = 16 bytes of token (lane&15) at d = 64*kk + 16*(lane>>4)   (kk = 0,1)
    // STAGE: k[i] = the tile's bytes 1024 i + 16 lane .. + 15: whole kilobytes in the order of memory, not yet an operand (see stage_keys)
    u32x4 k[FP8 ? 2 : 4];
    // bf16: v[e] = 8 bf16 of token 4*(lane>>4)+e at d = 8*(lane&15)
    // fp8 : v[e] = 8 bytes of the same
    typename std::conditional<FP8, u32x2, u32x4>::type v[4];
    float ks, vs;  // block scales (fp8), 1 otherwise
};
template <bool FP8>
struct PairRegs {
    TileRegs<FP8> t[2];
};

// All loads of one tile are vector loads issued back to back, so one counter orders them and the
// consumer can wait for exactly this tile.  `addr` = physical block * kv heads + kv head indexes
// both the 4 KB (2 KB for e4m3) tile and its scale.  Buffer loads through a descriptor of exactly the tile: a
// load with `live` false (past the span's end) has a descriptor of no bytes, returns zeros and moves nothing, so the ring's
// last steps need no code of their own.  KV tiles are read exactly once per call: non-temporal loads keep them from
// displacing what is reused (partials, queries, the pair list) in the caches.
// The keys of both tiles come first: they are used first.
constexpr int kNonTemporal = 2;
enum { kKeys = 1, kValues = 2 };   // what of a pair
template <bool FP8, bool STAGE, int WHAT>
__device__ __forceinline__ void load_pair_tiles(PairRegs<FP8> &p, const AttnArgs &a, const float *__restrict__ k_scale,
                                                const float *__restrict__ v_scale, int2 addr, bool live, int lane)
{
    constexpr int ES = FP8 ? 1 : 2, BYTES = kTile * D * ES;
    const int bytes = live ? BYTES : 0;
    const int ko = STAGE ? lane * 16 : (lane & 15) * (D * ES) + (lane >> 4) * 16, vo = (lane >> 4) * (4 * D * ES) + (lane & 15) * (8 * ES);
    if constexpr (WHAT & kKeys) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t blk = (int64_t)(h ? addr.y : addr.x) * BYTES;
            const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(static_cast<const char *>(a.k)) + blk, 0, bytes, 0x00020000);
#pragma unroll
            for (int i = 0; i < (FP8 ? 2 : 4); ++i)
                p.t[h].k[i] = __builtin_amdgcn_raw_buffer_load_b128(kr, ko + i * (STAGE ? 1024 : 64), 0, kNonTemporal);
        }
    }
    if constexpr (WHAT & kValues) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ad = h ? addr.y : addr.x;
            const int64_t blk = (int64_t)ad * BYTES;
            const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(static_cast<const char *>(a.v)) + blk, 0, bytes, 0x00020000);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (FP8)
                    p.t[h].v[e] = __builtin_amdgcn_raw_buffer_load_b64(vr, vo + e * (D * ES), 0, kNonTemporal);
                else
                    p.t[h].v[e] = __builtin_amdgcn_raw_buffer_load_b128(vr, vo + e * (D * ES), 0, kNonTemporal);
            }
            if constexpr (FP8) {
                p.t[h].ks = k_scale[ad];   // wave-uniform: scalar loads
                p.t[h].vs = v_scale[ad];
            } else {
                p.t[h].ks = 1.f;
                p.t[h].vs = 1.f;
            }
        }
    }
}

// A workgroup's LDS.  BLOCKS: the most row blocks of the kernel.
//   q    query operands, in operand order, one 1 KB line per row block and k-step of each wavefront (kQueriesInLds)
//   o    one 16-row block of a partial per wavefront, rows 33 float4 apart (the odd stride spreads the rows over the banks); teams
//        exchange blocks through it: two buffers, one barrier per block.  Between the ends of units, the keys of a pair
//   ml   references and sums of the rows
//   dep  CHAIN: the deposits.  The wavefronts of a workgroup own consecutive spans, so a unit that runs on from one span into the next
//        is combined inside the workgroup: the right-hand wave leaves the result of its part in its deposit slot, the left-hand one
//        folds it into its own.  Only what crosses a workgroup's edge goes to memory as a partial; a unit that lies inside one
//        workgroup is finished here.
template <int BLOCKS>
struct StreamLds {
    static constexpr bool CHAIN = BLOCKS <= kChainRowBlocks;
    uint4 q[kQueriesInLds<BLOCKS> ? kWavesPerWg * BLOCKS * 4 * 64 : 1];
    float4v o[2 * kWavesPerWg][kBlockStride];
    float2 ml[kWavesPerWg][BLOCKS * 16];
    float4v dep_o[CHAIN ? kWavesPerWg : 1][CHAIN ? BLOCKS * 16 * kPartRowStride : 1];
    float2 dep_ml[CHAIN ? kWavesPerWg : 1][CHAIN ? BLOCKS * 16 : 1];
    int dep_flag[kWavesPerWg];   // 0 nothing yet; 1 deposited; 2 deposited and it reaches the unit's last tile
};

// Where a run (units of one class inside a span) starts, and what the wave's first loads need.
struct Run {
    int p, g, b, n;       // place in the layout, KV head, request, pairs of the unit
    int unit_x;           // flat index of the unit's first pair
    int x0, x1;           // the run, flat
    int L, q0, q1;        // kv_len and query rows of the request
    int free_block;       // which of the wavefront's two block buffers in LDS nobody reads
    int2 addr[kDescPairs];   // of the wave's first pairs
};

// NB      16-row blocks of query rows the code is compiled for
// BLOCKS  those of the kernel
// TREE    the new tokens of a request form a draft tree: a row's visibility among them comes from its
//         mask word instead of the chain's "tokens up to my own"
// STAGE   the keys are read in the order of memory and turned in LDS (see stage_keys)
// CHAIN   wavefronts' spans, handed over; else `team` says whether the run is the workgroup's or the wavefront's own
template <int G, int NB, int BLOCKS, bool FP8, bool TREE, bool CHAIN, bool STAGE>
__device__ __forceinline__ void walk(const AttnArgs &a, StreamLds<BLOCKS> &lds, Run &run, bool team, const int2 *__restrict__ pair_addr,
                                     const AttnReq *__restrict__ req, const float *__restrict__ k_scale,
                                     const float *__restrict__ v_scale)
{
    constexpr bool QLDS = kQueriesInLds<NB>;
    const int lane = threadIdx.x & 63;
    const int wslot = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, jq = lane >> 4;
    uint4 *qs = lds.q + (QLDS ? wslot * BLOCKS * 4 * 64 + lane : 0);   // (not NB: wavefronts may be at different classes)
    auto &o_lds = lds.o;
    auto &ml_lds = lds.ml;
    auto &dep_o = lds.dep_o;
    auto &dep_ml = lds.dep_ml;
    auto &dep_flag = lds.dep_flag;
    int p = run.p, b = run.b, g = run.g, nb_tiles = run.n, unit_x = run.unit_x;
    const int x0 = run.x0, x1 = run.x1;
    int meta_b = b, meta_L = run.L, meta_q0 = run.q0, meta_q1 = run.q1, meta_nbt = nb_tiles;   // of the next unit to open

    // SINGLE: with many row blocks a step is longer than a read's latency, and one buffer that is refilled as soon as its
    // operands have been copied out keeps a pair in flight all the time, where two spill (32 requests of 256..4096, trees
    // of 8..16 nodes: 80 us a call with two buffers, 75 with one; with three row blocks both are level).
    constexpr bool SINGLE = NB >= 4;
    // ---- state of the unit being computed ----
    // A team takes the pairs of its span in turn: wavefront w every fourth from the w-th on, whatever units they belong to.
    const int step_log = team ? kWavesPerWgLog : 0, stride = 1 << step_log;
    int pos = x0 + (team ? wslot : 0);   // flat index of this wave's next pair
    int seg_x0 = x0, seg_x1 = x0;     // the current segment (the part of the unit inside the span), flat
    int seg_left = 0;                 // this wave's pairs of it that are left
    int L = 0, q0 = 0, q_len = 0, rows = 0, nbu = 0;   // nbu: 16-row blocks the unit really has (for its partial)
    bf16x8 qreg[QLDS ? 1 : NB][4];    // Q as B operand: lane holds row 16*nb + r16, 8 consecutive d per k-step
    int lim[TREE ? 1 : NB];           // chain: last visible cache position of this lane's row in block nb
    uint32_t newmask[TREE ? NB : 1];  // tree: which new tokens of the request the lane's row attends
    int ctx = 0;                      // cache positions before the unit's new tokens
    float m_run[NB], l_run[NB];
    float4v acc[8][NB];
    const float sc2 = a.sm_scale * kLog2e;
    // The keys' place in LDS: the wavefront's block buffer that nobody reads.  At a team's unit end the others may still be reading this
    // wavefront's last block when it goes on; its buffer before that one has been read by all.
    u32x4 *stage = STAGE ? reinterpret_cast<u32x4 *>(o_lds[run.free_block * kWavesPerWg + wslot]) : nullptr;

    u32x4 qw[NB][4];   // a unit's queries on their way (between begin_unit_issue and begin_unit_wait)
    // (the metadata of the unit after the current one is fetched a unit ahead)
    auto begin_unit_issue = [&]() __attribute__((always_inline)) {
        b = meta_b;
        L = meta_L;
        q0 = meta_q0;
        q_len = meta_q1 - meta_q0;
        const int q_here = window_q_len(q_len, a.q_lo, a.q_win);   // query tokens of this pass's window
        nb_tiles = meta_nbt;
        rows = q_here * G;
        nbu = (rows + 15) >> 4;
        ctx = L - q_len;
        {
            const int np = (g + 1 == a.num_kv_heads) ? p + 1 : p;   // place of the next unit's request
            if (np != p && np < a.batch) {
                const AttnReq r = req[np];
                meta_b = r.b;
                meta_L = r.L;
                meta_q0 = r.q0;
                meta_q1 = r.q1;
                meta_nbt = r.n;
            }
        }
        seg_x1 = unit_x + nb_tiles < x1 ? unit_x + nb_tiles : x1;
        seg_left = pos < seg_x1 ? (seg_x1 - pos + stride - 1) >> step_log : 0;
        // All query loads go out before any of them is waited for: buffer loads over the request's rows, whose
        // offset is out of range (zeros) for a row the unit does not have, so there is no branch between them.  (Under a branch
        // per block the LDS instances waited for every block's loads in turn, 7 us at the start of a span.)
        const long long q_row = (long long)a.num_q_heads * D * 2;   // bytes from one query token to the next
        const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char *>(static_cast<const char *>(a.q)) + (q0 * q_row + (long long)g * (G * D * 2)), 0, (int)(q_len * q_row),
            0x00020000);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = nb * 16 + r16;
            const bool ok = n < rows;
            const int qi = a.q_lo + n / G, hh = n % G;   // query token within the request, head within the group
            if constexpr (TREE)   // padding rows see every new token: harmless, and no row is empty
                newmask[nb] = a.tree_mask[q0 + (ok ? qi : 0)];
            else
                lim[nb] = ok ? L - q_len + qi : L - 1;
            const int off = ok ? qi * (int)q_row + hh * (D * 2) : 0x7fffff00;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int d0 = FP8 ? ((ks >> 1) * 64 + jq * 16 + (ks & 1) * 8) : (ks * 32 + jq * 8);
                qw[nb][ks] = __builtin_amdgcn_raw_buffer_load_b128(qr, off + d0 * 2, 0, 0);
            }
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            m_run[nb] = kNoMax;
            l_run[nb] = 0.f;
#pragma unroll
            for (int mb = 0; mb < 8; ++mb) {
                acc[mb][nb] = float4v{0.f, 0.f, 0.f, 0.f};
                to_accumulator_file(acc[mb][nb]);
            }
        }
    };
    // Have the queries arrive here, inside the rarely taken branch, so that the steady-state path
    // never carries a pending load of them.
    auto begin_unit_wait = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if constexpr (QLDS) {
                    qs[(nb * 4 + ks) * 64] = __builtin_bit_cast(uint4, qw[nb][ks]);
                } else {
                    qreg[nb][ks] = __builtin_bit_cast(bf16x8, qw[nb][ks]);
                    asm volatile("" : "+v"(qreg[nb][ks]));
                }
            }
        if constexpr (TREE) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if (nb * 16 + r16 >= rows) newmask[nb] = (2u << (q_len - 1)) - 1u;
                asm volatile("" : "+v"(newmask[nb]));
            }
        }
    };

    // The unit's row nn in the output, counted from the unit's first (in 32 bits: with 64-bit row numbers the addresses of a
    // block's rows took longer than its values), and four of a finished row's values: normalised, rounded to bf16 (nearest even), 256
    // bytes per half-wavefront.
    auto row_of = [&](int nn) __attribute__((always_inline)) { return nn / G * a.num_q_heads + nn % G; };
    auto first_row = [&]() __attribute__((always_inline)) { return (long long)(q0 + a.q_lo) * a.num_q_heads + g * G; };
    auto write_row = [&](__bf16 *out, int row, float4v v, float inv) __attribute__((always_inline)) {
        const float2v lo2 = {v[0] * inv, v[1] * inv}, hi2 = {v[2] * inv, v[3] * inv};
        uint2 pk;
        pk.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo2, bf16x2));
        pk.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi2, bf16x2));
        *reinterpret_cast<uint2 *>(out + (uint32_t)(row * D + (lane & 31) * 4)) = pk;
    };

    // The end of a segment without a hand-over, block by block through LDS: as finished output if the segment is the `whole` unit, else
    // as a partial.  A team's four wavefronts bring their results to a common reference and add them, each wavefront
    // adding (in a fixed order) and writing four of a block's sixteen rows.  The barriers wait for LDS only, not for the pairs in
    // flight.  Two block buffers: a wavefront that writes block nb + 2 has passed the barrier of block nb + 1, which the others
    // reach after reading block nb.  A wavefront by itself takes the same way with its own results only and all sixteen rows: LDS
    // serves a wave's requests in order.
    auto team_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
        if (team) __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto end_blocks = [&](bool whole, const float (&lsum)[NB]) __attribute__((always_inline)) {
        if (nbu == 0) return;   // (a request without rows in this window)
        // (a copy that the compiler does not see through: what follows from it alone, the places of all rows, would be worked out
        // at the start of the kernel and kept, 0.5 us of a short call)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        float m_all[NB], l_all[NB];
        if (team) {
            if (jq == 0) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) ml_lds[wslot][nb * 16 + r16] = make_float2(m_run[nb], lsum[nb]);
            }
            team_barrier();
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float2 ml[kWavesPerWg];
#pragma unroll
                for (int w = 0; w < kWavesPerWg; ++w) ml[w] = ml_lds[w][nb * 16 + r16];
                m_all[nb] = fmaxf(fmaxf(ml[0].x, ml[1].x), fmaxf(ml[2].x, ml[3].x));
                l_all[nb] = 0.f;
#pragma unroll
                for (int w = 0; w < kWavesPerWg; ++w) l_all[nb] += ml[w].y * __builtin_amdgcn_exp2f(ml[w].x - m_all[nb]);
            }
        } else {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                m_all[nb] = m_run[nb];
                l_all[nb] = lsum[nb];
            }
        }
        auto deposit = [&](int nb) __attribute__((always_inline)) {
            // (0 for a wave without a pair of this segment.  A wavefront by itself normalises finished rows here: a lane's accumulators
            // are of one row, and behind LDS every row's factor would have to come from another lane.)
            float mine = __builtin_amdgcn_exp2f(m_run[nb] - m_all[nb]);
            if (!team) mine = whole ? 1.f / l_all[nb] : 1.f;
            float4v *ol = o_lds[(nb & 1) * kWavesPerWg + wslot];
#pragma unroll
            for (int e = 0; e < 4; ++e) {   // accumulator row 4*jq+e of M-block mb is d = 8*(4*jq+e) + mb
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float4v x;
#pragma unroll
                    for (int c = 0; c < 4; ++c) x[c] = from_accumulator_file(acc[4 * h + c][nb][e]) * mine;
                    ol[r16 * kPartRowStride + jq * 8 + e * 2 + h] = x;
                }
            }
        };
        const long long slot = (long long)(team ? (int)blockIdx.x : (int)blockIdx.x * kWavesPerWg + wslot) + (long long)p * a.num_kv_heads + g;
        float *po = a.part_o + slot * a.rows_pad * D;
        float2 *pml = reinterpret_cast<float2 *>(a.part_ml) + slot * a.rows_pad;
        __bf16 *out = static_cast<__bf16 *>(a.out) + first_row() * D;
        float *lse = a.lse ? a.lse + first_row() : nullptr;
        // The eight reads of a block: two rows of each of the four wavefronts' blocks, or all sixteen rows of the own one.
        const float4v *from0 = o_lds[team ? 0 : wslot] + ((team ? wslot * 4 : 0) + (ln >> 5)) * kPartRowStride + (ln & 31);
        deposit(0);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if (nb < nbu) {
                team_barrier();
                float4v v[2][kWavesPerWg];
                auto read = [&](int from_one_to_next) __attribute__((always_inline)) {
#pragma unroll
                    for (int it = 0; it < 2; ++it)
#pragma unroll
                        for (int w = 0; w < kWavesPerWg; ++w)
                            v[it][w] = from0[(nb & 1) * (kWavesPerWg * kBlockStride) + w * from_one_to_next + it * 2 * kPartRowStride];
                };
                if (team) read(kBlockStride);   // (constant offsets cost no address arithmetic)
                else read(4 * kPartRowStride);
                if (nb + 1 < NB) deposit(nb + 1 < NB ? nb + 1 : 0);   // (under the latency of the reads)
                const int first = team ? wslot * 4 : 0, rows_here = team ? 4 : 16;   // of the block, written by this wavefront
                const bool mine = jq == 0 && (unsigned)(r16 - first) < (unsigned)rows_here && nb * 16 + r16 < rows;   // lanes that hold their (m, l)
                float inv = 1.f;
                if (whole) {
                    if (team) inv = 1.f / l_all[nb];
                    if (mine && lse) lse[row_of(nb * 16 + r16)] = (m_all[nb] + log2f(l_all[nb])) * kLn2;
                } else if (mine) {
                    pml[nb * 16 + r16] = make_float2(m_all[nb], l_all[nb]);
                }
                auto write = [&](int row, const float4v &x) __attribute__((always_inline)) {
                    const int nn = nb * 16 + row;
                    if (whole) {
                        const float iv = team ? __shfl(inv, row) : 1.f;
                        if (nn < rows) write_row(out, row_of(nn), x, iv);
                    } else if (nn < rows) {
                        *reinterpret_cast<float4v *>(po + nn * D + (ln & 31) * 4) = x;
                    }
                };
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int row = first + it * 2 + (ln >> 5);
                    if (team) v[it][0] = ((v[it][0] + v[it][1]) + v[it][2]) + v[it][3];
                    write(row, v[it][0]);
                    if (!team) {
#pragma unroll
                        for (int w = 1; w < kWavesPerWg; ++w) write(row + 4 * w, v[it][w]);
                    }
                }
            }
        }
    };

    // A segment (the part of a unit that lies in this span) has ended: `starts` / `ends` say whether it holds
    // the unit's first / last pair.
    auto end_unit = [&](bool starts, bool ends) __attribute__((always_inline)) {
        // The accumulators were last written by MFMAs in another basic block: give them the wait
        // states a read needs before anything below touches them.
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
        float lsum[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float l = l_run[nb];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            lsum[nb] = l;
        }
        if constexpr (!CHAIN) {
            end_blocks(starts && ends, lsum);
            return;
        }
        bool to_end = ends;   // does the result held here reach the unit's last tile?
        if constexpr (CHAIN) {
            if (!ends && wslot + 1 < kWavesPerWg) {
                // The unit runs on into the right-hand neighbour's span, where it is that wave's first
                // segment: finished long ago unless the spans are very short.  Fold its result into mine
                // (mine first: a fixed order, so the bits do not depend on timing).
                // (relaxed LDS accesses: a volatile or acquiring load would first wait for every tile in flight)
                // The wait is bounded (about a second): the neighbour is a wave of the same workgroup and reaches its
                // deposit without waiting for anything itself, so the bound is never met; if it ever were, the unit's
                // rows come out as NaN instead of the kernel hanging.
                int f = __hip_atomic_load(&dep_flag[wslot + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                for (int polls = 0; f == 0 && polls < kMaxFlagPolls; ++polls) {
                    __builtin_amdgcn_s_sleep(2);
                    f = __hip_atomic_load(&dep_flag[wslot + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                if (f == 0) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) lsum[nb] = __builtin_nanf("");
                }
                to_end = f == 2;
                // (the deposit is read after the flag: the hardware serves a wave's LDS requests in order; this
                // keeps the compiler from moving the reads ahead of the loop, at no instruction)
                asm volatile("" ::: "memory");
                const float4v *dq = dep_o[wslot + 1];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    if (nb < nbu) {
                        const float2 ml2 = dep_ml[wslot + 1][nb * 16 + r16];
                        const float m_new = fmaxf(m_run[nb], ml2.x);
                        const float wa = exp2f(m_run[nb] - m_new), wb = exp2f(ml2.x - m_new);
                        lsum[nb] = lsum[nb] * wa + ml2.y * wb;
                        m_run[nb] = m_new;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float4v lo = dq[(nb * 16 + r16) * kPartRowStride + jq * 8 + e * 2];
                            const float4v hi = dq[(nb * 16 + r16) * kPartRowStride + jq * 8 + e * 2 + 1];
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                acc[c][nb][e] = acc[c][nb][e] * wa + lo[c] * wb;
                                acc[4 + c][nb][e] = acc[4 + c][nb][e] * wa + hi[c] * wb;
                            }
                        }
                    }
                }
            }
            if (!starts && wslot > 0) {
                // The unit began in the left-hand neighbour's span: leave the result for it.
                float4v *dq = dep_o[wslot];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    if (nb < nbu) {
                        if (jq == 0) dep_ml[wslot][nb * 16 + r16] = make_float2(m_run[nb], lsum[nb]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float4v lo = {acc[0][nb][e], acc[1][nb][e], acc[2][nb][e], acc[3][nb][e]};
                            const float4v hi = {acc[4][nb][e], acc[5][nb][e], acc[6][nb][e], acc[7][nb][e]};
                            dq[(nb * 16 + r16) * kPartRowStride + jq * 8 + e * 2] = lo;
                            dq[(nb * 16 + r16) * kPartRowStride + jq * 8 + e * 2 + 1] = hi;
                        }
                    }
                }
                // The slot's contents are in LDS before the flag says so: LDS serves a wave's requests in order,
                // and the wait below covers LDS only (a release fence would also wait for the tiles in flight).
                asm volatile("" ::: "memory");        // (the compiler keeps the deposit's stores above this line)
                __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
                __builtin_amdgcn_wave_barrier();
                asm volatile("" ::: "memory");
                if (lane == 0) __hip_atomic_store(&dep_flag[wslot], to_end ? 2 : 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                return;
            }
        }
        // What is held here goes to memory: as the finished output if it covers the whole unit, else as a
        // partial in slot (workgroup, or wave without the hand-over) + unit, unique along the pair sequence.
        const bool whole = starts && to_end;
        const long long slot = (long long)blockIdx.x + (long long)p * a.num_kv_heads + g;
        float *po = a.part_o + slot * a.rows_pad * D;
        float *pml = a.part_ml + slot * a.rows_pad * 2;
        __bf16 *out = static_cast<__bf16 *>(a.out) + first_row() * D;
        float *lse = a.lse ? a.lse + first_row() : nullptr;
        // A lane holds 32 consecutive d of one row (d = 32*jq + 8*e + mb), in registers that are 16 bytes
        // apart in memory: written directly, every store would scatter 16-byte pieces over 64 cache lines.
        // The block goes through LDS instead and leaves as whole rows, two per store.
        int ln = lane;   // (as in end_blocks)
        asm volatile("" : "+v"(ln));
        float4v *ol = o_lds[wslot];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if (nb < nbu) {
                const int n = nb * 16 + r16;
                if (whole) {
                    if (jq == 0) ml_lds[wslot][r16] = make_float2(m_run[nb], lsum[nb]);
                } else if (n < rows && jq == 0) {
                    pml[n * 2 + 0] = m_run[nb];
                    pml[n * 2 + 1] = lsum[nb];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // accumulator row 4*jq+e of M-block mb is d = 8*(4*jq+e) + mb
                    const float4v lo = {acc[0][nb][e], acc[1][nb][e], acc[2][nb][e], acc[3][nb][e]};
                    const float4v hi = {acc[4][nb][e], acc[5][nb][e], acc[6][nb][e], acc[7][nb][e]};
                    ol[r16 * kPartRowStride + jq * 8 + e * 2] = lo;
                    ol[r16 * kPartRowStride + jq * 8 + e * 2 + 1] = hi;
                }
                __builtin_amdgcn_wave_barrier();
                // same wave, LDS keeps program order: no barrier.  All rows are read back first, in straight-line
                // code, so that the LDS latency is paid once and not in front of every store.
                float4v rowv[8];
                float2 rowml[8];
#pragma unroll
                for (int it = 0; it < 8; ++it) {
                    const int row = it * 2 + (ln >> 5);
                    rowv[it] = ol[row * kPartRowStride + (lane & 31)];
                    if (whole) rowml[it] = ml_lds[wslot][row];
                }
#pragma unroll
                for (int it = 0; it < 8; ++it) {
                    const int row = it * 2 + (ln >> 5), nn = nb * 16 + row;
                    const float4v v = rowv[it];
                    if (whole) {
                        const float2 ml = rowml[it];
                        if (nn < rows) {
                            write_row(out, row_of(nn), v, 1.f / ml.y);
                            if (lse && (lane & 31) == 0) lse[row_of(nn)] = (ml.x + log2f(ml.y)) * kLn2;
                        }
                    } else if (nn < rows) {
                        *reinterpret_cast<float4v *>(po + nn * D + (ln & 31) * 4) = v;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    };
    // (p, g) <- the unit after it (its metadata is already in meta_*)
    auto next_unit = [&]() __attribute__((always_inline)) {
        unit_x += nb_tiles;
        seg_x0 = unit_x;
        if (++g == a.num_kv_heads) {
            g = 0;
            ++p;
        }
    };

    // ---- load side: a linear walk over the span's pairs, the address of the next one read a step ahead ----
    int next_x = pos;                 // next pair to load
    int2 next_addr = run.addr[0];    // its addresses
    auto load_pair = [&](PairRegs<FP8> &t, int2 addr) __attribute__((always_inline)) {
        const bool live = next_x < x1;
        load_pair_tiles<FP8, STAGE, kKeys | kValues>(t, a, k_scale, v_scale, addr, live, lane);
        next_x += stride;
    };
    auto issue = [&](PairRegs<FP8> &t) __attribute__((always_inline)) {
        const int2 addr = next_addr;
        load_pair(t, addr);
        next_addr = pair_addr[next_x < x1 ? next_x : x1 - 1];
    };
    // in two halves, where the keys' registers are free before the values' (STAGE)
    auto issue_keys = [&](PairRegs<FP8> &t) __attribute__((always_inline)) {
        load_pair_tiles<FP8, STAGE, kKeys>(t, a, k_scale, v_scale, next_addr, next_x < x1, lane);
    };
    auto issue_values = [&](PairRegs<FP8> &t) __attribute__((always_inline)) {
        load_pair_tiles<FP8, STAGE, kValues>(t, a, k_scale, v_scale, next_addr, next_x < x1, lane);
        next_x += stride;
        next_addr = pair_addr[next_x < x1 ? next_x : x1 - 1];
    };

    // Keys as operands.  An operand register wants 16 bytes of sixteen tokens' rows in sixteen consecutive lanes, and reading memory
    // that way takes four times as long as reading whole lines (a compute unit 38 GB/s and 145 out of L2; the chip 6.0 and 7.1 TB/s out of
    // memory), with the wavefront standing still while its loads are accepted.  With STAGE the tiles are read in the order of memory and turned
    // here, through the wavefront's own place in LDS.  Rows stand one 16-byte word further apart than they are long, so that neither
    // side meets a bank twice.
    // Where it pays: e4m3 caches and batches that may be served by wavefronts' spans; the rule stands at launch_stream.  With fewer units the
    // round trip through LDS costs what the reads gain (20 requests 58.6 / 58.7, trees 58.0 / 59.2), with one or two row blocks more (159.1 / 160.5).
    // bf16 keys are twice the LDS traffic: 64 requests of 256..4096 105.5 / 106.6, 128 of 128..16384 276.4 / 277.3 at best.
    constexpr int KROW = (FP8 ? 8 : 16) + 1, KSEG = FP8 ? 8 : 16;   // 16-byte words of a row in LDS, in memory
    static_assert(!STAGE || 2 * 16 * KROW <= kBlockStride, "a pair's keys fit a block buffer");
    auto stage_keys = [&](const PairRegs<FP8> &t, u32x4 (&kw)[2][FP8 ? 2 : 4]) __attribute__((always_inline)) {
        u32x4 *to = stage + lane / KSEG * KROW + lane % KSEG;
        const u32x4 *from = stage + r16 * KROW + jq;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < (FP8 ? 2 : 4); ++i) to[h * 16 * KROW + i * (64 / KSEG) * KROW] = t.t[h].k[i];
        __builtin_amdgcn_wave_barrier();   // (LDS serves a wavefront's requests in order; this keeps the compiler to it)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < (FP8 ? 2 : 4); ++i) kw[h][i] = from[h * 16 * KROW + i * 4];
        __builtin_amdgcn_wave_barrier();
    };

    // One pair: S^T = K Q^T for both tiles and all row blocks, softmax, O^T += V^T P^T.  Row blocks beyond the
    // unit's rows hold zero queries; they are computed anyway and never stored (skipping them by wave-uniform branches was
    // measured again: the blocks' values then live across the branches, the compiler spills, and the spans are cut for
    // pairs of equal cost).  Three wave-uniform branches leave the straight line: the mask
    // selects (only pairs that reach into the request's new tokens), the clearing of V slots past the
    // end of the cache (only a cache's last pair) and the rare rescale.  The compiler
    // keeps the wait states between a matrix instruction and the first read of its result, also across
    // these branches; where the read is written out by hand (the rescale, from_accumulator_file) or
    // follows a scheduling barrier (the end of a unit), explicit wait states stand in front of it.
    // Once the scores are formed and the V operands packed, the pair's registers are free and (refill) the next
    // pair's loads go out into them, ahead of the softmax and the output product.
    auto compute = [&](PairRegs<FP8> &t, int ti, auto refill) __attribute__((always_inline)) {
        const int tok0 = ti * kPairTokens + jq * 4;   // first of this lane's four cache positions in the first tile
        const float kscale[2] = {sc2 * t.t[0].ks, sc2 * t.t[1].ks}, vscale[2] = {t.t[0].vs, t.t[1].vs};

        bf16x8 kop[2][4];
        auto widen_keys = [&](int h, const u32x4 *k) __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) kop[h][ks] = __builtin_bit_cast(bf16x8, fp8x8_to_bf16x8(k[ks >> 1][(ks & 1) * 2], k[ks >> 1][(ks & 1) * 2 + 1]));
        };
        u32x4 kw[2][FP8 ? 2 : 4];
        if constexpr (STAGE) {
            stage_keys(t, kw);
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if constexpr (FP8) {
                    widen_keys(h, t.t[h].k);
                } else {
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        u32x4 w = t.t[h].k[ks];
                        if constexpr (SINGLE) {   // a copy, so that the registers it came in are free for the refill
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                uint32_t x;
                                asm volatile("v_mov_b32 %0, %1" : "=v"(x) : "v"(w[c]));
                                w[c] = x;
                            }
                        }
                        kop[h][ks] = __builtin_bit_cast(bf16x8, w);
                    }
                }
            }
        }
        // V operand registers: vop[mb] = d-phase mb of tokens tok0 .. tok0+3 (words 0, 1) and tok0+16 .. tok0+19 (2, 3).
        uint32_t vop[8][4];
        auto pack_values = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
#pragma unroll
                for (int h = 0; h < 4; ++h) {   // word h of each token's 8 values holds d-phases 2h and 2h+1
                    uint32_t w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (FP8) {
                            const uint32_t src = (h < 2) ? t.t[t2].v[e].x : t.t[t2].v[e].y;   // two e4m3 bytes -> two bf16, exact
                            w[e] = (h & 1) ? fp8x2_to_bf16x2<true>(src) : fp8x2_to_bf16x2<false>(src);
                        } else {
                            w[e] = t.t[t2].v[e][h];
                        }
                    }
                    vop[2 * h][2 * t2] = pack_lo16(w[0], w[1]);
                    vop[2 * h][2 * t2 + 1] = pack_lo16(w[2], w[3]);
                    vop[2 * h + 1][2 * t2] = pack_hi16(w[0], w[1]);
                    vop[2 * h + 1][2 * t2 + 1] = pack_hi16(w[2], w[3]);
                }
            }
        };
        if constexpr (STAGE) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (decltype(refill)::value) issue_keys(t);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (SINGLE) {
            pack_values();
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (STAGE) issue_values(t);
            else issue(t);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (STAGE) {   // (e4m3)
#pragma unroll
            for (int h = 0; h < 2; ++h) widen_keys(h, kw[h]);
        }

        float4v s[NB][2];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) s[nb][0] = s[nb][1] = float4v{0.f, 0.f, 0.f, 0.f};
        {
            // Operands from LDS are requested eight steps (16 matrix instructions) ahead of their use, so that its latency is covered;
            // the barriers keep the compiler from gathering the reads in pairs right in front of their use, where each pair
            // waited for LDS (96 requests e4m3 at depth 8, five row blocks: 234 us a call and 227; decode step of two layers of e4m3
            // trees 138 and 130).
            constexpr int NOPS = 4 * NB, AHEAD = QLDS ? (NOPS < 8 ? NOPS : 8) : 1;
            uint4 qb[AHEAD];
            if constexpr (QLDS) {
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) qb[i] = qs[((i % NB) * 4 + i / NB) * 64];
            }
#pragma unroll
            for (int i = 0; i < NOPS; ++i) {
                const int ks = i / NB, nb = i % NB;
                bf16x8 qop;
                if constexpr (QLDS) {
                    qop = __builtin_bit_cast(bf16x8, qb[i % AHEAD]);
                    if (i + AHEAD < NOPS) {
                        const int i2 = i + AHEAD;
                        qb[i % AHEAD] = qs[((i2 % NB) * 4 + i2 / NB) * 64];
                    }
                } else {
                    qop = qreg[nb][ks];
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) s[nb][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[h][ks], qop, s[nb][h], 0, 0, 0);
                if constexpr (QLDS) __builtin_amdgcn_sched_barrier(0);
            }
        }

        {
            if constexpr (!SINGLE) {
                pack_values();
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (decltype(refill)::value) {
                    if constexpr (STAGE) issue_values(t);
                    else issue(t);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // Slots at or past kv_len may hold anything (NaN, inf): they are cleared so that 0 * garbage cannot
            // occur.  Only the last pair of a cache has such slots.
            if (ti * kPairTokens + kPairTokens > L) {
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    const int p0 = tok0 + t2 * kTile;
                    const uint32_t m01 = (p0 + 0 < L ? 0x0000ffffu : 0u) | (p0 + 1 < L ? 0xffff0000u : 0u);
                    const uint32_t m23 = (p0 + 2 < L ? 0x0000ffffu : 0u) | (p0 + 3 < L ? 0xffff0000u : 0u);
#pragma unroll
                    for (int mb = 0; mb < 8; ++mb) {
                        vop[mb][2 * t2] &= m01;
                        vop[mb][2 * t2 + 1] &= m23;
                    }
                }
            }
        }

        // Online softmax with a lagging reference: p = 2^(s - m_ref).  The reference only moves
        // (and the accumulators are rescaled) when some score exceeds it by more than kSlack, so
        // p <= 2^kSlack and the common pair needs no cross-lane traffic and no rescale.  The common path forms
        // the exponent's argument with one fused multiply-add per score and tests all of them against the slack
        // at once; the scores themselves are only formed on the rare path (before a unit's first pair the
        // reference is so low that the argument has absorbed them).
        // Every row sees all of the context before the request's new tokens, so only the last pair or two of a
        // unit need the selects: the wave-uniform test skips them for the rest.
        const bool tail = ti * kPairTokens + kPairTokens > ctx;
        auto arguments = [&](int nb, const float4v (&s)[2], float (&pd)[2][4]) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) pd[h][e] = __builtin_fmaf(s[h][e], kscale[h], -m_run[nb]);
        };
        auto mask = [&](int nb, float (&pd)[2][4]) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int p0 = tok0 + h * kTile;
                if constexpr (TREE) {
                    // Positions past the cache end are past the mask's last set bit.
                    const uint32_t vis = tree_visible4(newmask[nb], p0 - ctx);
#pragma unroll
                    for (int e = 0; e < 4; ++e) pd[h][e] = ((vis >> e) & 1u) ? pd[h][e] : -INFINITY;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)   // causal limit among the new tokens / end of the cache
                        pd[h][e] = (p0 + e > lim[nb]) ? -INFINITY : pd[h][e];
                }
            }
        };
        auto top8 = [](const float (&pd)[2][4]) __attribute__((always_inline)) {
            return fmaxf(fmaxf(fmaxf(pd[0][0], pd[0][1]), fmaxf(pd[0][2], pd[0][3])),
                         fmaxf(fmaxf(pd[1][0], pd[1][1]), fmaxf(pd[1][2], pd[1][3])));
        };
        auto rescale = [&](int nb, const float4v (&s)[2], float (&pd)[2][4]) __attribute__((always_inline)) {
            float sv[2][4];   // the scores, masked where the argument was
            float mx = -INFINITY;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sv[h][e] = pd[h][e] == -INFINITY ? -INFINITY : s[h][e] * kscale[h];
                    mx = fmaxf(mx, sv[h][e]);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run[nb], mx);
            // (Before a unit's first pair there is nothing to rescale.  Not by the reference: scores of exactly kNoMax leave
            // it where it was, and their mass has to go with the first larger score.)
            if (__any(l_run[nb] != 0.f)) {
                const float alpha = __builtin_amdgcn_exp2f(m_run[nb] - m_new);
                l_run[nb] *= alpha;
#pragma unroll
                for (int mb = 0; mb < 8; ++mb) {
                    const float4v c = acc[mb][nb];
                    float4v r = {from_accumulator_file(c[0]) * alpha, from_accumulator_file(c[1]) * alpha,
                                 from_accumulator_file(c[2]) * alpha, from_accumulator_file(c[3]) * alpha};
                    to_accumulator_file(r);
                    acc[mb][nb] = r;
                }
            }
            m_run[nb] = m_new;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) pd[h][e] = sv[h][e] - m_new;
        };
        auto output = [&](int nb, const float (&pd)[2][4]) __attribute__((always_inline)) {
            uint32_t pw[4];
            float sum[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(pd[h][e]);
                sum[h] = (p[0] + p[1]) + (p[2] + p[3]);
                const float2v lo = {p[0] * vscale[h], p[1] * vscale[h]}, hi = {p[2] * vscale[h], p[3] * vscale[h]};
                pw[2 * h] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
                pw[2 * h + 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
            }
            l_run[nb] += sum[0] + sum[1];
            const bf16x8 pop = __builtin_bit_cast(bf16x8, make_uint4(pw[0], pw[1], pw[2], pw[3]));
#pragma unroll
            for (int mb = 0; mb < 8; ++mb)
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8, make_uint4(vop[mb][0], vop[mb][1], vop[mb][2], vop[mb][3])), pop, acc[mb][nb], 0, 0, 0);
        };

        {
            float pd[NB][2][4];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) arguments(nb, s[nb], pd[nb]);
            if (tail) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) mask(nb, pd[nb]);
            }
            float top = top8(pd[0]);
#pragma unroll
            for (int nb = 1; nb < NB; ++nb) top = fmaxf(top, top8(pd[nb]));
            if (__any(top > kSlack)) {
                accumulator_read_guard();
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    if (__any(top8(pd[nb]) > kSlack)) rescale(nb, s[nb], pd[nb]);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) output(nb, pd[nb]);
        }
    };

    // ---- the walk: a ring of two pairs in registers ----
    begin_unit_issue();   // queries of the first unit go out before any KV tile
    PairRegs<FP8> buf[SINGLE ? 1 : 2];
    load_pair(buf[0], run.addr[0]);   // the first pairs' addresses come with the descriptor
    if constexpr (!SINGLE) load_pair(buf[1], run.addr[1]);
    next_addr = run.addr[SINGLE ? 1 : 2];
    begin_unit_wait();
    for (;;) {
        int tile = pos - unit_x;
        if constexpr (SINGLE) {
            for (; seg_left > 0; --seg_left) {
                compute(buf[0], tile, std::true_type{});
                tile += stride;
            }
        } else {
            // A segment of odd length begins with a step of its own, so that the loop takes both buffers in turn with one way
            // out: with an exit after either buffer the compiler either sees a path on which the first buffer's loads are the
            // newest, and drains the whole ring at the top, or spills.
            if (seg_left & 1) {
                compute(buf[0], tile, std::false_type{});
                tile += stride;
                --seg_left;
                buf[0] = buf[SINGLE ? 0 : 1];
                issue(buf[SINGLE ? 0 : 1]);
            }
            for (; seg_left > 0; seg_left -= 2) {
                compute(buf[0], tile, std::true_type{});
                compute(buf[SINGLE ? 0 : 1], tile + stride, std::true_type{});
                tile += 2 * stride;
            }
        }
        pos = unit_x + tile;
        end_unit(seg_x0 == unit_x, seg_x1 == unit_x + nb_tiles);
        if constexpr (STAGE) {
            if (team && nbu) run.free_block = nbu & 1;
            stage = reinterpret_cast<u32x4 *>(o_lds[run.free_block * kWavesPerWg + wslot]);
        }
        if (seg_x1 >= x1) break;
        next_unit();
        begin_unit_issue();
        begin_unit_wait();
    }
}

// A span of the class kernels, class by class: units of k row blocks are walked by the code for k.
//   cls, class_end  class of the span's first unit, and where that class ends
template <int G, int BLOCKS, bool FP8, bool TREE, bool STAGE>
__device__ __forceinline__ void walk_classes(const AttnArgs &a, StreamLds<BLOCKS> &lds, Run run, bool team, int cls, int class_end,
                                             const AttnPlan *__restrict__ plan, const int2 *__restrict__ pair_addr,
                                             const AttnReq *__restrict__ req, const float *__restrict__ k_scale,
                                             const float *__restrict__ v_scale)
{
    const int end = run.x1;
    // (the first class's end comes with the descriptor: the plan's record would be one more read in a row before the
    // first pair, 0.5 % of the whole call: 221.8 -> 220.5 us with 96 e4m3 requests, 278.8 -> 277.4 with 128 ragged ones)
    run.x1 = class_end < end ? class_end : end;
    for (int c = cls;;) {
        if (run.x0 < run.x1) {
            const int blocks = BLOCKS - c;
            if (blocks == 1) walk<G, 1, BLOCKS, FP8, TREE, false, STAGE>(a, lds, run, team, pair_addr, req, k_scale, v_scale);
            else if (blocks == 2) walk<G, 2, BLOCKS, FP8, TREE, false, STAGE>(a, lds, run, team, pair_addr, req, k_scale, v_scale);
            else if (blocks == 3) walk<G, 3, BLOCKS, FP8, TREE, false, STAGE>(a, lds, run, team, pair_addr, req, k_scale, v_scale);
            else {
                if constexpr (BLOCKS >= 5) {
                    if (blocks == 5) walk<G, 5, BLOCKS, FP8, TREE, false, STAGE>(a, lds, run, team, pair_addr, req, k_scale, v_scale);
                    else walk<G, 4, BLOCKS, FP8, TREE, false, STAGE>(a, lds, run, team, pair_addr, req, k_scale, v_scale);
                }
            }
        }
        if (run.x1 >= end) break;
        // the next class begins with its first request
        const int place = plan->class_req[c];
        ++c;
        if (place >= a.batch) break;
        const AttnReq r = req[place];
        run.p = place; run.g = 0; run.b = r.b; run.n = r.n;
        run.x0 = run.unit_x = run.x1;
        run.L = r.L; run.q0 = r.q0; run.q1 = r.q1;
#pragma unroll
        for (int j = 0; j < kDescPairs; ++j) {
            const int x = run.x0 + (team ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + j * kWavesPerWg : j);
            run.addr[j] = pair_addr[x < end ? x : end - 1];
        }
        const int next_end = plan->class_x[c];
        run.x1 = next_end < end ? next_end : end;
    }
}

// BLOCKS  the most 16-row blocks of query rows a unit can have
// MIXED   more than two row blocks: the spans may be wavefronts' as well as teams' (with fewer than two units to a team they never
//         are, and the code of a team alone is 0.5 to 0.8 us faster in a call of 16 us)
// STAGE   keys turned through LDS (see stage_keys)
template <int G, int BLOCKS, bool FP8, bool TREE, bool MIXED, bool STAGE>
__global__ __launch_bounds__(64 * kWavesPerWg, 1) void attn_stream_kernel(
    AttnArgs a, const AttnPlan *__restrict__ plan, const int2 *__restrict__ pair_addr, const int32_t *__restrict__ wave_desc,
    const AttnReq *__restrict__ req, const float *__restrict__ k_scale, const float *__restrict__ v_scale)
{
    // The metadata arrays come in as separate no-alias arguments so that their wave-uniform reads
    // become scalar loads (own counter, no ordering against the vector KV loads).
    __shared__ StreamLds<BLOCKS> lds;
    const int wslot = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // where this wave's span starts: written by the plan kernel (waves past the partition count start at the end of all pairs).  It
    // ends where the next one starts.
    const int32_t *d = wave_desc + (long long)(blockIdx.x * kWavesPerWg + wslot) * kDescInts;
    Run run;
    run.p = d[0]; run.g = d[1]; run.b = d[16]; run.n = d[17];
    run.x0 = d[4];
    const int next_team = wave_desc[(long long)(blockIdx.x + 1) * kWavesPerWg * kDescInts + 4], next_wave = d[kDescInts + 4];
    const bool team = !MIXED || __builtin_amdgcn_readfirstlane(d[15]) == kSpanTeam;   // (the same for the whole call)
    run.x1 = team ? next_team : next_wave;
    run.unit_x = run.x0 - d[2];
    run.L = d[6]; run.q0 = d[7]; run.q1 = d[8];
    run.free_block = 1;   // (wavefronts that hand over write finished blocks through the other one)
#pragma unroll
    for (int j = 0; j < kDescPairs; ++j) run.addr[j] = make_int2(d[9 + 2 * j], d[10 + 2 * j]);
    if constexpr (BLOCKS <= kChainRowBlocks) {
        if (team) {
            if (run.x0 >= run.x1) return;
            walk<G, BLOCKS, BLOCKS, FP8, TREE, false, false>(a, lds, run, true, pair_addr, req, k_scale, v_scale);
        } else {
            if ((threadIdx.x & 63) == 0) lds.dep_flag[wslot] = 0;
            __syncthreads();   // every wave's flag is clear before any neighbour can look at it
            if (run.x0 >= run.x1) return;
            walk<G, BLOCKS, BLOCKS, FP8, TREE, true, false>(a, lds, run, false, pair_addr, req, k_scale, v_scale);
        }
    } else {
        // (In one trip to memory: left to the compiler, some of it is read behind the test for an empty span, and some again further
        // down: 0.3 us of a short call.  The kernels above read it so by themselves.)
        int cls = d[3], class_end = d[5];
        asm volatile("" : "+s"(run.p), "+s"(run.g), "+s"(run.b), "+s"(run.n), "+s"(run.x0), "+s"(run.unit_x), "+s"(run.L), "+s"(run.q0), "+s"(run.q1), "+s"(cls), "+s"(class_end));
        asm volatile("" : "+s"(run.addr[0].x), "+s"(run.addr[0].y), "+s"(run.addr[1].x), "+s"(run.addr[1].y), "+s"(run.addr[2].x), "+s"(run.addr[2].y));
        if (run.x0 >= run.x1) return;
        walk_classes<G, BLOCKS, FP8, TREE, STAGE>(a, lds, run, team, cls, class_end, plan, pair_addr, req, k_scale, v_scale);
    }
}

// ---------------------------------------------------------------------------------------------
// merge: workgroup (unit, slab) combines the partials of 8 * PER query rows of one unit, PER rows to a lane.  Most workgroups find
// their unit finished or their rows past its own and end at once, so a call with more of them than the chip holds is better off with
// half as many (PER 2; 96 requests of up to 72 rows over 8 KV heads 9.8 -> 7.9 us, 128 of up to 36 7.8 -> 5.7, 128 short ones of
// up to 72 81.8 -> 78.5 a whole call); below that a lane's second row only lengthens its chain of additions (one request of 8000
// tokens 25.3 -> 28.2 a call).
// ---------------------------------------------------------------------------------------------
constexpr int kMergeBusy = 2048;   // workgroups of 8 rows that the chip holds at once (eight to a compute unit)

template <int G, int PER>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a)
{
    const int slabs = a.rows_pad / (8 * PER);
    const int unit = blockIdx.x / slabs, slab = blockIdx.x % slabs;
    const int g = unit % a.num_kv_heads;
    const AttnReq r = a.req[unit / a.num_kv_heads];
    const int q0 = r.q0;
    const int rows = window_q_len(r.q1 - q0, a.q_lo, a.q_win) * G;   // rows of this pass's window
    const int n = slab * (8 * PER) + (threadIdx.x >> 5), d4 = threadIdx.x & 31;
    SpanCuts cuts;
    cuts.total_w = a.plan->total_cost;
    cuts.nw = a.plan->spans;
    if ((n >= rows) | (cuts.nw == cuts.total_w)) return;   // (a span per unit: nothing is left; read together with the request's record)
    // The spans were cut at w*total_cost/spans in the weighted coordinate (every unit: what opening it costs, then its
    // pairs); the last wave whose cut lies at or before coordinate t is ((t+1)*spans - 1) / total_cost.  A cut
    // inside the opening's part starts at the unit's first pair, so the unit's first wave is the last one at
    // or before the end of that part and the first pair, its last wave the last one before the next unit's stretch.
    const int cost = a.plan->class_cost[r.cls], weight = a.plan->class_weight[r.cls];
    int w_first, w_last;
    cuts.unit_spans(r.cpre * a.num_kv_heads + (long long)g * (weight + (long long)r.n * cost), r.n, weight, cost, w_first, w_last);
    if (a.plan->mode == kSpanChain) {   // the streaming kernel has combined the spans of each workgroup: one partial per workgroup
        w_first /= kWavesPerWg;
        w_last /= kWavesPerWg;
    }
    if (w_first == w_last) return;   // the unit lies in one span (of a wavefront, of a workgroup): finished there

    // running merge: (m, l, o) <- (m, l, o) (+) partial, both relative to their own reference m
    float m_all[PER], l_all[PER];
    float4v o[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        m_all[i] = kNoMax;
        l_all[i] = 0.f;
        o[i] = float4v{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll 4
    for (int w = w_first; w <= w_last; ++w) {
        const long long first = ((long long)w + unit) * a.rows_pad + n;   // (rows past the unit's are inside its slot: rows_pad)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const long long row = first + i * 8;
            const float2 ml = *reinterpret_cast<const float2 *>(a.part_ml + row * 2);
            const float4v op = *reinterpret_cast<const float4v *>(a.part_o + row * D + d4 * 4);
            const float m_new = fmaxf(m_all[i], ml.x);
            const float wa = exp2f(m_all[i] - m_new), wb = exp2f(ml.x - m_new);  // a partial without visible tokens has l = 0
            l_all[i] = l_all[i] * wa + ml.y * wb;
            o[i] = o[i] * wa + op * wb;
            m_all[i] = m_new;
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int nn = n + i * 8;
        if (nn >= rows) return;
        const float inv = 1.f / l_all[i];
        const int qi = a.q_lo + nn / G, hh = nn % G;
        const long long orow = (long long)(q0 + qi) * a.num_q_heads + g * G + hh;
        const float2v lo = {o[i].x * inv, o[i].y * inv}, hi = {o[i].z * inv, o[i].w * inv};
        uint2 pk;
        pk.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
        pk.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
        *reinterpret_cast<uint2 *>(static_cast<__bf16 *>(a.out) + orow * D + d4 * 4) = pk;
        if (a.lse && d4 == 0) a.lse[orow] = (m_all[i] + log2f(l_all[i])) * kLn2;
    }
}

template <int G, int BLOCKS, bool FP8, bool TREE>
int32_t launch_stream(const AttnArgs &a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1)
{
    // One wavefront per SIMD (the whole register file; a ring of two pairs, three or four spill in most instances and
    // were slower where they just fit): two waves on a SIMD
    // do not share the memory pipeline fairly under saturation (the older one wins), which turns
    // into a long tail.
    // When a profile is being taken the two events are attached to the dispatch itself, so that
    // their difference is the kernel's own duration on this stream (what a kernel trace shows).
    const bool few = BLOCKS > kChainRowBlocks && (long long)a.batch * a.num_kv_heads < 2 * (a.launch_waves / kWavesPerWg);
    // Keys turned through LDS or read as operands, where a call may have two units to a team (direct / turned, 64 heads over 8 unless said; the
    // two forms in turn).  Up to three row blocks from 24 tiles on: 300 requests of 20..100 tokens, depth 2..4, 49.8 / 50.2 us, of 50..500 76.0 /
    // 73.6, of 100..1000 114.3 / 106.8, 96 of 512..8192 196.7 / 179.3.  With four and five the turn costs what the reads gain while a call is
    // short (depth 2..8: 160 of 20..1300 61.9 / 63.2, 300 of 50..500 89.9 / 91.4, 80 of 300..3000 97.0 / 97.7) and pays from 256 tiles of table to a
    // wavefront on (64 of 512..8192 159.8 / 154.1, 96 223.5 / 216.9, 500 of 100..1500 242.9 / 232.3; 96 trees of 8..16 nodes, 32 heads, 213.5 / 208.4;
    // all requests at depth 8, every unit of five row blocks, 230.8 / 233.9 and 266.2 / 266.7, which the bound of the rows does not tell).
    constexpr bool CLASSES = BLOCKS > kChainRowBlocks;
    const bool deep = a.q_win * G > 48;
    const bool stage = FP8 && CLASSES && !few && (deep ? (long long)a.batch * a.num_kv_heads * a.max_blocks >= 256ll * a.launch_waves : a.max_blocks >= 24);
    const auto kernel = few     ? attn_stream_kernel<G, BLOCKS, FP8, TREE, !CLASSES, false>
                        : stage ? attn_stream_kernel<G, BLOCKS, FP8, TREE, true, FP8 && CLASSES>
                                : attn_stream_kernel<G, BLOCKS, FP8, TREE, true, false>;
    hipExtLaunchKernelGGL(kernel, dim3((unsigned)(a.launch_waves / kWavesPerWg)),
                          dim3(64 * kWavesPerWg), 0, stream, ev0, ev1, 0, a, a.plan, a.pair_addr, a.wave_desc, a.req, a.k_scale,
                          a.v_scale);
    SS_HIP_CHECK(hipGetLastError(), "launch attn_stream_kernel");
    const long long slabs = (long long)a.batch * a.num_kv_heads * (a.rows_pad / 8);   // of 8 rows
    if (slabs >= kMergeBusy)
        hipLaunchKernelGGL((attn_merge_kernel<G, 2>), dim3((unsigned)(slabs / 2)), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((attn_merge_kernel<G, 1>), dim3((unsigned)slabs), dim3(256), 0, stream, a);
    SS_HIP_CHECK(hipGetLastError(), "launch attn_merge_kernel");
    return SS_OK;
}

template <int G, int BLOCKS>
int32_t launch_nb(const AttnArgs &a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1)
{
    if (a.tree_mask) {
        if (a.kv_dtype == SS_FP8_E4M3) return launch_stream<G, BLOCKS, true, true>(a, stream, ev0, ev1);
        return launch_stream<G, BLOCKS, false, true>(a, stream, ev0, ev1);
    }
    if (a.kv_dtype == SS_FP8_E4M3) return launch_stream<G, BLOCKS, true, false>(a, stream, ev0, ev1);
    return launch_stream<G, BLOCKS, false, false>(a, stream, ev0, ev1);
}

template <int G>
int32_t launch_for_group(const AttnArgs &a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1)
{
    const int nb = (a.q_win * G + 15) / 16;   // row blocks of one pass's window
    if constexpr (attn_team_blocks(G) > kChainRowBlocks)
        if (nb > kChainRowBlocks) return launch_nb<G, attn_team_blocks(G)>(a, stream, ev0, ev1);
    if (nb == 2) return launch_nb<G, 2>(a, stream, ev0, ev1);
    return launch_nb<G, 1>(a, stream, ev0, ev1);
}

}  // namespace
}  // namespace ss
