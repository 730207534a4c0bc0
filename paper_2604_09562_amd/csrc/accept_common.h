// Pieces shared by the acceptance kernels (chain rule in accept.hip, sampled tree walk in accept_tree.hip):
// constants, the workspace carve-up of the row-statistics and resampling passes, vocabulary loads, block
// reductions with a fixed order and the fp64 exponential.
#pragma once

#include "common.h"

namespace ss {
namespace {

constexpr int kThreads = 256;
constexpr int kSub = 2048;                     // vocabulary entries per workgroup in the fp64 passes
constexpr int kSubPer = kSub / kThreads;       // 8 logits per lane there
constexpr int kMaxRows = 2 * SS_MAX_DEPTH + 1; // rows of one request: k+1 target, k draft
constexpr double kLog2eD = 1.4426950408889634;

struct RowPick {      // written by decide, read by the resampling passes
    int32_t p_row;    // target row the new token is drawn from
    int32_t q_row;    // draft row of the rejected position, -1 if every draft was accepted
    float m_p, m_q;   // exact row maxima
    float temperature;
    int32_t n;        // accepted length
    // The difference of the two logits at which p == q, T log(Zp/Zq) + m_p - m_q with Zp/Zq as known from the fp32 row statistics
    // (relative error below 2e-5), and the half-width of the zone around it that is left to the exact normalisers.
    float theta, width;
};

constexpr int kAmbCap = 4096;       // listed boundary entries per request; beyond that the slow exact path runs
constexpr double kAmbEps = 1.0e-4;  // relative half-width of the boundary zone around p == q
constexpr int kPickWgs = 8;         // workgroups per request in the last pass (all but one idle unless the list overflowed)

struct Workspace {
    float *cmax, *csum;   // [rows][nchunks]
    int32_t *carg;        // [rows][nchunks]
    RowPick *pick;        // [batch]
    double *zp, *zq, *sc; // [batch][nsub]: sums of exp over all entries of the block (p row, q row), block mass
    double *pp, *qq;      // [batch][nsub]: the same sums over the entries with p clearly above q
    int32_t *amb_cnt;     // [batch] entries in the boundary zone (may exceed kAmbCap: then the list is not used)
    int32_t *done;        // [batch] workgroups of the last pass that have delivered their block masses
    int32_t *blk_base, *blk_cnt;  // [batch][nsub] where in the list a block's entries start, and how many they are
    double *amb_ep, *amb_eq;  // [batch][kAmbCap] their unnormalised exponentials, each block's entries contiguous
    int nchunks, nsub, rows;
};

__host__ __device__ inline int num_chunks(int vocab) { return (vocab + kChunk - 1) / kChunk; }
__host__ __device__ inline int num_sub(int vocab) { return (vocab + kSub - 1) / kSub; }

__host__ Workspace carve(void *ws, int batch, int total_rows, int vocab)
{
    Workspace w;
    w.nchunks = num_chunks(vocab);
    w.nsub = num_sub(vocab);
    w.rows = 2 * total_rows - batch;
    char *p = static_cast<char *>(ws);
    const size_t per = align_up(sizeof(float) * (size_t)w.rows * w.nchunks, 256);
    w.cmax = reinterpret_cast<float *>(p); p += per;
    w.csum = reinterpret_cast<float *>(p); p += per;
    w.carg = reinterpret_cast<int32_t *>(p); p += per;
    w.pick = reinterpret_cast<RowPick *>(p); p += align_up(sizeof(RowPick) * (size_t)batch, 256);
    const size_t perd = align_up(sizeof(double) * (size_t)batch * w.nsub, 256);
    w.zp = reinterpret_cast<double *>(p); p += perd;
    w.zq = reinterpret_cast<double *>(p); p += perd;
    w.sc = reinterpret_cast<double *>(p); p += perd;
    w.pp = reinterpret_cast<double *>(p); p += perd;
    w.qq = reinterpret_cast<double *>(p); p += perd;
    const size_t pera = align_up(sizeof(double) * (size_t)batch * kAmbCap, 256);
    w.amb_ep = reinterpret_cast<double *>(p); p += pera;
    w.amb_eq = reinterpret_cast<double *>(p); p += pera;
    const size_t peri = align_up(sizeof(int32_t) * (size_t)batch * w.nsub, 256);
    w.blk_base = reinterpret_cast<int32_t *>(p); p += peri;
    w.blk_cnt = reinterpret_cast<int32_t *>(p); p += peri;
    w.amb_cnt = reinterpret_cast<int32_t *>(p); p += align_up(sizeof(int32_t) * (size_t)batch, 256);
    w.done = reinterpret_cast<int32_t *>(p); p += align_up(sizeof(int32_t) * (size_t)batch, 256);
    return w;
}

// ---- loading one lane's share of a block of N*TH vocabulary entries (TH lanes share the block) ----
// Coalesced order: lane t owns entries base + it*(TH*vec) + t*vec + j (vec = 8 for bf16, 4 for f32).
// Sequential order (the inverse-CDF search): lane t owns base + t*N .. + N-1.
// Out-of-vocabulary positions read as -inf.  index_of() gives the vocabulary id of slot s.
// DT is the logit dtype (SS_BF16 or SS_F32): the kernels are compiled once per dtype.
template <int DT, int N, bool SEQ, int TH = kThreads>
__device__ __forceinline__ int index_of(int base, int tid, int s)
{
    if (SEQ) return base + tid * N + s;
    constexpr int vec = DT == SS_BF16 ? 8 : 4;
    return base + (s / vec) * (TH * vec) + tid * vec + (s % vec);
}

template <int DT, int N, bool SEQ, int TH = kThreads>
__device__ __forceinline__ void load_slots(const void *row, int vocab, int base, int tid, float (&x)[N])
{
    constexpr int vec = DT == SS_BF16 ? 8 : 4;
    if (base + N * TH <= vocab) {   // whole block inside the vocabulary (uniform): plain 16-byte loads
        uint4 w[N / vec];
#pragma unroll
        for (int it = 0; it < N / vec; ++it) {
            const int i0 = index_of<DT, N, SEQ, TH>(base, tid, it * vec);
            if constexpr (DT == SS_BF16)
                w[it] = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(row) + i0);
            else
                w[it] = *reinterpret_cast<const uint4 *>(static_cast<const float *>(row) + i0);
        }
#pragma unroll
        for (int it = 0; it < N / vec; ++it) {
            const uint32_t ww[4] = {w[it].x, w[it].y, w[it].z, w[it].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (DT == SS_BF16) {
                    x[it * 8 + 2 * j] = __uint_as_float(ww[j] << 16);
                    x[it * 8 + 2 * j + 1] = __uint_as_float(ww[j] & 0xffff0000u);
                } else {
                    x[it * 4 + j] = __uint_as_float(ww[j]);
                }
            }
        }
        return;
    }
    // The block that holds the end of the vocabulary.  Every lane still issues 16-byte loads (from a
    // clamped, in-bounds address, so that they pipeline); lanes whose vector lies past the end drop
    // the data, and the one vector that straddles the end is read element by element.
    const int last_full = vocab >= vec ? (vocab - vec) / vec * vec : -1;
#pragma unroll
    for (int it = 0; it < N / vec; ++it) {
        const int i0 = index_of<DT, N, SEQ, TH>(base, tid, it * vec);
        uint4 w = make_uint4(0, 0, 0, 0);
        if (last_full >= 0) {
            const int ic = i0 < last_full ? i0 : last_full;
            if constexpr (DT == SS_BF16)
                w = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(row) + ic);
            else
                w = *reinterpret_cast<const uint4 *>(static_cast<const float *>(row) + ic);
        }
        const bool whole = i0 + vec <= vocab;
        const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (DT == SS_BF16) {
                x[it * 8 + 2 * j] = whole ? __uint_as_float(ww[j] << 16) : -INFINITY;
                x[it * 8 + 2 * j + 1] = whole ? __uint_as_float(ww[j] & 0xffff0000u) : -INFINITY;
            } else {
                x[it * 4 + j] = whole ? __uint_as_float(ww[j]) : -INFINITY;
            }
        }
        if (!whole && i0 < vocab) {
#pragma unroll
            for (int j = 0; j < vec; ++j) {
                if (i0 + j < vocab) {
                    if constexpr (DT == SS_BF16)
                        x[it * vec + j] = __uint_as_float((uint32_t) static_cast<const uint16_t *>(row)[i0 + j] << 16);
                    else
                        x[it * vec + j] = static_cast<const float *>(row)[i0 + j];
                }
            }
        }
    }
}

template <int DT>
__device__ __forceinline__ void unpack(const uint4 &w, float (&x)[DT == SS_BF16 ? 8 : 4])
{
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if constexpr (DT == SS_BF16) {
            x[2 * j] = __uint_as_float(ww[j] << 16);
            x[2 * j + 1] = __uint_as_float(ww[j] & 0xffff0000u);
        } else {
            x[j] = __uint_as_float(ww[j]);
        }
    }
}

// Eight logits of a row from vocabulary id i0 on (a multiple of 8); positions past the vocabulary read as -inf.
template <int DT>
struct Raw8 {
    uint4 w[DT == SS_BF16 ? 1 : 2];
};
template <int DT>
__device__ __forceinline__ void load8(const void *row, int vocab, int i0, Raw8<DT> &r)
{
    if (i0 + 8 <= vocab) {
        const uint4 *p = reinterpret_cast<const uint4 *>(static_cast<const char *>(row) + (int64_t)i0 * (DT == SS_BF16 ? 2 : 4));
#pragma unroll
        for (int j = 0; j < (DT == SS_BF16 ? 1 : 2); ++j) r.w[j] = p[j];
        return;
    }
    uint32_t e[8];   // the end of the vocabulary, entry by entry
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if constexpr (DT == SS_BF16)
            e[j] = i0 + j < vocab ? static_cast<const uint16_t *>(row)[i0 + j] : 0xff80u;
        else
            e[j] = i0 + j < vocab ? static_cast<const uint32_t *>(row)[i0 + j] : 0xff800000u;
    }
    if constexpr (DT == SS_BF16) {
        r.w[0] = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
    } else {
        r.w[0] = make_uint4(e[0], e[1], e[2], e[3]);
        r.w[1] = make_uint4(e[4], e[5], e[6], e[7]);
    }
}
template <int DT>
__device__ __forceinline__ void unpack8(const Raw8<DT> &r, float (&x)[8])
{
    if constexpr (DT == SS_BF16) {
        unpack<DT>(r.w[0], x);
    } else {
        float lo[4], hi[4];
        unpack<DT>(r.w[0], lo);
        unpack<DT>(r.w[1], hi);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[j] = lo[j];
            x[4 + j] = hi[j];
        }
    }
}

__device__ __forceinline__ const void *row_ptr(const void *base, int64_t row, int64_t stride, int dtype)
{
    return static_cast<const char *>(base) + row * stride * (dtype == SS_BF16 ? 2 : 4);
}

__device__ __forceinline__ float load_logit(const void *base, int64_t row, int64_t stride, int dtype, int v)
{
    const void *r = row_ptr(base, row, stride, dtype);
    if (dtype == SS_BF16) return __uint_as_float((uint32_t) static_cast<const uint16_t *>(r)[v] << 16);
    return static_cast<const float *>(r)[v];
}

// ---- block reductions with a fixed order ---------------------------------------------------
__device__ __forceinline__ float block_max(float v, float *sh)
{
    for (int off = 32; off; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}
template <typename T>
__device__ __forceinline__ T block_sum(T v, T *sh)
{
    for (int off = 32; off; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// ---- sums across a wavefront in lane order, by data-parallel moves (no LDS round trips) -----------
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double x)
{
    constexpr bool all = ROWS == 0xf;   // lanes without a source read 0 by the instruction itself, not from a register cleared for them
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, all);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, all);
    return x + __hiloint2double(hi, lo);
}
// Inclusive running sums of x over the lanes; lane 63 holds the total.  A fixed association.
__device__ __forceinline__ double wave_scan(double x)
{
    x = dpp_add<0x111, 0xf>(x);   // row_shr 1, 2, 4, 8: running sums inside each row of 16 lanes
    x = dpp_add<0x112, 0xf>(x);
    x = dpp_add<0x114, 0xf>(x);
    x = dpp_add<0x118, 0xf>(x);
    x = dpp_add<0x142, 0xa>(x);   // row_bcast 15: the sum of row 0 to row 1, of row 2 to row 3
    x = dpp_add<0x143, 0xc>(x);   // row_bcast 31: the sum of rows 0 and 1 to rows 2 and 3
    return x;
}
// Lanes 0..31: x of the lane and of the lane 32 further; lanes 32..63: y of the lane and of the lane 32 in front.
__device__ __forceinline__ double fold32(double x, double y)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(y), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// Rows of 16 lanes in pairs: even rows get x of both rows of their pair, odd rows y.
__device__ __forceinline__ double fold16(double x, double y)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(y), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// Sums of four values over the wavefront, in a fixed association: lanes 0..15 hold that of a, then c, b and d, each in its
// row's last lane (15, 31, 47, 63).  Every step halves the values that a lane still carries: a third of the instructions of
// four scans, which were a quarter of what a block of the fp64 passes issues.
__device__ __forceinline__ double wave_sum4(double a, double b, double c, double d)
{
    double x = fold16(fold32(a, b), fold32(c, d));
    x = dpp_add<0x111, 0xf>(x);
    x = dpp_add<0x112, 0xf>(x);
    x = dpp_add<0x114, 0xf>(x);
    return dpp_add<0x118, 0xf>(x);
}
// Which of the four values the caller's row of lanes holds.
__device__ __forceinline__ int sum4_index(int lane) { return ((lane >> 4) & 1) * 2 + (lane >> 5); }
__device__ __forceinline__ double lane_value(double x, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// ---- fp64 exponential for non-positive arguments -----------------------------------------------
// Arguments come in steps of the table, y = x * 64/ln2 (RowArg folds the factor into 1 / T): exp(x) = 2^e * 2^(j/64) * exp(f ln2/64) with
// y = 64 e + j + f, |f| <= 1/2 and exact, a 64-entry table of 2^(j/64) in LDS and a degree-5 Taylor polynomial in f (remainder <
// 4e-17 relative).  Reducing x itself takes a two-part ln2/64 and one instruction more: 11 fp64 ones with the conversion and the
// argument, instead of 12.
// 2^(j/64), j = 0..63, each the double nearest to the exact value (tests/test_exp_table.py recomputes them)
static __device__ const double kExp2Sixtyfourths[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};

constexpr double kExpSteps = 92.33248261689366;   // 64 / ln2
constexpr double kExpNormal = -700.0 * kExpSteps;   // from here up ExpTable::normal may be used
constexpr double kExpMass = -722.0 * kExpSteps;     // from here down an exponential (2^-1041) is not worth a place in a list of boundary entries

struct ExpTable {
    // 2^(j/64) with j << 14 taken from its upper word: k << 14, k = 64 e + j, added to that makes it 2^(e + j/64)
    double t[64];
    __device__ void init()
    {
        if (threadIdx.x < 64) {
            const double v = kExp2Sixtyfourths[threadIdx.x];
            t[threadIdx.x] = __hiloint2double(__double2hiint(v) - ((int)threadIdx.x << 14), __double2loint(v));
        }
        __syncthreads();
    }
    // 2^(f/64), f in steps of the table, and k, the nearest integer to y
    __device__ __forceinline__ double fraction(double y, int &k) const
    {
        // y to the nearest integer: added to 1.5 * 2^52 it lands in the low bits of the significand
        constexpr double magic = 0x1.8p52, step = 0.010830424696249145;   // ln2 / 64
        const double kd = y + magic;
        k = __double2loint(kd);
        const double f = y - (kd - magic);
        constexpr double c1 = step, c2 = step * step / 2, c3 = step * step * step / 6, c4 = step * step * step * step / 24,
                         c5 = step * step * step * step * step / 120;
        return fma(fma(fma(fma(fma(f, c5, c4), f, c3), f, c2), f, c1), f, 1.0);
    }
    __device__ __forceinline__ double operator()(double y) const
    {
        int k;
        const double p = fraction(fmax(y, -746.0 * kExpSteps), k);   // exp underflows to 0 from there on (also covers -inf)
        const double v = t[k & 63];
        return ldexp(__hiloint2double(__double2hiint(v) + ((k & 63) << 14), __double2loint(v)) * p, k >> 6);
    }
    // the same bits for -700 <= x <= 1, where the result is normal and the power of two goes into the table's exponent
    __device__ __forceinline__ double normal(double y) const
    {
        int k;
        const double p = fraction(y, k);
        const double v = t[k & 63];
        return __hiloint2double(__double2hiint(v) + (k << 14), __double2loint(v)) * p;
    }
};

// Argument of the exponential of a logit, (x - max) / T, in steps of the table.  As one fused multiply-add x / T - max / T where max / T is small
// enough: its rounding (below 1.2e-10 there) is a factor common to all of the row's exponentials, which the normaliser takes
// out again, and far inside the boundary zone of p == q.  Beyond that (a tiny temperature, enormous logits) the rounding would
// be as large as the arguments themselves -- at T = 1e-18 every exponential of a row underflowed or overflowed -- so there
// the difference is formed first, which is exactly 0 at the row's maximum.
constexpr double kFusedArgMax = 0x1p20;
struct RowArg {
    double inv_t, c;
    float sub;
    bool fused;   // uniform: all lanes of a workgroup hold the same row
    __device__ __forceinline__ RowArg(double inv_t_, float m) : inv_t(inv_t_ * kExpSteps)
    {
        const double mt = (double)m * inv_t;
        const bool f = fabs(mt) < kFusedArgMax * kExpSteps;   // (false for a row without a finite maximum)
        c = f ? -mt : 0.0;
        fused = __builtin_amdgcn_readfirstlane(f);
        sub = fused ? 0.f : m;
    }
    __device__ __forceinline__ double operator()(float x) const { return fma((double)x - (double)sub, inv_t, c); }
    __device__ __forceinline__ double fma_form(float x) const { return fma((double)x, inv_t, c); }   // the same bits if `fused`
};

// What is left of r where q is taken from it (nothing, if that is no number), of two products of an exponential and a reciprocal.  Both are
// rounded before they are subtracted: a fused multiply-add, which rounds one of them only, leaves 1e-17 of two equal ones, and a
// residual that has vanished would have mass.
__device__ __forceinline__ double residual_of(double r, double q)
{
#pragma clang fp contract(off)
    return fmax(r - q, 0.0);
}

// The smaller of two logits, NaN if either is (one instruction for three operands): the tests that admit a wavefront to
// ExpTable::normal must see a NaN, which the general form takes as no mass.
__device__ __forceinline__ float min_or_nan(float a, float b) { return __builtin_elementwise_minimum(a, b); }

// Exponentials of eight logits.  Whether all of the wavefront's are normal numbers (those of masked logits are not) is
// one test.
__device__ __forceinline__ void exp8(const ExpTable &ex, const RowArg &arg, const float (&x)[8], double (&e)[8])
{
    float low = x[0];
#pragma unroll
    for (int s = 1; s < 8; ++s) low = min_or_nan(low, x[s]);
    if (arg.fused && !__any(!(arg.fma_form(low) >= kExpNormal))) {
#pragma unroll
        for (int s = 0; s < 8; ++s) e[s] = ex.normal(arg.fma_form(x[s]));
    } else {
#pragma unroll
        for (int s = 0; s < 8; ++s) e[s] = ex(arg(x[s]));
    }
}

// ---- row statistics of one request: a 256-lane workgroup merges the chunk statistics -------------------------
// Rows target0 .. target0 + k and draft0 .. draft0 + k - 1 (offsets into the statistics) become row_m[0 .. 2k] and
// row_z[0 .. 2k].  Sixteen rows at a time: every quarter of a wavefront (16 lanes over the chunks) merges one row, so
// the rows of an ordinary request are done in one trip.  The caller's barrier publishes them.
__device__ __forceinline__ void merge_row_stats(const Workspace &w, int64_t target0, int64_t draft0, int k, double inv_t,
                                                float *row_m, double *row_z)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quarter = lane >> 4, ql = lane & 15;
    const int nrows = 2 * k + 1;
    for (int j0 = 0; j0 < nrows; j0 += 16) {
        const int j = j0 + wave * 4 + quarter;
        const bool live = j < nrows;
        const int64_t ry = !live ? 0 : (j <= k ? target0 + j : draft0 + (j - k - 1));
        const float *cmax = w.cmax + ry * w.nchunks, *csum = w.csum + ry * w.nchunks;
        // (the lane's first chunk, usually its only one, is read once and both of its numbers together)
        const bool has = live && ql < w.nchunks;
        const float cm0 = has ? cmax[ql] : -INFINITY, cs0 = has ? csum[ql] : 0.f;
        float m = cm0;
        if (live)
            for (int c = ql + 16; c < w.nchunks; c += 16) m = fmaxf(m, cmax[c]);
        for (int off = 8; off; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));   // (stays inside the quarter)
        double z = 0.0;
        if (cm0 != -INFINITY) z = (double)cs0 * exp2(((double)cm0 - (double)m) * inv_t * kLog2eD);
        if (live)
            for (int c = ql + 16; c < w.nchunks; c += 16) {
                const float cm = cmax[c];
                if (cm != -INFINITY) z += (double)csum[c] * exp2(((double)cm - (double)m) * inv_t * kLog2eD);
            }
        for (int off = 8; off; off >>= 1) z += __shfl_xor(z, off);
        if (live && ql == 0) {
            row_m[j] = m;
            row_z[j] = z;
        }
    }
}

// ---- the draw: inverse-CDF search of a 256-lane workgroup ------------------------------------------------------
// Lane t owns a contiguous run of 2048-entry blocks (one, up to vocabularies of 512k entries), so that one scan of
// the lanes' sums serves any number of blocks.
__device__ __forceinline__ int blocks_per_lane(int nsub) { return (nsub + kThreads - 1) / kThreads; }

struct DrawShared {
    double scan[4], entry[4], prefix;
    int first[4], last[4], efirst[4], elast[4], cstar, tok;
};

// mass_of(c): mass of block c, asked for the lane's own blocks only; entries(c, r): the masses of the lane's entries
// c * 2048 + 8 * tid .. of block c.  Returns, in every lane, the first token whose running sum of masses exceeds u times
// their total (the last one with mass if rounding leaves none), or -1 if there is no mass.
template <class MassOf, class Entries>
__device__ __forceinline__ int draw_token(int nsub, float u, DrawShared &sh, MassOf mass_of, Entries entries)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = blocks_per_lane(nsub), c0 = tid * per, c1 = min(c0 + per, nsub);
    // Running sum of the lanes' masses in block order: the total S, and the first lane with mass whose running sum
    // exceeds u * S.
    double own = 0.0;
    int own_last = -1;   // last block of this lane with mass
    for (int c = c0; c < c1; ++c) {
        const double v = mass_of(c);
        own += v;
        if (v > 0.0) own_last = c;
    }
    const double incl_w = wave_scan(own);
    if (lane == 63) sh.scan[wave] = incl_w;
    __syncthreads();
    double before_w = 0.0;
    for (int wv = 0; wv < wave; ++wv) before_w += sh.scan[wv];
    const double S = ((sh.scan[0] + sh.scan[1]) + sh.scan[2]) + sh.scan[3];
    if (!(S > 0.0)) return -1;
    const double thr = (double)u * S;
    const double cum = before_w + incl_w;   // running sum through this lane's last block
    const unsigned long long over = __ballot(own > 0.0 && cum > thr), some = __ballot(own > 0.0);
    if (lane == 0) {
        sh.first[wave] = over ? wave * 64 + (__ffsll((long long)over) - 1) : 0x7fffffff;
        sh.last[wave] = some ? wave * 64 + (63 - __clzll((long long)some)) : -1;
    }
    __syncthreads();
    const int first_lane = min(min(sh.first[0], sh.first[1]), min(sh.first[2], sh.first[3]));
    const bool take_last = first_lane == 0x7fffffff;  // rounding left u*S at or past the total: last entry with mass
    const int owner = take_last ? max(max(sh.last[0], sh.last[1]), max(sh.last[2], sh.last[3])) : first_lane;
    if (tid == owner) {
        // inside the lane's run of blocks: the first with mass whose running sum crosses (rounding may leave none: then
        // the last with mass)
        double run = cum - own;
        double pre = run;
        int cs = own_last;
        if (per > 1) {
            bool found = false;
            for (int c = c0; c < c1; ++c) {
                const double v = mass_of(c);
                if (v > 0.0 && !found) {
                    cs = c;
                    pre = run;
                    found = !take_last && run + v > thr;
                }
                run += v;
            }
        }
        sh.cstar = cs;
        sh.prefix = pre;
    }
    __syncthreads();
    const int cstar = sh.cstar;
    double r[kSubPer];
    entries(cstar, r);
    double local = 0.0;
    int my_last = -1;
#pragma unroll
    for (int i = 0; i < kSubPer; ++i) {
        local += r[i];
        if (r[i] > 0.0) my_last = cstar * kSub + tid * kSubPer + i;
    }
    // exclusive prefix of `local` over lanes in index order
    const double incl = wave_scan(local);
    if (lane == 63) sh.entry[wave] = incl;
    int lw = my_last;
    for (int off = 32; off; off >>= 1) lw = max(lw, __shfl_xor(lw, off));
    if (lane == 0) sh.elast[wave] = lw;
    __syncthreads();
    double before = sh.prefix;
    for (int wv = 0; wv < wave; ++wv) before += sh.entry[wv];
    const double excl = before + (incl - local);
    // first lane with mass whose running sum crosses the threshold (the scan groups its additions differently for every lane,
    // so the sum at a lane without mass may lie an ulp above that of the lane in front of it)
    const unsigned long long bal = __ballot(!take_last && local > 0.0 && excl + local > thr);
    if (lane == 0) sh.efirst[wave] = bal ? wave * 64 + (__ffsll((long long)bal) - 1) : 0x7fffffff;
    __syncthreads();
    const int first = min(min(sh.efirst[0], sh.efirst[1]), min(sh.efirst[2], sh.efirst[3]));
    if (first == 0x7fffffff) return max(max(sh.elast[0], sh.elast[1]), max(sh.elast[2], sh.elast[3]));
    if (tid == first) {
        double c = excl;
        int tok = -1;
#pragma unroll
        for (int i = 0; i < kSubPer; ++i) {
            if (r[i] > 0.0) {
                c += r[i];
                if (tok < 0 && c > thr) tok = cstar * kSub + tid * kSubPer + i;
            }
        }
        // the lane total crossed but the element-wise sum may round differently: then its last entry with mass
        sh.tok = tok >= 0 ? tok : my_last;
    }
    __syncthreads();
    return sh.tok;
}

// Lowest vocabulary id of a row that holds `value` (in every lane of a 256-lane workgroup).
__device__ __forceinline__ int lowest_index_of(const void *rows, int64_t row, int64_t stride, int dtype, int vocab, float value,
                                               DrawShared &sh)
{
    int arg = 0x7fffffff;
    for (int v = threadIdx.x; v < vocab; v += kThreads)
        if (load_logit(rows, row, stride, dtype, v) == value) { arg = v; break; }
    for (int off = 32; off; off >>= 1) arg = min(arg, __shfl_xor(arg, off));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.first[threadIdx.x >> 6] = arg;
    __syncthreads();
    return min(min(sh.first[0], sh.first[1]), min(sh.first[2], sh.first[3]));
}

}  // namespace
}  // namespace ss
