// Per-tile arithmetic of the mean-of-probabilities score stage (Sec. 3.1 Eq. 1;
// Sec. 4.1 Eq. 8-9 with the softmax taken per text query, then averaged), used
// by score_prob.hip.
//
// A 16 x 16 product tile holds, in lane (lr, lg), the logits of keys
// 16 t + 4 lg + r (r = 0..3) against query lr of a 16-query block.  The form of the terms
// is decided for a whole query chunk, and each lane's sums run over its tiles in
// ascending order, so the results do not depend on how many tiles a wave takes at once
// (the library is compiled without floating-point contraction).
#pragma once

#include "e2s_device.h"
#include "score_common.h"

namespace e2s {

typedef float f32x4v __attribute__((ext_vector_type(4)));

namespace prob {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;

// expm1(s y) = s y P(y) with P the Taylor series of the scaled argument:
// coefficients s^k / (k+1)! for k = 1 .. DEG-1.  Degree 5 on |s y| <= 1/8 and
// degree 6 on |s y| <= 1/4 (truncation x^7 / 5040, below 6e-8 relative there)
// stay under one float32 ulp.  The scale is applied once per sum instead of once
// per logit, and the callers fold the last product into their running sums.
template <int DEG>
struct ScaledSeries {
    float c[DEG - 1];
    __device__ explicit ScaledSeries(float s) {
        float pk = 1.0f, f = 1.0f;
#pragma unroll
        for (int kk = 1; kk < DEG; ++kk) {
            pk *= s;
            f *= static_cast<float>(kk + 1);
            c[kk - 1] = pk / f;
        }
    }
    __device__ __forceinline__ float operator()(float y) const {
        float p = c[DEG - 2];
#pragma unroll
        for (int kk = DEG - 3; kk >= 0; --kk) p = fmaf(p, y, c[kk]);
        return fmaf(p, y, 1.0f);
    }
};

// 16 keys x 16 queries on the matrix cores, fp32 accumulation from zero.
template <int NA>
__device__ __forceinline__ f32x4v tile_mma(const bf16x8 (&a)[NA], const bf16x8 (&b)[NA]) {
    f32x4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NA; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[s], acc, 0, 0, 0);
    return acc;
}
template <int NA>
__device__ __forceinline__ f32x4v tile_mma(const f16x8 (&a)[NA], const f16x8 (&b)[NA]) {
    f32x4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NA; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s], b[s], acc, 0, 0, 0);
    return acc;
}
template <int NA>
__device__ __forceinline__ f32x4v tile_mma(const float (&a)[NA], const float (&b)[NA]) {
    f32x4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NA; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], acc, 0, 0, 0);
    return acc;
}

// Range of the tight path: every centred logit |s (z - c_t)| of a query chunk
// within 1/16.  There expm1 to degree 4 (terms up to x^4 / 24) truncates below
// x^5 / 120, i.e. 1.3e-7 of the term at the edge and far less for the bulk of the
// logits (about 1/100 at the workloads' scale).
constexpr float kTightRange = 0.0625f;
// Up to here expm1 is taken to degree 8: the first term left out, (1/2)^8 / 9! relative to
// the argument, is below 1.4e-8 of the result on either side.
constexpr float kMidRange = 0.5f;
// The scales the degree-8 series takes: its coefficients s^k / (k + 1)!, k <= 7, are
// finite and normal there (at s = 10^6, s^7 is not).  Other scales skip that form.
constexpr float kMidScaleMin = 0x1p-15f, kMidScaleMax = 0x1p18f;
// Beyond kMidRange the terms are e^(s y) itself where every row of the query chunk is
// spread (block_spread).  A term's rounding is then about 2^-24 whatever its distance from
// 1, which the rounding of such a row's logits outweighs.  A row near its mean would lose
// digits (its N P - 1 is small): a chunk that has one takes expm1(s y).
constexpr float kSpreadDistance = 0.15f;
// The largest |s y| without the row's largest logit as reference: e^(s y) stays below 2^87.
constexpr float kReferenceRange = 60.0f;
constexpr float kLog2e = 1.44269504088896340736f, kLn2 = 0.69314718055994530942f;

// Reference of a query (in logit units, before the scale): the mean logit
// Q_t.K_n over keys 0..15, summed pairwise so that equal logits give exactly
// their value, or key 0's logit when N < 16.  z: the product of key tile 0 with
// the query block; every lane of the wave gets the value of its query lr.
__device__ __forceinline__ float block_reference(const f32x4v& z, int N, int lr) {
    float sum = (z[0] + z[1]) + (z[2] + z[3]);
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    const float z0 = __shfl(z[0], lr);            // key 0, from lane (lr, 0)
    return (N >= 16) ? sum * (1.0f / 16.0f) : z0;
}

// Pass 1, near uniform: E += expm1(s y) = s y P(y) (in units of s) for the
// tile's logits with y = z - c_t / s; keys past N count as y = 0.  P: the
// degree-4 series in the tight range (|s y| <= 1/16), else degree 5 (<= 1/8).
// amax: the largest |y| seen, to confirm afterwards that the range held.  WHOLE:
// the caller knows that every key of the tile is below N (the same arithmetic
// without the masking).  SPLIT: x = y P(y) is rounded before it is added (as the
// weighted column sums take it), else added in one fused step.
template <bool WHOLE, bool SPLIT, typename Series>
__device__ __forceinline__ void series_tile(const f32x4v& z, float cz, int key0, int N,
                                            const Series& p, float& E, float& amax) {
    const bool full = WHOLE || key0 + 4 <= N;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float y = z[r] - cz;
        if (!full) y = (key0 + r < N) ? y : 0.f;
        amax = fmaxf(amax, fabsf(y));
        if constexpr (SPLIT)
            E += p(y) * y;
        else
            E = fmaf(p(y), y, E);
    }
}

// Every row of a query block is spread: of keys 0..3, 4..7, 8..11 and 12..15 at least three
// groups have a key kSpreadDistance or more from the row's reference in s y (one far key
// does not make a row spread).  From the product of key tile 0 with the block (keys past
// N: the last one again); rows: how many of its rows count.  64 Gaussian rows: deviation
// 0.2 one head in twenty, 0.3 most, 1 all.
__device__ __forceinline__ bool block_spread(const f32x4v& z, float cz, float scale, int rows) {
    const float m = fmaxf(fmaxf(fabsf(z[0] - cz), fabsf(z[1] - cz)),
                          fmaxf(fabsf(z[2] - cz), fabsf(z[3] - cz)));
    const uint64_t far = __ballot(m * scale >= kSpreadDistance);     // lane (lr, lg): bit 16 lg + lr
    const uint32_t a = ~static_cast<uint32_t>(far), b = ~static_cast<uint32_t>(far >> 32);
    const uint32_t a1 = a >> 16, b1 = b >> 16;
    const uint32_t close = (a & a1) | (b & b1) | ((a | a1) & (b | b1));   // two groups without
    return (close & ((1u << min(max(rows, 0), 16)) - 1u)) == 0u;
}

// expm1(t ln 2) to about an ulp at any distance from 0: 2^t - 1 = 2^n (2^f - 1) + (2^n - 1)
// with n the nearest integer and |f| <= 1/2, 2^f - 1 by its Taylor series (the first term
// left out, (ln 2 / 2)^7 / 8! of the argument, is below 1.8e-8 of it).
__device__ __forceinline__ float expm1_base2(float t) {
    constexpr double L = 0.69314718055994530942;
    t = t < -126.0f ? -126.0f : t;                // (-1 from there; NaN stays)
    const float n = __builtin_rintf(t);
    const float f = t - n;
    float p = static_cast<float>(L * L * L * L * L * L * L / 5040.0);
    p = fmaf(p, f, static_cast<float>(L * L * L * L * L * L / 720.0));
    p = fmaf(p, f, static_cast<float>(L * L * L * L * L / 120.0));
    p = fmaf(p, f, static_cast<float>(L * L * L * L / 24.0));
    p = fmaf(p, f, static_cast<float>(L * L * L / 6.0));
    p = fmaf(p, f, static_cast<float>(L * L / 2.0));
    p = fmaf(p, f, static_cast<float>(L)) * f;
    const float s = __builtin_ldexpf(1.0f, static_cast<int>(n));
    return fmaf(p, s, s - 1.0f);
}

// Pass 1, expm1 form: E += expm1(s y), its argument as in exp_tile.
template <bool WHOLE>
__device__ __forceinline__ void expm1_tile(const f32x4v& z, float k2, float ck, int key0, int N,
                                           float& E, float& amax) {
    const bool full = WHOLE || key0 + 4 <= N;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float t = fmaf(z[r], k2, -ck);
        if (!full) t = (key0 + r < N) ? t : 0.f;
        amax = fmaxf(amax, fabsf(t));
        E += expm1_base2(t);
    }
    // (tile after tile: interleaved, the series' registers would cost the kernel a
    // workgroup per CU at d = 64)
    __builtin_amdgcn_sched_barrier(0);
}

// Pass 1, exponential form: S += e^(s y) by the hardware exponential, its argument
// s y log2(e) = z k2 - ck in one rounding (ck rounds alike for the whole row, so its
// error cancels in the softmax).  amax: the largest argument (in base 2).
template <bool WHOLE>
__device__ __forceinline__ void exp_tile(const f32x4v& z, float k2, float ck, int key0, int N,
                                         float& S, float& amax) {
    const bool full = WHOLE || key0 + 4 <= N;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float t = fmaf(z[r], k2, -ck);
        if (!full) t = (key0 + r < N) ? t : 0.f;
        amax = fmaxf(amax, fabsf(t));
        float v = __builtin_amdgcn_exp2f(t);
        if (!full) v = (key0 + r < N) ? v : 0.f;
        S += v;
    }
}

// Pass 2, near uniform: col += expm1(s y) / s = y P(y) with y = z - shift, per key
// of the tile, over the query blocks in order; P: the degree-6 series (|s y| <=
// 1/4), or in the tight range degree 4 (|s y| <= 1/16) or 5 (<= 1/8).
template <typename Series>
__device__ __forceinline__ void column_series_tile(const f32x4v& z, float sz, const Series& p,
                                                   float (&col)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float y = z[r] - sz;
        col[r] = fmaf(p(y), y, col[r]);
    }
}

// Sum over a head's queries of a per-query value held by lane t of one wave (0 in
// lanes past N_T; at most 64 queries): the butterfly of wave_sum, whose order
// depends only on the lanes, so every kernel that takes it gets the same bits.
__device__ __forceinline__ float query_sum(float v) { return wave_sum(v); }

// Pass 2, series with weights: col += w_t x with x = y P(y), y = z - c_t, evaluated
// exactly as pass 1 evaluates it (series_tile, SPLIT), over the query blocks in order.
// Keys past N are not masked: their sums are never kept.
template <typename Series>
__device__ __forceinline__ void column_weighted_tile(const f32x4v& z, float cz, const Series& p,
                                                     float w, float (&col)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float y = z[r] - cz;
        col[r] = fmaf(w, p(y) * y, col[r]);
    }
}

// The same in the exponential form: col += w_t e^(s y).
__device__ __forceinline__ void column_exp_tile(const f32x4v& z, float k2, float ck, float w,
                                                float (&col)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
        col[r] = fmaf(w, __builtin_amdgcn_exp2f(fmaf(z[r], k2, -ck)), col[r]);
}

// The same in the expm1 form: col += w_t x - b_t, b_t = E_t / S_t.
__device__ __forceinline__ void column_expm1_tile(const f32x4v& z, float k2, float ck, float w,
                                                  float b, float (&col)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) col[r] += fmaf(w, expm1_base2(fmaf(z[r], k2, -ck)), -b);
    __builtin_amdgcn_sched_barrier(0);
}

// Sums of four values over the 16 lanes of a DPP row: lane p of each quad ends with
// the sum of col[p].  The first two steps halve the values each lane carries (it sends
// the ones it drops), so 11 operations do what four full butterflies and the choice
// between their results take 19 for.  Lanes of equal p hold the same bits.
__device__ __forceinline__ float row_sums4(const float (&col)[4], int lr) {
    constexpr int kRowRor4 = 0x124, kRowRor8 = 0x128;
    const bool odd = lr & 1, high = lr & 2;
    const float a = (odd ? col[1] : col[0]) + dpp<kQuadSwap1>(odd ? col[0] : col[1]);
    const float b = (odd ? col[3] : col[2]) + dpp<kQuadSwap1>(odd ? col[2] : col[3]);
    float v = (high ? b : a) + dpp<kQuadSwap2>(high ? a : b);
    v += dpp<kRowRor8>(v);
    v += dpp<kRowRor4>(v);
    return v;
}

}  // namespace prob
}  // namespace e2s
