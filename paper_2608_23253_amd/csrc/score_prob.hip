// Score stage, mean-of-probabilities reading: for every text query t a softmax
// over the visual tokens of the scaled logits z[t, n] = Q_t.K_n * scale, then the
// mean over the queries, r_n = mean_t P[t, n]; support as in Eq. 9 (Sec. 4.1).
//
// Unlike the mean-of-logits reading this is a genuine dense contraction
// (N_T x N_V logits per head), computed on the matrix cores with
// v_mfma_f32_16x16x32_bf16 / _f16 (bf16 / fp16 storage) or v_mfma_f32_16x16x4_f32
// (fp32 storage), fp32 accumulation.  One workgroup owns one (image, layer, query head).
// Its text queries (chunks of up to 128 rows) are staged in LDS as the B operand;
// key tiles of 16 rows are loaded from HBM straight into A-operand registers, so a
// 16x16 result tile holds 16 keys (4 per lane) x 16 queries (one per lane).  Two
// passes over the keys:
//
//   pass 1  row statistics of the lane's query: with a reference c_t (the mean
//           scaled logit of keys 0..15), E_t = sum_n expm1(z s - c_t), then
//           L_t = log(S_t / N) with S_t = N + E_t, so that z s - c_t - L_t is the
//           centred logit
//   pass 2  per key: sum over queries of  N P[t,n] - 1 = expm1(z s - c_t - L_t),
//           accumulated in-lane over all query blocks, then summed across the 16
//           query lanes of a DPP row
//
// so u_n = N r_n - 1 = (1/N_T) sum_t expm1(z[t,n] s - c_t - L_t) is accumulated in
// centred form; e_n = u_n / (2 (2 + u_n)), r_n = (1 + u_n) / N.
//
// The form of the terms goes by the largest |s y| of a query chunk, y = z - c_t / s:
//   up to 1/16 (Gaussian keys at the 1/sqrt(d) scale)  expm1 by the series of degree 4
//      in both passes (5 in pass 2 when some |L_t| widens its range): five to seven
//      vector operations per logit and pass
//   up to 1/8    degree 5, in pass 2 degree 6 (|s y - L_t| <= 1/4, since L_t lies
//      between the smallest and largest s y)
//   up to 1/2    x = expm1(s y) by degree 8; with S_t = N + E_t the softmax is
//      (1 + x) / S_t, so N P - 1 = w_t x - E_t / S_t with w_t = N / S_t: the column
//      sums weight the pass-1 terms instead of re-centring them (scales far from 1,
//      whose powers leave float32's range, skip this form)
//   beyond, every row spread (the attention of a trained model; prob::block_spread)
//      e^(s y) itself by the hardware exponential (quarter rate, 6.5 issue slots per logit with
//      its argument and sum), N P - 1 = w_t e^(s y) - 1; where some logit lies more than
//      60 from its row's reference, the row's largest logit becomes the reference first
//   beyond, some row near its mean  x = expm1(s y) from 2^n and a series (16 slots),
//      N P - 1 = w_t x - E_t / S_t per term; where a logit lies more than 60 from the
//      reference or some S_t = N + E_t is below N / 2, the log of the row's mean e^(s z)
//      (by the exponential form) becomes the reference first.  The exponential form
//      rounds every term at 2^-24 of 1, this one at 2^-24 of x: 63 rows of deviation
//      0.005 and one of 0.2 over 576 keys, rms error of u 1e-8 and 4e-10; 64 rows of
//      0.2, 1.0e-8 and 3.1e-9
// Every truncation stays within about one float32 ulp of the term at its range's edge
// (degree 4 at 1/16: x^5 / 120, 1.07 ulp of x) and far below it for the bulk.  Pass 1
// starts in the first form and a wave leaves it after its first key group when that
// is out of range.  The exponential form took the place of online statistics with
// the library's expm1f: unit-spread logits, 13 images of up to 2013 tokens, 28 heads
// over 4: 421 -> 178 us, and 9 times closer to the float64 result (one rounding in the
// exponent instead of a rounded shift, expm1f and a rescaled sum).
// The reference is subtracted from the product after the matrix core, not
// started in its accumulator: a product started from -c_t rounds differently from
// the product minus c_t, and exactly uniform attention (identical keys) would then
// give supports of ~1e-11 instead of exactly 0.
// The query-block loops are not unrolled (the per-lane sums live in LDS), which keeps
// the kernel's code within the instruction cache.
//
// Heads of 16-bit storage with at most 64 text queries and 385 to 576 tokens (the
// LLaVA shape) take the weighted form already in the tight range: a register-resident
// kernel keeps every x of a wave's 9 key tiles in registers, so pass 2 is one
// multiply-add per logit, with no second product, no second series and no second
// read of the keys.
//
// Query heads that share a key head (grouped-query attention) run in workgroups
// with consecutive logical ids; the ids are remapped so that those workgroups land
// on the same XCD (blocks are dispatched round-robin over the 8 XCDs) and re-read
// the shared keys from that XCD's L2.
#include <type_traits>

#include "e2s_kernels.h"
#include "score_prob_common.h"

namespace e2s {
namespace {

using prob::kThreads;
using prob::kWaves;
using prob::ScaledSeries;
using prob::tile_mma;

// Every lane's v is true, as a scalar (a branch on it is one the compiler knows to be
// taken by the whole wave: neither side's registers outlive the other's).
__device__ __forceinline__ bool wave_all(bool v) {
    return __builtin_amdgcn_readfirstlane(__all(v)) != 0;
}
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
    const int q = nblocks / 8, r = nblocks % 8;
    const int x = bid % 8, i = bid / 8;
    return x * q + min(x, r) + i;
}

constexpr int64_t kColumnsInLds = 16384;
constexpr size_t kLdsPerCu = 160 * 1024;

// Heads of 16-bit storage with at most 16 kResMaxQueryBlocks text queries whose key
// tiles give each wave kResMinTiles to kResTiles of them (385 to 576 tokens) can run
// register-resident (below; every wave runs kResTiles, so fewer tiles would waste more
// of them), and smaller heads beside them (takes_resident).  The two-pass kernel takes
// such a head with the same arithmetic in the same order, so a head's bits do not depend
// on its batch.  (Two launches for a ragged batch of both kinds measured 136 against
// 110 us for 47 images, a kernel with both bodies no gain above 1000 workgroups.)
constexpr int kResTiles = 9, kResMinTiles = 7, kResMaxQueryBlocks = 4;
// (the per-query statistics of such a head fit one wave: lane t holds query t)
static_assert(16 * kResMaxQueryBlocks <= kWave, "a head's queries in one wave");
__host__ __device__ constexpr int tiles_per_wave(int64_t N) {
    return static_cast<int>(((N + 15) / 16 + kWaves - 1) / kWaves);
}
__host__ __device__ constexpr bool resident_head(int64_t NT, int64_t N) {
    return NT <= 16 * kResMaxQueryBlocks && tiles_per_wave(N) >= kResMinTiles &&
           tiles_per_wave(N) <= kResTiles;
}
// The two-pass kernel takes the weighted form from the tight range on for those heads
// (the register-resident kernel's arithmetic) and for shorter ones, where the
// logarithm of the centred form's shift costs more latency than the weights' extra
// operation per logit (52 queries, 72 tokens: 27.0 against 25.2 us per call).
__host__ __device__ constexpr bool weighted_head(int64_t NT, int64_t N) {
    return NT <= 16 * kResMaxQueryBlocks && tiles_per_wave(N) <= kResTiles;
}

// The scale allows the degree-8 series.
__device__ __forceinline__ bool mid_scale(float scale) {
    return scale >= prob::kMidScaleMin && scale <= prob::kMidScaleMax;
}

template <typename T, int D> struct ProbCfg;
template <int D> struct ProbCfg<uint16_t, D> {
    static constexpr int QC = 128;           // query rows per LDS chunk
    static constexpr int QS = D + 8;         // padded LDS row (elements)
    static constexpr int NA = D / 32;        // A registers (bf16x8) per key tile
    using AFrag = bf16x8;
};
template <int D> struct ProbCfg<_Float16, D> {
    static constexpr int QC = 128;
    static constexpr int QS = D + 8;
    static constexpr int NA = D / 32;        // A registers (f16x8) per key tile
    using AFrag = f16x8;
};
template <int D> struct ProbCfg<float, D> {
    static constexpr int QC = 64;
    static constexpr int QS = D + 4;
    static constexpr int NA = D / 4;
    using AFrag = float;
};

// A operand (keys) of one 16-key tile for all k steps.
//   bf16, fp16: lane (lr, lg) holds key lr, elements 32 s + 8 lg .. +7 of step s.
//   fp32: lane holds key lr, element d(s, lg) = 16 (s/4) + 4 lg + s%4 of step s.
// The B operand (queries, from LDS) uses the same element mapping.
// Loads are unconditional (callers clamp the row into range and discard the
// results of keys past N), so no branch separates a load from its use and the
// next group's loads stay in flight while the current group is used.  They are
// ordinary cached loads: pass 2 (and the other query heads of a key head) read
// the same keys again, from L2 where they are still there (non-temporal loads
// measured 4-20 % slower).
template <int NS>
__device__ __forceinline__ void load_keys(bf16x8 (&a)[NS], const uint16_t* row) {
#pragma unroll
    for (int s = 0; s < NS; ++s) a[s] = *reinterpret_cast<const bf16x8*>(row + 32 * s);
}
template <int NS>
__device__ __forceinline__ void load_keys(f16x8 (&a)[NS], const _Float16* row) {
#pragma unroll
    for (int s = 0; s < NS; ++s) a[s] = *reinterpret_cast<const f16x8*>(row + 32 * s);
}
template <int NS>
__device__ __forceinline__ void load_keys(float (&a)[NS], const float* row) {
#pragma unroll
    for (int t = 0; t < NS / 4; ++t) {
        const f32x4v v = *reinterpret_cast<const f32x4v*>(row + 16 * t);
        a[4 * t + 0] = v.x;
        a[4 * t + 1] = v.y;
        a[4 * t + 2] = v.z;
        a[4 * t + 3] = v.w;
    }
}

// Query operand (B) of one 16-query block, all k steps, read from LDS once and
// reused for every key tile.  Same element mapping as the keys.
template <int D>
__device__ __forceinline__ void load_queries(bf16x8 (&b)[D / 32], const uint16_t* qs, int qrow,
                                             int lr, int lg) {
    const uint16_t* brow = qs + (qrow + lr) * (D + 8) + 8 * lg;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) b[s] = *reinterpret_cast<const bf16x8*>(brow + 32 * s);
}
template <int D>
__device__ __forceinline__ void load_queries(f16x8 (&b)[D / 32], const _Float16* qs, int qrow,
                                             int lr, int lg) {
    const _Float16* brow = qs + (qrow + lr) * (D + 8) + 8 * lg;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) b[s] = *reinterpret_cast<const f16x8*>(brow + 32 * s);
}
template <int D>
__device__ __forceinline__ void load_queries(float (&b)[D / 4], const float* qs, int qrow, int lr,
                                             int lg) {
    const float* brow = qs + (qrow + lr) * (D + 4) + 4 * lg;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        const f32x4v v = *reinterpret_cast<const f32x4v*>(brow + 16 * t);
        b[4 * t + 0] = v.x;
        b[4 * t + 1] = v.y;
        b[4 * t + 2] = v.z;
        b[4 * t + 3] = v.w;
    }
}

// TG key tiles per group, two groups in flight per wave: 4 tiles (2 workgroups per
// CU by registers, 3 at d = 64) when a chunk has 8 query blocks, else 2 (3 per CU) or 1
// (4 per CU with 16-bit keys, 5 at d = 64, where the LDS allows it; fp32 keys always take
// 1, 3 per CU).  d = 64 is bounded here because the expm1 form's registers, left to
// themselves, cost it a workgroup per CU (64 images of 289 tokens, 40 queries: 180 us
// without the bound, 169 with it).
template <typename T, int D, int TG>
constexpr int mp_workgroups_per_cu() {
    if (!std::is_same<T, float>::value && D == 64 && TG != 2) return TG >= 4 ? 3 : 5;
    return TG >= 4 ? 2 : (TG == 1 && !std::is_same<T, float>::value ? 4 : 3);
}
// The arguments of every kernel of the stage.
template <typename T> struct ProbArgs {
    const T* q;
    const T* k;
    float* e_out;
    float* r_out;                // or null
    BatchGeom bg;
    int group;                   // query heads per key head
    float scale;
    int nblocks, qcap;
    bool cols_over_stats;
};

template <typename T, int D, int TG, bool GLOBAL>
__device__ __forceinline__ void mean_prob_two_pass(const ProbArgs<T>& p, int tid) {
    using C = ProbCfg<T, D>;
    constexpr int QS = C::QS, NA = C::NA;
    using AFrag = typename C::AFrag;
    const BatchGeom& bg = p.bg;
    const int qcap = p.qcap;
    const float scale = p.scale;

    extern __shared__ __align__(16) unsigned char smem[];
    // qcap = min(QC, N_T rounded up to 16) query rows per chunk
    const int qbcap = qcap / 16;
    T* qs = reinterpret_cast<T*>(smem);                          // [qcap][QS]
    float* st_m = reinterpret_cast<float*>(qs + qcap * QS);      // [qcap] shift of each query
    float* st_c = st_m + qcap;                                   // [qcap] reference c_t
    float* wpart = st_c + qcap;                                  // [kWaves][qcap]
    float* lstat = wpart + kWaves * qcap;                        // [qbcap][kThreads]
    __shared__ unsigned s_amax;                                  // max |z - c_t| (float bits)
    __shared__ unsigned s_lmax;                                  // max |L_t| (float bits)
    __shared__ float s_fsum[2];                                  // sum_t E_t / S_t (waves 0, 1)
    __shared__ int s_close;                                      // some row is near its mean

    const int64_t bid = xcd_remap(blockIdx.x, p.nblocks);        // (b*L + l)*H + h
    const int64_t b = bid / (bg.L * bg.H);
    const int lh = static_cast<int>(bid - b * bg.L * bg.H);
    const int l = lh / bg.H, h = lh - l * bg.H;
    const ImageGeom ig = image_geom(bg, b);
    const int NT = ig.NT, N = ig.N;
    const T* qh = query_rows(p.q, bg, ig, b, l, h);
    const T* kg = key_rows(p.k, bg, ig, b, l, h / p.group);
    const int64_t qld = query_ld(bg), kld = key_ld(bg);
    const int64_t row = bg.L * bg.H * ig.tok + static_cast<int64_t>(lh) * N;
    // [N] column sums: LDS, or (GLOBAL) the head's output row, overwritten at the
    // end.  cols_over_stats: every head has one query chunk and the sums fit in the
    // per-lane statistics, which are dead once pass 1 has been merged, so the sums
    // take their place (less LDS per workgroup, more workgroups per CU).
    float* colsum = GLOBAL ? p.e_out + row
                           : (p.cols_over_stats ? lstat : lstat + qbcap * kThreads);
    const int wave = tid / kWave, lane = tid % kWave;
    const int lr = lane % 16, lg = lane / 16;
    // Key tiles of 16 rows go to the waves round-robin (wave w: tiles w, w + 4,
    // w + 8, ...), and a wave takes its own tiles TG at a time, in ascending order.
    // The tile a lane sees, and the order in which its sums run, do not depend on
    // TG, so the results do not either.
    const int ntiles = (N + 15) / 16;
    const int ntw = wave < ntiles ? (ntiles - wave + kWaves - 1) / kWaves : 0;  // this wave's
    const int ngw = (ntw + TG - 1) / TG;                                       // groups
    auto tile_of = [&](int j, int tt) { return wave + kWaves * (j * TG + tt); };
    const float fN = static_cast<float>(N);
    const int koff = std::is_same<T, float>::value ? 4 * lg : 8 * lg;
    // this lane's sum of query block qb: of x (series) or of e^(s y)
    float* lE = lstat + tid;

    // keys of this wave's group j (TG tiles of 16 rows) into A-operand registers;
    // rows past N repeat row N - 1
    auto load_group = [&](AFrag (&a)[TG][NA], int j) {
#pragma unroll
        for (int tt = 0; tt < TG; ++tt) {
            const int key = tile_of(j, tt) * 16 + lr;
            load_keys<NA>(a[tt], kg + static_cast<int64_t>(min(key, N - 1)) * kld + koff);
        }
    };

    // body(a, j) for every group j of this wave until it returns false, the next
    // group's keys requested before the current one is used.  The requests are unconditional (past the
    // last group they repeat it), so every path has the same loads in flight and
    // the wait before a group's first use leaves the next group's loads pending.
    auto stream_groups = [&](auto&& body) {
        AFrag a0[TG][NA], a1[TG][NA];
        const int last = max(ngw - 1, 0);
        load_group(a0, 0);
        for (int j = 0; j < ngw; j += 2) {
            load_group(a1, min(j + 1, last));
            if (!body(a0, j) || j + 1 >= ngw) break;
            load_group(a0, min(j + 2, last));
            body(a1, j + 1);
        }
    };

    for (int t0 = 0; t0 < NT; t0 += qcap) {
        const int rows = min(qcap, NT - t0);
        const int QB = (rows + 15) / 16;
        __syncthreads();
        // ---- stage this chunk of queries (rows past NT are zero): the thread's
        // packets are requested in two batches, each before its first store (two
        // round trips instead of one per packet, half the registers of one batch);
        // the requests are unconditional (indices past the chunk repeat its last
        // packet), so no branch makes a store wait for more than its batch
        constexpr int EPV = 16 / sizeof(T);                       // elements per 16 bytes
        constexpr int QPT = (C::QC * (D / EPV) + kThreads - 1) / kThreads;
        constexpr int QPB = (QPT + 1) / 2;                        // packets per batch
        const int packets = QB * 16 * (D / EPV);
#pragma unroll 1
        for (int i0 = 0; i0 < QPT; i0 += QPB) {
            f32x4v qv[QPB];
#pragma unroll
            for (int i = 0; i < QPB; ++i) {
                const int idx = min(tid + (i0 + i) * kThreads, packets - 1);
                const int row = idx / (D / EPV), c = idx % (D / EPV);
                qv[i] = *reinterpret_cast<const f32x4v*>(
                    qh + static_cast<int64_t>(t0 + min(row, rows - 1)) * qld + c * EPV);
            }
#pragma unroll
            for (int i = 0; i < QPB; ++i) {
                const int idx = tid + (i0 + i) * kThreads;
                const int row = idx / (D / EPV), c = idx % (D / EPV);
                const f32x4v zero = {0.f, 0.f, 0.f, 0.f};
                if (idx < packets)
                    *reinterpret_cast<f32x4v*>(qs + row * QS + c * EPV) = row < rows ? qv[i] : zero;
            }
        }
        for (int qb = 0; qb < QB; ++qb) lE[qb * kThreads] = 0.f;
        if (tid == 0) {
            s_amax = 0u;
            s_lmax = 0u;
            s_close = 0;
        }
        __syncthreads();

        // ---- reference of each query (block_reference); zero query rows past
        // N_T get 0
        {
            AFrag a0[NA];
            load_keys<NA>(a0, kg + static_cast<int64_t>(min(lr, N - 1)) * kld + koff);
            for (int qb = wave; qb < QB; qb += kWaves) {
                AFrag bq[NA];
                load_queries<D>(bq, qs, qb * 16, lr, lg);
                const f32x4v z = tile_mma<NA>(a0, bq);
                const float c = prob::block_reference(z, N, lr);
                if (lg == 0) st_c[qb * 16 + lr] = c;
                if (!prob::block_spread(z, c, scale, rows - qb * 16)) s_close = 1;
            }
        }
        __syncthreads();

        // ---- pass 1: the sums over the keys, by groups of keys, double-buffered; first
        // in the tight range (a wave stops at its first group when that leaves it),
        // then, by the largest |s y| of the chunk's logits (y = z - c_t), in the near,
        // the mid or the exponential form
        const ScaledSeries<4> p4(scale);
        const ScaledSeries<5> p5(scale);
        const ScaledSeries<6> p6(scale);
        const ScaledSeries<8> p8(scale);
        const float k2 = scale * prob::kLog2e;
        const bool weighted = weighted_head(NT, N);
        // one group of keys through every query block: add(z, query, key0, E, amax)
        auto sums_group = [&](const AFrag (&a)[TG][NA], int j, float& amax, auto&& add) {
            for (int qb = 0; qb < QB; ++qb) {
                AFrag bq[NA];
                load_queries<D>(bq, qs, qb * 16, lr, lg);
                const float cz = st_c[qb * 16 + lr];
                float E = lE[qb * kThreads];
#pragma unroll
                for (int tt = 0; tt < TG; ++tt)
                    add(tile_mma<NA>(a[tt], bq), cz, tile_of(j, tt) * 16 + 4 * lg, E, amax);
                lE[qb * kThreads] = E;
            }
        };
        // pass 1 over this wave's keys; add(whole) gives the tile step for groups with
        // and without keys past N.  first_range: stop after the first group when that
        // leaves it.
        auto sums = [&](float unit, float first_range, auto&& add) {
            float amax = 0.f;                                     // largest |y| seen
            stream_groups([&](const AFrag (&a)[TG][NA], int j) {
                // the group's last tile ends at or before N: no key of the group is
                // masked (tile_of is the same for every lane of the wave)
                if (__builtin_amdgcn_readfirstlane(tile_of(j, TG - 1)) * 16 + 16 <= N)
                    sums_group(a, j, amax, add(std::true_type{}));
                else
                    sums_group(a, j, amax, add(std::false_type{}));
                return j > 0 || wave_all(amax * unit <= first_range);
            });
            // (non-negative floats order as their bits)
            const float wmax = wave_max(amax);
            if (lane == 0) atomicMax(&s_amax, __float_as_uint(wmax * unit));
            __syncthreads();
            return __uint_as_float(s_amax);
        };
        auto series = [&](const auto& p, auto split) {
            return [&](auto whole) {
                return [&](const f32x4v& z, float cz, int key0, float& E, float& m) {
                    prob::series_tile<decltype(whole)::value, decltype(split)::value>(z, cz, key0,
                                                                                      N, p, E, m);
                };
            };
        };
        auto expm1s = [&](auto whole) {
            return [&](const f32x4v& z, float cz, int key0, float& E, float& m) {
                prob::expm1_tile<decltype(whole)::value>(z, k2, cz * k2, key0, N, E, m);
            };
        };
        auto exps = [&](auto whole) {
            return [&](const f32x4v& z, float cz, int key0, float& E, float& m) {
                prob::exp_tile<decltype(whole)::value>(z, k2, cz * k2, key0, N, E, m);
            };
        };
        // between two attempts at pass 1: the sums and the range start again
        auto restart = [&] {
            __syncthreads();                                      // (s_amax has been read)
            for (int qb = 0; qb < QB; ++qb) lE[qb * kThreads] = 0.f;
            if (tid == 0) s_amax = 0u;
            __syncthreads();
        };
        float range = weighted ? sums(scale, prob::kTightRange, series(p4, std::true_type{}))
                               : sums(scale, prob::kTightRange, series(p4, std::false_type{}));
        // each wave's part of this chunk's sums, the 4 lane groups merged
        auto wave_parts = [&] {
            for (int qb = 0; qb < QB; ++qb) {
                float e = lE[qb * kThreads];
                e += __shfl_xor(e, 16);
                e += __shfl_xor(e, 32);
                if (lg == 0) wpart[wave * qcap + qb * 16 + lr] = e;
            }
            __syncthreads();
        };
        // query tid's sum from the waves' parts
        auto query_total = [&] {
            float e = 0.f;
            for (int w = 0; w < kWaves; ++w) e += wpart[w * qcap + tid];
            return e;
        };
        // the row's largest logit becomes the reference (every s y <= 0 then), and the
        // sums of e^(s y) are taken again (S_t >= 1)
        auto sums_below_maximum = [&] {
            for (int qb = 0; qb < QB; ++qb) lE[qb * kThreads] = -INFINITY;
            float unused = 0.f;
            stream_groups([&](const AFrag (&a)[TG][NA], int j) {
                sums_group(a, j, unused,
                           [&](const f32x4v& z, float, int key0, float& E, float&) {
#pragma unroll
                               for (int r = 0; r < 4; ++r)
                                   if (key0 + r < N) E = fmaxf(E, z[r]);
                           });
                return true;
            });
            for (int qb = 0; qb < QB; ++qb) {
                float m = lE[qb * kThreads];
                m = fmaxf(m, __shfl_xor(m, 16));
                m = fmaxf(m, __shfl_xor(m, 32));
                if (lg == 0) wpart[wave * qcap + qb * 16 + lr] = m;
            }
            __syncthreads();
            if (tid < QB * 16) {
                float m = wpart[tid];
                for (int w = 1; w < kWaves; ++w) m = fmaxf(m, wpart[w * qcap + tid]);
                st_c[tid] = m;
            }
            restart();
            sums(prob::kLn2, INFINITY, exps);
        };
        enum { kTight, kNear, kMid, kExpm1, kExp } form = kTight;
        if (!(range <= prob::kTightRange)) {
            form = kExp;
            const bool near = !weighted && range <= kSeriesRange;
            if (near || (mid_scale(scale) && range <= prob::kMidRange)) {
                restart();
                range = near ? sums(scale, INFINITY, series(p5, std::false_type{}))
                             : sums(scale, INFINITY, series(p8, std::true_type{}));
                if (range <= (near ? kSeriesRange : prob::kMidRange)) {
                    form = near ? kNear : kMid;
                } else if (near && mid_scale(scale) && range <= prob::kMidRange) {
                    restart();
                    range = sums(scale, INFINITY, series(p8, std::true_type{}));
                    form = kMid;
                }
            }
            if (form == kExp && !s_close) {
                restart();
                range = sums(prob::kLn2, INFINITY, exps);
                if (!(range <= prob::kReferenceRange)) sums_below_maximum();
            } else if (form == kExp) {
                form = kExpm1;
                restart();
                range = sums(prob::kLn2, INFINITY, expm1s);
                wave_parts();
                // (a NaN sum counts as below: its results are NaN by either way)
                const bool below = tid < rows && !(query_total() >= -0.5f * fN);
                if (__syncthreads_or(below || !(range <= prob::kReferenceRange))) {
                    sums_below_maximum();
                    wave_parts();
                    if (tid < rows) st_c[tid] += logf(query_total() / fN) / scale;
                    restart();
                    sums(prob::kLn2, INFINITY, expm1s);
                    wave_parts();
                }
            }
        }

        // ---- merge the sums: the 4 lane groups, then the waves ----
        if (form != kExpm1) wave_parts();                         // (done there)
        {
            const bool centred = form == kNear || (form == kTight && !weighted);
            float ft = 0.f;
            if (tid < QB * 16) {
                const float e = query_total();
                float m = 0.f;
                if (centred) {
                    // the shift of pass 2 in logit units: c_t + L_t / s
                    float L = 0.f;
                    if (tid < rows) {
                        L = log1pf((scale * e) / fN);
                        m = st_c[tid] + L / scale;
                    }
                    atomicMax(&s_lmax, __float_as_uint(fabsf(L)));
                } else if (tid < rows) {
                    // w_t = N / S_t and E_t / S_t (rows past N_T: no weight)
                    const float Et = form == kExpm1 ? e : scale * e;
                    const float S = form == kExp ? e : fN + Et;
                    m = fN / S;
                    ft = Et / S;
                }
                st_m[tid] = m;
                if (form == kExpm1) wpart[tid] = ft;              // (only this thread reads it yet)
            }
            // (a chunk's queries lie in waves 0 and 1)
            if (!centred && wave < 2) {
                const float fs = prob::query_sum(ft);
                if (lane == 0) s_fsum[wave] = fs;
            }
        }
        __syncthreads();

        // ---- pass 2: per key, the sum over the queries of N P - 1 ----------------
        // (zero query rows past N_T have z = 0 and shift 0, or no weight: they add 0)
        // (one lane per key and one LDS access per tile: with one lane for four keys, each
        // its own access, the vector instructions of a Qwen2-VL batch were 9.9e7 against
        // 9.2e7, its time 301 against 296 us; 64 x 64 images 1346 against 1289)
        auto add_columns = [&](const float (&col)[TG][4], int j, float unit, float base) {
#pragma unroll
            for (int tt = 0; tt < TG; ++tt) {
                const float sum = prob::row_sums4(col[tt], lr);
                const int key = tile_of(j, tt) * 16 + 4 * lg + lr;
                // a key's sums are kept by one lane through every chunk, the first
                // chunk starting them (every key below N is written then)
                if (lr < 4 && key < N) {
                    const float add = unit * sum - base;
                    colsum[key] = t0 == 0 ? add : colsum[key] + add;
                }
            }
        };
        // column sums of every group: col starts at `start`; step(z, c_t, w_t, t, col)
        // adds a tile's terms of one query block (this lane's query t); unit and base as
        // in add_columns
        auto columns = [&](float start, float unit, float base, auto&& step) {
            stream_groups([&](const AFrag (&a)[TG][NA], int j) {
                float col[TG][4];
#pragma unroll
                for (int tt = 0; tt < TG; ++tt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) col[tt][r] = start;
                for (int qb = 0; qb < QB; ++qb) {
                    AFrag bq[NA];
                    load_queries<D>(bq, qs, qb * 16, lr, lg);
                    const int t = qb * 16 + lr;
                    const float cz = st_c[t], m = st_m[t];
#pragma unroll
                    for (int tt = 0; tt < TG; ++tt) step(tile_mma<NA>(a[tt], bq), cz, m, t, col[tt]);
                }
                add_columns(col, j, unit, base);
                return true;
            });
        };
        // centred: N P - 1 = expm1(s (z - shift)), in units of s; |s (z - shift)| <=
        // range + max |L_t| <= 2 range (L_t lies between the smallest and largest s y)
        auto centred = [&](const auto& p) {
            columns(0.f, scale, 0.f, [&](const f32x4v& z, float, float shift, int, float (&col)[4]) {
                prob::column_series_tile(z, shift, p, col);
            });
        };
        // weighted: N P - 1 = w_t x - E_t / S_t with x recomputed exactly as in pass 1
        auto weighted_series = [&](const auto& p) {
            const float fsum = QB * 16 > kWave ? s_fsum[0] + s_fsum[1] : s_fsum[0];
            columns(0.f, scale, fsum, [&](const f32x4v& z, float cz, float w, int, float (&col)[4]) {
                prob::column_weighted_tile(z, cz, p, w, col);
            });
        };
        if (form == kTight && weighted) {
            weighted_series(p4);
        } else if (form == kTight) {
            if (range + __uint_as_float(s_lmax) <= prob::kTightRange)
                centred(p4);
            else
                centred(p5);
        } else if (form == kNear) {
            centred(p6);
        } else if (form == kMid) {
            weighted_series(p8);
        } else if (form == kExpm1) {
            columns(0.f, 1.0f, 0.f, [&](const f32x4v& z, float cz, float w, int t, float (&col)[4]) {
                prob::column_expm1_tile(z, k2, cz * k2, w, wpart[t], col);
            });
        } else {
            // N P - 1 = w_t e^(s y) - 1, the lane's ones (its queries) taken first
            float ones = 0.f;
            for (int qb = 0; qb < QB; ++qb) ones += qb * 16 + lr < rows ? 1.f : 0.f;
            columns(-ones, 1.0f, 0.f, [&](const f32x4v& z, float cz, float w, int, float (&col)[4]) {
                prob::column_exp_tile(z, k2, cz * k2, w, col);
            });
        }
    }
    __syncthreads();

    const float inv_nt = 1.0f / static_cast<float>(NT);
    for (int n = tid; n < N; n += kThreads) {
        const float u = colsum[n] * inv_nt;
        __builtin_nontemporal_store(u / (2.0f * (2.0f + u)), p.e_out + row + n);
        if (p.r_out) p.r_out[row + n] = (1.0f + u) / fN;
    }
}

template <typename T, int D, int TG, bool GLOBAL>
__global__ __launch_bounds__(kThreads, (mp_workgroups_per_cu<T, D, TG>())) void score_mean_prob_kernel(
    ProbArgs<T> p) {
    mean_prob_two_pass<T, D, TG, GLOBAL>(p, threadIdx.x);
}

// Register-resident variant for heads of at most 16 QBN text queries whose key tiles
// give every wave at most MAXT of them (the LLaVA shape: 64 queries, 576 tokens, 9 tiles
// per wave).  Pass 1 keeps the x (or e^(s y)) of the wave's tiles in registers; the column
// sums then take one multiply-add per logit.  The forms are those above without the
// near one; a head that leaves one form's range starts over in the next (in the tight
// form after its first tile; in the two-pass stage, which computes the same bits, with
// one or two query blocks or for the expm1 form).  Each form is a body of its own from
// the products to the stored supports: with the forms meeting inside one body the
// compiler keeps two copies of the x and spills.  Measured at 64 LLaVA images in fp16 with unit-spread
// logits: 860 us per call with the two-pass kernel's library exponentials, 298 us
// here (the tight form: 260 us, 5.1 TB/s).
// A head as a workgroup of the resident kernel sees it.
template <typename T, int D, int QBN> struct ResidentHead {
    using C = ProbCfg<T, D>;
    using AFrag = typename C::AFrag;
    static constexpr int NA = C::NA, QR = 16 * QBN;
    const T* kg;                 // its key rows
    int64_t kld;
    float* e_row;                // its supports
    float* r_row;                // its shares, or null
    int NT, N;
    int wave, lane, lr, lg;
    int ntw;                     // this wave's tiles (tile j: keys key_of(j) .. + 15)
    float scale;

    __device__ __forceinline__ int key_of(int j) const { return (wave + kWaves * j) * 16; }
    // a tile past the wave's last one repeats that tile (its logits are masked), so
    // that no branch separates the loads from their uses
    __device__ __forceinline__ void load_tile(AFrag (&a)[NA], int j) const {
        const int jj = min(j, max(ntw - 1, 0));
        load_keys<NA>(a, kg + static_cast<int64_t>(min(key_of(jj) + lr, N - 1)) * kld + 8 * lg);
    }
    // key 4 lg + r of tile j counts
    __device__ __forceinline__ bool counts(int j, int r) const {
        return j < ntw && key_of(j) + 4 * lg + r < N;
    }
    // every key of tile j counts (the same for every lane; so for the first
    // kResMinTiles - 1 tiles of every wave)
    __device__ __forceinline__ bool whole(int j) const {
        return __builtin_amdgcn_readfirstlane(j < ntw && key_of(j) + 16 <= N);
    }
    // u = N r - 1 of one key per lane of each row's first four: from the row's four
    // key sums col[r], lane r taking key key0 + r, so each division runs once per key
    template <typename Centre>
    __device__ __forceinline__ void store_tile(int j, const float (&col)[4], Centre&& centre) const {
        const float sum = prob::row_sums4(col, lr);
        const int key = key_of(j) + 4 * lg + lr;
        if (j < ntw && lr < 4 && key < N) {
            const float u = centre(sum);
            __builtin_nontemporal_store(u / (2.0f * (2.0f + u)), e_row + key);
            if (r_row) r_row[key] = (1.0f + u) / static_cast<float>(N);
        }
    }
};

// LDS of the resident kernel: the queries [QR][QS], then a sum per wave and query.
template <typename T, int D, int QBN>
constexpr size_t resident_lds() {
    return 16 * QBN * ProbCfg<T, D>::QS * sizeof(T) + kWaves * 16 * QBN * sizeof(float);
}

// How a head's terms x are taken: in units of s by the series of degree 4 or 8 on
// y = z - c_t, or as e^(s y) by the hardware exponential.
enum Terms { kTightTerms, kMidTerms, kExpTerms };

// Pass 1 of a head into registers, its sums and its column sums; false if a logit
// leaves the range of TERMS (nothing is stored then).  qs: the staged queries; a: key
// tiles 0 .. KB - 2, requested; part: [kWaves][QR] floats of LDS; s_max: an LDS word
// that holds 0 bits or more of |s y| (read before the caller writes it again).
constexpr int kResKeys = 3;                                      // key tiles in registers
template <Terms TERMS, typename T, int D, int MAXT, int QBN>
__device__ __forceinline__ bool resident_terms(
    const ResidentHead<T, D, QBN>& hd, const T* qs, float* part, unsigned* s_max,
    typename ProbCfg<T, D>::AFrag (&a)[kResKeys][ProbCfg<T, D>::NA], const float (&cz)[QBN],
    bool last) {
    using AFrag = typename ProbCfg<T, D>::AFrag;
    constexpr int NA = ProbCfg<T, D>::NA, QR = 16 * QBN, KB = kResKeys;
    const int lr = hd.lr, lg = hd.lg, lane = hd.lane, wave = hd.wave, NT = hd.NT, N = hd.N;
    const float scale = hd.scale;
    constexpr bool EXP = TERMS == kExpTerms;
    constexpr float kRange = TERMS == kTightTerms ? prob::kTightRange
                             : TERMS == kMidTerms ? prob::kMidRange
                                                  : prob::kReferenceRange;
    // the first QKEEP query blocks' operands stay in registers for every tile (the
    // others are read from LDS per tile); not with two blocks, where the registers
    // would cost a wave per SIMD
    constexpr int QKEEP = QBN == 2 || TERMS != kTightTerms ? 0 : (QBN < 2 ? QBN : 2);
    AFrag bkeep[QKEEP > 0 ? QKEEP : 1][NA];
#pragma unroll
    for (int qb = 0; qb < QKEEP; ++qb) load_queries<D>(bkeep[qb], qs, qb * 16, lr, lg);
    const ScaledSeries<TERMS == kTightTerms ? 4 : 8> series(scale);
    const float k2 = scale * prob::kLog2e;
    float ref[QBN];                                              // c_t, or s c_t log2(e)
#pragma unroll
    for (int qb = 0; qb < QBN; ++qb) ref[qb] = EXP ? cz[qb] * k2 : cz[qb];
    const float unit = EXP ? prob::kLn2 : scale;                  // of amax
    float x[MAXT][QBN][4];
    float E[QBN];
#pragma unroll
    for (int qb = 0; qb < QBN; ++qb) E[qb] = 0.f;
    float amax = 0.f;
    auto step = [&](int j) {
        if (j + KB - 1 < MAXT) hd.load_tile(a[(j + KB - 1) % KB], j + KB - 1);
        // MASKED: some key of the tile is past N or the tile is past the wave's last
        // (the same values either way: masking only zeroes such keys)
        int again = 0;                                           // (the queries are read again
        if (TERMS != kTightTerms) asm volatile("" : "+v"(again));   // for every tile, not kept)
        auto tile = [&](auto masked) {
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb) {
                AFrag bq[NA];
                if (qb < QKEEP) {
#pragma unroll
                    for (int t = 0; t < NA; ++t) bq[t] = bkeep[qb < QKEEP ? qb : 0][t];
                } else {
                    load_queries<D>(bq, qs, qb * 16 + again, lr, lg);
                }
                const f32x4v z = tile_mma<NA>(a[j % KB], bq);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float y = EXP ? fmaf(z[r], k2, -ref[qb]) : z[r] - ref[qb];
                    if constexpr (decltype(masked)::value) y = hd.counts(j, r) ? y : 0.f;
                    amax = fmaxf(amax, fabsf(y));
                    float xv = EXP ? __builtin_amdgcn_exp2f(y) : series(y) * y;
                    if constexpr (EXP && decltype(masked)::value) xv = hd.counts(j, r) ? xv : 0.f;
                    x[j][qb][r] = xv;
                    E[qb] += xv;
                }
            }
        };
        if (hd.whole(j))
            tile(std::false_type{});
        else
            tile(std::true_type{});
        // keep the tiles in program order: the compiler would otherwise sink each
        // tile's loads down to its first use, which leaves none in flight
        __builtin_amdgcn_sched_barrier(0);
    };
    step(0);
    // (a head outside the tight range mostly shows it in the first tile)
    if (TERMS != kTightTerms || wave_all(amax * unit <= kRange)) {
#pragma unroll
        for (int j = 1; j < MAXT; ++j) step(j);
    }
    {
        // (non-negative floats order as their bits)
        const float wmax = wave_max(amax);
        if (lane == 0) atomicMax(s_max, __float_as_uint(wmax * unit));
    }
#pragma unroll
    for (int qb = 0; qb < QBN; ++qb) {
        float e = E[qb];
        e += __shfl_xor(e, 16);
        e += __shfl_xor(e, 32);
        if (lg == 0) part[wave * QR + qb * 16 + lr] = e;
    }
    __syncthreads();
    if (!last && __builtin_amdgcn_readfirstlane(!(__uint_as_float(*s_max) <= kRange))) return false;
    // every wave merges the statistics itself, lane t for query t (no barrier)
    const float fN = static_cast<float>(N);
    float ft = 0.f, wt = 0.f;                                    // rows past N_T: no weight
    if (lane < NT) {
        float e = 0.f;
        for (int w = 0; w < kWaves; ++w) e += part[w * QR + lane];
        const float Et = scale * e;
        const float S = EXP ? e : fN + Et;
        wt = fN / S;
        ft = Et / S;
    }
    const float fsum = EXP ? 0.f : prob::query_sum(ft);
    float wq[QBN], ones = 0.f;                                   // ones: this lane's queries
#pragma unroll
    for (int qb = 0; qb < QBN; ++qb) {
        wq[qb] = __shfl(wt, qb * 16 + lr);
        ones += EXP && qb * 16 + lr < NT ? 1.f : 0.f;
    }

    // ---- column sums: per key, sum over the queries of w_t x' -----------------
    const float inv_nt = 1.0f / static_cast<float>(NT);
#pragma unroll
    for (int j = 0; j < MAXT; ++j) {
        float col[4] = {-ones, -ones, -ones, -ones};
        if constexpr (!EXP) col[0] = col[1] = col[2] = col[3] = 0.f;
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
            for (int r = 0; r < 4; ++r) col[r] = fmaf(wq[qb], x[j][qb][r], col[r]);
        hd.store_tile(j, col, [&](float sum) { return (EXP ? sum : scale * sum - fsum) * inv_nt; });
    }
    return true;
}

template <typename T, int D, int MAXT, int QBN>
__device__ __forceinline__ void mean_prob_resident(const ProbArgs<T>& p) {
    using C = ProbCfg<T, D>;
    const BatchGeom& bg = p.bg;
    const float scale = p.scale;
    constexpr int QS = C::QS, NA = C::NA, QR = 16 * QBN, KB = kResKeys;
    static_assert(QBN >= 1 && QR <= kWave && MAXT >= KB, "resident kernel shape");
    using AFrag = typename C::AFrag;

    extern __shared__ __align__(16) unsigned char smem[];
    T* qs = reinterpret_cast<T*>(smem);                          // [QR][QS]
    float* part = reinterpret_cast<float*>(qs + QR * QS);        // [kWaves][QR]
    __shared__ unsigned s_max[3];                                // max |s (z - c_t)| (float bits)

    const int64_t bid = xcd_remap(blockIdx.x, p.nblocks);        // (b*L + l)*H + h
    const int64_t b = bid / (bg.L * bg.H);
    const int lh = static_cast<int>(bid - b * bg.L * bg.H);
    const int l = lh / bg.H, h = lh - l * bg.H;
    const ImageGeom ig = image_geom(bg, b);
    const int NT = ig.NT, N = ig.N;
    const T* qh = query_rows(p.q, bg, ig, b, l, h);
    const int64_t qld = query_ld(bg);
    const int tid = threadIdx.x;
    ResidentHead<T, D, QBN> hd;
    hd.kg = key_rows(p.k, bg, ig, b, l, h / p.group);
    hd.kld = key_ld(bg);
    const int64_t row = bg.L * bg.H * ig.tok + static_cast<int64_t>(lh) * N;
    hd.e_row = p.e_out + row;
    hd.r_row = p.r_out ? p.r_out + row : nullptr;
    hd.NT = NT;
    hd.N = N;
    hd.wave = tid / kWave;
    hd.lane = tid % kWave;
    hd.lr = hd.lane % 16;
    hd.lg = hd.lane / 16;
    // the thread's index for the two-pass stage: its wave's in a scalar register and the
    // lane's own, so that no vector register holds it through the forms (one more and the
    // kernel of four query blocks spills: 64 LLaVA images 261 -> 272 us)
    const int first_thread = __builtin_amdgcn_readfirstlane(tid);
    auto thread_again = [&] {
        return first_thread +
               static_cast<int>(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
    };
    const int ntiles = (N + 15) / 16;
    hd.ntw = hd.wave < ntiles ? (ntiles - hd.wave + kWaves - 1) / kWaves : 0;
    hd.scale = scale;
    const int lr = hd.lr, lg = hd.lg;

    // the queries are requested first, then keys 0..15 for the references and the
    // wave's first key tiles, so that staging the queries waits for them alone
    constexpr int EPV = 16 / sizeof(T);                          // elements per 16 bytes
    constexpr int QPT = (QR * (D / EPV) + kThreads - 1) / kThreads;   // packets per thread
    f32x4v qv[QPT];
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int idx = min(tid + i * kThreads, QR * (D / EPV) - 1);
        const int r = idx / (D / EPV), c = idx % (D / EPV);
        qv[i] = *reinterpret_cast<const f32x4v*>(qh + static_cast<int64_t>(min(r, NT - 1)) * qld +
                                                 c * EPV);
    }
    __builtin_amdgcn_sched_barrier(0);                           // (the request order)
    AFrag a0[NA];
    load_keys<NA>(a0, hd.kg + static_cast<int64_t>(min(lr, N - 1)) * hd.kld + 8 * lg);
    AFrag a[KB][NA];
    auto first_tiles = [&] {
#pragma unroll
        for (int j = 0; j < KB - 1; ++j) hd.load_tile(a[j], j);
    };
    first_tiles();
    __builtin_amdgcn_sched_barrier(0);

    // ---- stage the queries (rows past N_T are zero) and their references ----
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int idx = tid + i * kThreads;
        if (idx < QR * (D / EPV)) {
            const int r = idx / (D / EPV), c = idx % (D / EPV);
            const f32x4v zero = {0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<f32x4v*>(qs + r * QS + c * EPV) = r < NT ? qv[i] : zero;
        }
    }
    if (tid == 0) s_max[0] = s_max[1] = s_max[2] = 0u;
    __syncthreads();
    // every wave takes all the references itself (a few products; no barrier)
    float cz[QBN];
    bool spread = true;                                          // every row is
#pragma unroll
    for (int qb = 0; qb < QBN; ++qb) {
        AFrag bq[NA];
        load_queries<D>(bq, qs, qb * 16, lr, lg);
        const f32x4v z = tile_mma<NA>(a0, bq);
        cz[qb] = prob::block_reference(z, N, lr);
        if (QBN > 2) spread &= prob::block_spread(z, cz[qb], scale, NT - qb * 16);
    }

    if (resident_terms<kTightTerms, T, D, MAXT, QBN>(hd, qs, part, s_max, a, cz, false)) return;
    __syncthreads();                                             // (part is written again)
    if constexpr (QBN <= 2) {
        // one or two query blocks: the later forms' registers would cost the tight form
        // a workgroup per CU (26 images, 18 queries, 450 tokens, 4 heads per key head:
        // 60.7 -> 64.0 us), so the two-pass stage takes the head from the start
        mean_prob_two_pass<T, D, 1, false>(p, thread_again());
        return;
    }
    if (__builtin_amdgcn_readfirstlane(__uint_as_float(s_max[0]) <= prob::kMidRange &&
                                       mid_scale(scale))) {
        first_tiles();
        if (resident_terms<kMidTerms, T, D, MAXT, QBN>(hd, qs, part, s_max + 1, a, cz, false))
            return;
        __syncthreads();
    }
    if (!spread) {
        // a row near its mean: the expm1 form, in the two-pass stage (its LDS is at least
        // this kernel's)
        mean_prob_two_pass<T, D, 1, false>(p, thread_again());
        return;
    }
    first_tiles();
#pragma unroll
    for (int attempt = 0; attempt < 2; ++attempt) {              // (unrolled: fewer live registers)
        if (resident_terms<kExpTerms, T, D, MAXT, QBN>(hd, qs, part, s_max + 2, a, cz,
                                                       attempt > 0))
            return;
        // some logit lies far from its row's reference: the row's largest logit
        // becomes the reference (every s y <= 0 then, and S_t >= 1)
        __syncthreads();
        float mx[QBN];
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) mx[qb] = -INFINITY;
#pragma unroll 1
        for (int j = 0; j < hd.ntw; ++j) {
            hd.load_tile(a[0], j);
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb) {
                AFrag bq[NA];
                load_queries<D>(bq, qs, qb * 16, lr, lg);
                const f32x4v z = tile_mma<NA>(a[0], bq);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (hd.counts(j, r)) mx[qb] = fmaxf(mx[qb], z[r]);
            }
        }
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            mx[qb] = fmaxf(mx[qb], __shfl_xor(mx[qb], 16));
            mx[qb] = fmaxf(mx[qb], __shfl_xor(mx[qb], 32));
            if (lg == 0) part[hd.wave * QR + qb * 16 + lr] = mx[qb];
        }
        __syncthreads();
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            cz[qb] = part[qb * 16 + lr];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) cz[qb] = fmaxf(cz[qb], part[w * QR + qb * 16 + lr]);
        }
        __syncthreads();                                         // (part is written again)
        first_tiles();
    }
}

// Workgroups per CU: as many as the registers of the x allow.
template <typename T, int D, int QBN>
__global__ __launch_bounds__(kThreads, QBN == 1 ? 4 : QBN == 2 ? 3 : 2) void score_mean_prob_resident_kernel(
    ProbArgs<T> p) {
    mean_prob_resident<T, D, kResTiles, QBN>(p);
}

// LDS of one workgroup: the column sums in LDS up to kColumnsInLds keys, else in
// the output rows; in the statistics' place when every head has one query chunk
// and they fit (over).
template <typename T, int D>
size_t mp_lds(const Dims& d, int qcap, bool& global, bool& over) {
    using C = ProbCfg<T, D>;
    global = d.N > kColumnsInLds;
    const int64_t stats = (qcap / 16) * kThreads;                // floats
    over = !global && d.NT <= qcap && d.N <= stats;
    return static_cast<size_t>(qcap) * C::QS * sizeof(T) +
           (2 * qcap + kWaves * qcap + stats) * sizeof(float) +
           (global || over ? 0 : static_cast<size_t>(d.N) * sizeof(float));
}

template <typename T, typename Kern>
hipError_t launch_prob(Kern kern, size_t lds, const ProbArgs<T>& p, hipStream_t st) {
    if (lds > 64 * 1024) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             static_cast<int>(lds));
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(p.nblocks)), dim3(kThreads), lds, st, p);
    return hipGetLastError();
}

template <typename T, int D, int TG>
hipError_t launch_mp(const Dims& d, ProbArgs<T> p, hipStream_t st) {
    bool global = false;
    const size_t lds = mp_lds<T, D>(d, p.qcap, global, p.cols_over_stats);
    return global ? launch_prob(score_mean_prob_kernel<T, D, TG, true>, lds, p, st)
                  : launch_prob(score_mean_prob_kernel<T, D, TG, false>, lds, p, st);
}

template <typename T, int D, int QBN>
hipError_t launch_mp_resident(const Dims& d, ProbArgs<T> p, hipStream_t st) {
    bool global = false;
    const size_t two_pass = mp_lds<T, D>(d, p.qcap, global, p.cols_over_stats);
    const size_t lds = std::max(resident_lds<T, D, QBN>(), two_pass);
    return launch_prob(score_mean_prob_resident_kernel<T, D, QBN>, lds, p, st);
}

// The register-resident kernel takes a batch whose largest head qualifies and whose heads
// fill it: it runs kResTiles tiles per wave for every head, the two-pass kernel the head's
// own, at more each.  A contiguous eighth of the heads runs on each XCD (xcd_remap), so
// the fullest eighth decides: from an average of kResFill key tiles per head (of 36) there.
// 64 LLaVA-size images (bf16, 64 queries; us per call, two-pass / resident, near-uniform
// and unit-spread logits): 63 of 24 x 24 and one of 18 x 18 420 / 265; 6 of 24 x 24 and 58
// of 8 x 8 (28 tiles in the fullest eighth) 268 / 203 and 295 / 283; 4 and 60 (20 tiles)
// 214 / 186 and 240 / 284; one and 63 (8 tiles) 145 / 187 and 164 / 282; 16 of 24 x 24
// among 48 of 8 x 8 in turn (12 tiles) 187 / 202 and 206 / 284.
constexpr int64_t kXcds = 8, kResFill = 21;
bool takes_resident(const Dims& d) {
    if (!resident_head(d.NT, d.N)) return false;
    if (d.images_host == nullptr) return true;
    // eighth x: heads x B L H / 8 on, in units of an eighth of an image's
    int64_t tiles[kXcds] = {}, most = 0;
    for (int64_t b = 0; b < d.B; ++b) {
        const e2s_image& im = d.images_host[b];
        const int64_t t = (static_cast<int64_t>(im.grid_h) * im.grid_w + 15) / 16;
        for (int64_t x = kXcds * b / d.B; x < kXcds && x * d.B < kXcds * (b + 1); ++x)
            tiles[x] += t * (std::min((x + 1) * d.B, kXcds * (b + 1)) - std::max(x * d.B, kXcds * b));
    }
    for (int64_t t : tiles) most = std::max(most, t);
    return most >= kResFill * d.B;
}

template <typename T, int D>
hipError_t dispatch_mp(const Dims& d, float scale, const void* q, const void* k, float* e,
                       float* r, hipStream_t st) {
    using C = ProbCfg<T, D>;
    ProbArgs<T> p{};
    p.q = static_cast<const T*>(q);
    p.k = static_cast<const T*>(k);
    p.e_out = e;
    p.r_out = r;
    p.bg = batch_geom(d);
    p.group = static_cast<int>(d.group);
    p.scale = scale;
    p.nblocks = static_cast<int>(d.B * d.L * d.H);
    // qcap = min(QC, N_T rounded up to 16) query rows per chunk
    p.qcap = static_cast<int>(std::min<int64_t>(C::QC, (d.NT + 15) / 16 * 16));
    if constexpr (!std::is_same<T, float>::value) {
        if (takes_resident(d)) {
            switch ((d.NT + 15) / 16) {
                case 1: return launch_mp_resident<T, D, 1>(d, p, st);
                case 2: return launch_mp_resident<T, D, 2>(d, p, st);
                case 3: return launch_mp_resident<T, D, 3>(d, p, st);
                default: return launch_mp_resident<T, D, 4>(d, p, st);
            }
        }
    }
    if constexpr (std::is_same<T, float>::value) {
        return launch_mp<T, D, 1>(d, p, st);
    } else {
        // measured: 4 tiles per group pays when a chunk has 8 query blocks; one tile
        // per group (under 128 VGPRs: 4 workgroups per CU) up to 4 query blocks when
        // the LDS also leaves room for 4 (the LLaVA shape, before the register-resident
        // kernel took it: stage 413 -> 397 us), else 2 (Qwen2-VL, 6 query blocks: one
        // tile measured 276 -> 280 us, the queries' LDS reads per tile weighing more)
        if (p.qcap >= 128) return launch_mp<T, D, 4>(d, p, st);
        bool global = false, over = false;
        if (p.qcap <= 64 && 4 * mp_lds<T, D>(d, p.qcap, global, over) <= kLdsPerCu)
            return launch_mp<T, D, 1>(d, p, st);
        return launch_mp<T, D, 2>(d, p, st);
    }
}

}  // namespace

hipError_t launch_score_mean_prob(const Dims& d, int dtype, float scale, const void* q,
                                  const void* k, float* support_c, float* r_opt,
                                  hipStream_t stream) {
    if (dtype == E2S_DTYPE_BF16) {
        if (d.D == 128) return dispatch_mp<uint16_t, 128>(d, scale, q, k, support_c, r_opt, stream);
        return dispatch_mp<uint16_t, 64>(d, scale, q, k, support_c, r_opt, stream);
    }
    if (dtype == E2S_DTYPE_F16) {
        if (d.D == 128) return dispatch_mp<_Float16, 128>(d, scale, q, k, support_c, r_opt, stream);
        return dispatch_mp<_Float16, 64>(d, scale, q, k, support_c, r_opt, stream);
    }
    if (d.D == 128) return dispatch_mp<float, 128>(d, scale, q, k, support_c, r_opt, stream);
    return dispatch_mp<float, 64>(d, scale, q, k, support_c, r_opt, stream);
}

}  // namespace e2s
