// World Retrieval (paper Sec. 4.2, Eq. 4) with the camera/action distance of Sec. 5.1.
//
// One launch, fp64 throughout.  M is a few hundred for minute-long rollouts, a few thousand at most, so the step is bound
// by latency: launch, pose loads, one chain of trigonometry, two reductions, ranks.  Ranks are all-pairs counts of the
// (D, id) pairs that precede a candidate (broadcast reads from LDS), which gives the Top-k already ordered, with
// ties to the lower chunk id, and no sort.  They are what grows with M*M, so each workgroup ranks 16 candidates only
// -- a lane per candidate, each row of 16 lanes counting over its share of the others -- and works out all M distances for
// itself: that costs less than a second launch would.  One workgroup ranking everything with a thread per candidate took
// 7.4 / 47 / 662 us at M = 60 / 1,000 / 4,096; workgroups of 64 candidates (and reductions by shuffles) 3.8 / 9.1 / 24.8; with trigonometry of the
// library and the order of ids in every comparison 3.3 / 5.8 / 15.5; this takes 2.9 / 4.9 / 12.0 us, of which an empty launch is about 2.
#include <cmath>
#include <type_traits>

#include "wk_internal.h"

namespace {

constexpr int kThreads = 1024;

struct Pose5 { float v[5]; };

// The trigonometry of a distance on one compute unit, 1,000 times over, is what bounds the kernel, so it is written for what it has to do here: which
// quadrant an angle lies in only swaps squares, and of the two values whose squares sum to 1 the smaller one gives the angle, so that nothing is divided.
// With the library's sincos and atan2 1,000 candidates take 5.8 us, with this 5.1 (4,096: 15.6 and 13.1; four: 3.2 and 3.0).  Polynomials are Chebyshev interpolations in 60 digits of sin, cos and asin; their errors, relative, are
// below 2e-17.  Distances by rotation alone, over the largest (rms of 48 times 4,096 poses, and the largest error), with the library's functions and with this: yaws all round 5.2e-17 (2.5e-16) and
// 5.0e-17 (2.2e-16), many times round 5.5e-17 (2.8e-16) and 5.0e-17 (2.3e-16), beside a quarter turn 1.11e-16 (4.6e-16) and 1.03e-16 (4.2e-16), beside a half
// turn 6.4e-17 (1.9e-16) and 6.6e-17 (2.0e-16), where both are as exact as pi's last place, within 0.1 8.6e-17 and 6.6e-17, within 1e-4 9.3e-17 and 7.2e-17.
__device__ inline double horner(const double (&a)[19], double w) {
    double p = a[18];
#pragma unroll
    for (int k = 17; k >= 0; --k) p = fma(p, w, a[k]);
    return p;
}

// |sin x| and |cos x| up to sign.  Cody and Waite's reduction: by pi/2 in two parts, exact to 2^-106 of it, so for whole multiples below 2^20 (beyond, infinities
// and NaN: the library's)
__device__ inline void sin_cos(double x, double &s, double &c) {
    if (!(fabs(x) < 0x1p20)) {
        sincos(x, &s, &c);
        return;
    }
    const double n = __builtin_rint(x * 0.6366197723675814);
    const double near = fma(n, -1.5707963267948966, x), r = fma(n, -6.123233995736766e-17, near), rest = fma(n, -6.123233995736766e-17, near - r);
    const double w = r * r;
    double p = fma(w, 1.5918115263265974e-10, -2.505113165023518e-08);
    p = fma(p, w, 2.7557316101617874e-06);
    p = fma(p, w, -0.00019841269836756774);
    p = fma(p, w, 0.008333333333330948);
    p = fma(p, w, -0.16666666666666666);
    const double sn = fma(w * r, p, rest) + r;
    p = fma(w, -1.1382623647474604e-11, 2.087614614655861e-09);
    p = fma(p, w, -2.7557317271145144e-07);
    p = fma(p, w, 2.480158729876456e-05);
    p = fma(p, w, -0.0013888888888887398);
    p = fma(p, w, 0.041666666666666664);
    const double cs = 1.0 - fma(w, 0.5, -fma(w * w, p, -r * rest));
    const bool odd = (int)n & 1;
    s = odd ? cs : sn;
    c = odd ? sn : cs;
}

// square root of 0 or of a number that is nowhere near the ends of fp64's range, by Goldschmidt's iteration: root and half the inverse root side by side
__device__ inline double root(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return x == 0.0 ? 0.0 : g;
}

// Rotation angle of R_a^T R_b for R = R_y(yaw) R_x(pitch).  The relative rotation depends only on
// the yaw difference D and the pitch difference e:  cos(phi/2) = |cos(D/2) cos(e/2)|.  Evaluated
// from that or, where it is the smaller one, from sin^2(phi/2) = sin^2(D/2) + cos^2(D/2) sin^2(e/2),
// which stays accurate for small and for near-pi angles.
__device__ inline double geodesic(double yaw_a, double pitch_a, double yaw_b, double pitch_b) {
    constexpr double kAsin[19] = {   // asin(x) = x + x^3 * that of x^2, up to 1/2
        0.16666666666666669, 0.07499999999998404, 0.04464285714667406, 0.030381944083323155, 0.022372177086213967,
        0.017352219235510297, 0.01397577415595673, 0.011398660985318401, 0.011316548027917967, -0.0033341907871940585,
        0.07398716283974083, -0.28185916822883483, 0.9549127456157286, -2.359626130266744, 4.39509156816716,
        -5.895898686806016, 5.44685467754684, -3.100105228135179, 0.8399728912312339};
    double sD, cD, se, ce;
    sin_cos(0.5 * (yaw_b - yaw_a), sD, cD);
    sin_cos(0.5 * (pitch_b - pitch_a), se, ce);
    const double s = root(fma(sD, sD, cD * cD * (se * se))), c = fabs(cD * ce);
    const double x = s <= c ? s : c, w = x * x;
    // Both are rounded, and their squares then sum to 1 but for a rest, which is taken from the smaller one as an arctangent of both would: with y the larger one, by
    // least squares, x^2 / (x^4 + y^4) of it times the slope of asin, for which 2.5 x^2 stands here (1 % more error than with that itself).
    const double beyond = fma(s, s, fma(c, c, -1.0));
    const double rest = x * w * fma(-1.25, beyond, horner(kAsin, w));
    // pi, in two parts, less that or nothing: rounded once, what the difference loses goes to the small terms
    const double times = s <= c ? 2.0 : -2.0, from = s <= c ? 0.0 : 3.141592653589793, from_low = s <= c ? 0.0 : 1.2246467991473532e-16;
    const double near = fma(times, x, from);
    return near + (fma(times, rest, from_low) + fma(times, x, from - near));
}

enum { RED_MAX = 0, RED_MIN = 1, RED_SUM = 2 };

template <int OP>
__device__ inline double combine(double a, double b) {
    if constexpr (OP == RED_MAX) return fmax(a, b);
    else if constexpr (OP == RED_MIN) return fmin(a, b);
    else return a + b;
}

// reduces two values over the workgroup of WAVES waves, in a fixed order
template <int OP, int WAVES>
__device__ inline void block_reduce(double &x, double &y, double2 *scratch /*[WAVES]*/) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        x = combine<OP>(x, __shfl_xor(x, o));
        y = combine<OP>(y, __shfl_xor(y, o));
    }
    if constexpr (WAVES > 1) {
        __syncthreads();   // scratch may still be read from the reduction before
        if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = double2{x, y};
        __syncthreads();
        const double2 v = scratch[threadIdx.x % WAVES];
        x = v.x;
        y = v.y;
#pragma unroll
        for (int o = WAVES / 2; o >= 1; o >>= 1) {
            x = combine<OP>(x, __shfl_xor(x, o));
            y = combine<OP>(y, __shfl_xor(y, o));
        }
    }
}

__device__ inline double normalise(double v, int mode, double mx, double mn, double sum, int M) {
    if (mode == WK_NORM_MAX) return mx > 0.0 ? v / mx : 0.0;
    if (mode == WK_NORM_MINMAX) return mx > mn ? (v - mn) / (mx - mn) : 0.0;
    return sum > 0.0 ? v / (sum / (double)M) : 0.0;
}

// max or min over a row of 16 lanes, in all of them: rotations inside the vector pipe, where shuffles go through the LDS
template <int OP>
__device__ inline double row_reduce(double x) {
    auto rotated = [](double v, auto by) {
        const long long b = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x120 + decltype(by)::value, 0xf, 0xf, false);
        const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x120 + decltype(by)::value, 0xf, 0xf, false);
        return __longlong_as_double((long long)(unsigned)lo | (long long)hi << 32);
    };
    x = combine<OP>(x, rotated(x, std::integral_constant<int, 8>{}));
    x = combine<OP>(x, rotated(x, std::integral_constant<int, 4>{}));
    x = combine<OP>(x, rotated(x, std::integral_constant<int, 2>{}));
    return combine<OP>(x, rotated(x, std::integral_constant<int, 1>{}));
}

// the same for max and min, whose order is free: rows of 16 lanes first, and every thread over the rows
template <int OP, int WAVES>
__device__ inline void block_extreme(double &x, double &y, double2 *scratch /*[4 * WAVES]*/) {
    x = row_reduce<OP>(x);
    y = row_reduce<OP>(y);
    __syncthreads();   // scratch may still be read from the reduction before
    if ((threadIdx.x & 15) == 0) scratch[threadIdx.x >> 4] = double2{x, y};
    __syncthreads();
#pragma unroll
    for (int r = 0; r < WAVES / 4; ++r) {
        const double2 v = scratch[16 * r + (threadIdx.x & 15)];
        x = r ? combine<OP>(x, v.x) : v.x;
        y = r ? combine<OP>(y, v.y) : v.y;
    }
    x = row_reduce<OP>(x);
    y = row_reduce<OP>(y);
}

constexpr int kRankPerBlock = 16;   // candidates a workgroup ranks

// workgroups of WAVES waves, up to PER_THREAD candidates per thread: WAVES * 64 * PER_THREAD >= M
template <int WAVES, int PER_THREAD>
__global__ __launch_bounds__(WAVES * 64) void k_score_chunks(const float *__restrict__ poses, int M, Pose5 cur,
                                                             int norm_mode, int R, int32_t *__restrict__ ids_out,
                                                             double *__restrict__ dist_out,
                                                             int32_t *__restrict__ n_found) {
    constexpr int THREADS = WAVES * 64;
    __shared__ __attribute__((aligned(16))) double D[THREADS * PER_THREAD];
    __shared__ double2 scratch[4 * WAVES];
    __shared__ int part[WAVES][kRankPerBlock];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int found = R < M ? R : M;
    if (blockIdx.x == 0) {
        if (tid == 0) *n_found = found;
        for (int r = found + tid; r < R; r += THREADS) {
            ids_out[r] = -1;
            if (dist_out) dist_out[r] = INFINITY;
        }
    }
    if (M == 0 || R == 0) return;

    double dt[PER_THREAD], dr[PER_THREAD];
    double t_max = 0.0, t_min = INFINITY, t_sum = 0.0, r_max = 0.0, r_min = INFINITY, r_sum = 0.0;
#pragma unroll
    for (int e = 0; e < PER_THREAD; ++e) {
        const int i = tid + e * THREADS;
        dt[e] = dr[e] = 0.0;
        if (i < M) {
            const float *a = poses + (size_t)i * 5;
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double df = (double)cur.v[c] - (double)a[c];
                s += df * df;
            }
            dt[e] = s;
            dr[e] = geodesic((double)cur.v[3], (double)cur.v[4], (double)a[3], (double)a[4]);
            t_max = fmax(t_max, dt[e]); t_min = fmin(t_min, dt[e]); t_sum += dt[e];
            r_max = fmax(r_max, dr[e]); r_min = fmin(r_min, dr[e]); r_sum += dr[e];
        }
    }
    if (norm_mode != WK_NORM_MEAN) block_extreme<RED_MAX, WAVES>(t_max, r_max, scratch);
    if (norm_mode == WK_NORM_MINMAX) block_extreme<RED_MIN, WAVES>(t_min, r_min, scratch);
    if (norm_mode == WK_NORM_MEAN) block_reduce<RED_SUM, WAVES>(t_sum, r_sum, scratch);
#pragma unroll
    for (int e = 0; e < PER_THREAD; ++e) {
        const int i = tid + e * THREADS;
        D[i] = i < M ? normalise(dt[e], norm_mode, t_max, t_min, t_sum, M) + normalise(dr[e], norm_mode, r_max, r_min, r_sum, M)
                     : INFINITY;   // behind all others
    }
    __syncthreads();
    // a lane's candidate, in every row of 16 lanes; the rows share the others, two at a time
    const int i = blockIdx.x * kRankPerBlock + (lane & 15), row = tid >> 4;
    const double di = i < M ? D[i] : INFINITY;
    int rank = 0;
    // In front of the workgroup's candidates a distance precedes theirs if it is not larger, behind them if it is smaller: one comparison each, where
    // asking for the order of ids too takes five instructions.  (unrolled: the reads of several distances are in flight at once, where one read per trip
    // took 140 cycles)
    constexpr int kApart = 2 * (THREADS / 16);
    const int first = blockIdx.x * kRankPerBlock;
    int j = 2 * row;
#pragma unroll 4
    for (; j < first; j += kApart) {
        const double2 dj = *reinterpret_cast<const double2 *>(D + j);
        rank += (dj.x <= di ? 1 : 0) + (dj.y <= di ? 1 : 0);
    }
    if (j < first + kRankPerBlock) {   // (a row has a pair of the workgroup's own at most)
        const double2 dj = *reinterpret_cast<const double2 *>(D + j);
        rank += (dj.x < di || (dj.x == di && j < i)) ? 1 : 0;
        rank += (dj.y < di || (dj.y == di && j + 1 < i)) ? 1 : 0;
        j += kApart;
    }
#pragma unroll 4
    for (; j < M; j += kApart) {
        const double2 dj = *reinterpret_cast<const double2 *>(D + j);
        rank += (dj.x < di ? 1 : 0) + (dj.y < di ? 1 : 0);
    }
    rank += __shfl_xor(rank, 16);
    rank += __shfl_xor(rank, 32);
    if (lane < 16) part[wave][lane] = rank;
    __syncthreads();
    if (tid >= 16) return;
    rank = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) rank += part[w][lane];
    if (i < M && rank < found) {
        ids_out[rank] = i;
        if (dist_out) dist_out[rank] = di;
    }
}

}  // namespace

extern "C" wk_status wk_score_chunks(const float *poses, int32_t M, const float *cur_pose, int32_t norm_mode,
                                     int32_t R, int32_t *ids_out, double *dist_out, int32_t *n_found,
                                     void *hip_stream) {
    if (M < 0 || R < 0 || !cur_pose || !n_found) return WK_ERR_INVALID_ARG;
    if (M > 0 && !poses) return WK_ERR_INVALID_ARG;
    if (R > 0 && !ids_out) return WK_ERR_INVALID_ARG;
    if (norm_mode != WK_NORM_MAX && norm_mode != WK_NORM_MINMAX && norm_mode != WK_NORM_MEAN)
        return WK_ERR_INVALID_ARG;
    if (M > WK_SCORE_MAX_CHUNKS) return WK_ERR_UNSUPPORTED;
    Pose5 cur;
    for (int c = 0; c < 5; ++c) cur.v[c] = cur_pose[c];
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    const dim3 grid(M > 0 ? (M + kRankPerBlock - 1) / kRankPerBlock : 1);
    // sixteen waves share the distances and the ranking's all-pairs count best (M = 256: 3.8 us); up to 128 candidates four waves are
    // enough and meet at the barriers sooner (M = 128: 3.5 us)
    auto launch = [&](auto waves, auto per_thread) {
        constexpr int W = decltype(waves)::value, P = decltype(per_thread)::value;
        hipLaunchKernelGGL((k_score_chunks<W, P>), grid, dim3(W * 64), 0, st, poses, (int)M, cur, (int)norm_mode, (int)R,
                           ids_out, dist_out, n_found);
    };
    if (M <= 128) launch(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
    else if (M <= 1024) launch(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{});
    else launch(std::integral_constant<int, 16>{}, std::integral_constant<int, 4>{});
    WK_LAUNCH_CHECK();
    return WK_OK;
}

// ---- query-based retrieval (paper Sec. 4.2, App. C) -------------------------------------------------
//
// Input: lse[c][r] = log sum_k exp(q_r . k / sqrt(d)) over the keys k of stored chunk c, for every
// (head, query) row r -- what wk_attention writes as `lse` when run over one chunk.  In a softmax
// over the keys of all M chunks, chunk c receives mass exp(lse[c][r] - logsumexp_c' lse[c'][r]) from
// row r; the relevance of a chunk is the mean of that mass over the rows.  fp64 throughout.
namespace {

constexpr int kQThreads = 256;
constexpr int kQBatch = 8;   // chunks whose values a lane has in flight

// sum over the wave's lanes, in all of them: the tree of __shfl_xor(x, 32), 16, .. 1, without its ways through the LDS
__device__ inline double wave_sum(double x) {
    auto split = [](double v, unsigned &lo, unsigned &hi) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(v);
        lo = (unsigned)b;
        hi = (unsigned)(b >> 32);
    };
    auto join = [](unsigned lo, unsigned hi) { return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo)); };
    unsigned lo, hi;
    split(x, lo, hi);
    auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), c = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    x = join(a[0], c[0]) + join(a[1], c[1]);
    split(x, lo, hi);
    a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    c = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    x = join(a[0], c[0]) + join(a[1], c[1]);
    auto rotated = [&](auto by) {   // inside a row of 16 lanes, whose halves, quarters, .. are alike by then
        constexpr int kRor = 0x120 + decltype(by)::value;
        split(x, lo, hi);
        return join((unsigned)__builtin_amdgcn_mov_dpp((int)lo, kRor, 0xf, 0xf, false), (unsigned)__builtin_amdgcn_mov_dpp((int)hi, kRor, 0xf, 0xf, false));
    };
    x += rotated(std::integral_constant<int, 8>{});
    x += rotated(std::integral_constant<int, 4>{});
    x += rotated(std::integral_constant<int, 2>{});
    return x + rotated(std::integral_constant<int, 1>{});
}

// A lane per row, three walks over the chunks: the largest, the sum of exponentials, the masses.  Three waves a SIMD do not cover the latency of one load
// at a time, so a lane has eight; and a wave's sum of a chunk's masses stays in the vector pipe.  With both
// kernels: 120 chunks of 187,200 rows 174 -> 98 us (16 of them the second kernel's), 400 of 187,200 727 -> 328, 400 of 20,000 454 -> 202, 60 of 31,680
// 50 -> 30, bit for bit the same (with sixteen loads 104, 320, 181 and 30).
__global__ __launch_bounds__(kQThreads) void k_query_mass_partial(const float *__restrict__ lse, int M,
                                                                  long long n_rows, double *__restrict__ partial) {
    __shared__ double acc[kQThreads / 64][WK_QUERY_MAX_CHUNKS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int c = lane; c < M; c += 64) acc[wave][c] = 0.0;
    // (each wave only touches its own row of acc: no barrier needed until the end)
    for (long long r0 = (long long)blockIdx.x * kQThreads; r0 < n_rows; r0 += (long long)gridDim.x * kQThreads) {
        const bool ok = r0 + tid < n_rows;
        const float *row = lse + (ok ? r0 + tid : n_rows - 1);
        auto walk = [&](auto use) {   // use(values, first chunk): chunks behind the last one repeat it
            for (int c0 = 0; c0 < M; c0 += kQBatch) {
                float v[kQBatch];
#pragma unroll
                for (int u = 0; u < kQBatch; ++u) v[u] = row[(size_t)min(c0 + u, M - 1) * n_rows];
                use(v, c0);
            }
        };
        double mx = -INFINITY;
        walk([&](const float (&v)[kQBatch], int) {
#pragma unroll
            for (int u = 0; u < kQBatch; ++u) mx = fmax(mx, (double)v[u]);
        });
        double sum = 0.0;
        if (mx > -INFINITY)
            walk([&](const float (&v)[kQBatch], int c0) {
#pragma unroll
                for (int u = 0; u < kQBatch; ++u) {
                    const double e = exp((double)v[u] - mx);
                    if (c0 + u < M) sum += e;
                }
            });
        const double L = mx + log(sum);   // -inf or NaN for rows that see no key at all: they are skipped
        const bool counts = ok && sum > 0.0;
        walk([&](const float (&v)[kQBatch], int c0) {
#pragma unroll
            for (int u = 0; u < kQBatch; ++u) {
                const double w = wave_sum(counts ? exp((double)v[u] - L) : 0.0);
                if (lane == 0 && c0 + u < M) acc[wave][c0 + u] += w;
            }
        });
    }
    __syncthreads();
    for (int c = tid; c < M; c += kQThreads) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kQThreads / 64; ++w) s += acc[w][c];
        partial[(size_t)c * gridDim.x + blockIdx.x] = s;   // (k_query_topk reads a chunk's sums side by side)
    }
}

// mass[c] = sum of the blocks' partial sums / n_rows; the min(R, M) largest, ties to the lower id
__global__ __launch_bounds__(kThreads) void k_query_topk(const double *__restrict__ partial, int n_blocks, int M,
                                                         long long n_rows, int R, double *__restrict__ mass_all,
                                                         int32_t *__restrict__ ids_out,
                                                         double *__restrict__ mass_out,
                                                         int32_t *__restrict__ n_found) {
    __shared__ double mass[WK_QUERY_MAX_CHUNKS];
    const int tid = threadIdx.x;
    const int found = R < M ? R : M;
    if (tid == 0) *n_found = found;
    for (int r = found + tid; r < R; r += kThreads) {
        ids_out[r] = -1;
        if (mass_out) mass_out[r] = -INFINITY;
    }
    if (M == 0) return;
    // one wave per chunk: lanes sum interleaved blocks, then a fixed-shape tree over the lanes.  Up to 16 blocks per lane
    // (1024 in all), requested eight at a time: 120 chunks of 732 blocks 16 us, 36 us one by one and M doubles apart.
    for (int c = tid >> 6; c < M; c += kThreads / 64) {
        const double *mine = partial + (size_t)c * n_blocks;
        double s = 0.0;
        for (int b = tid & 63; b < n_blocks; b += 8 * 64) {
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = b + u * 64 < n_blocks ? mine[b + u * 64] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) s += t[u];
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        s /= (double)n_rows;
        if ((tid & 63) == 0) {
            mass[c] = s;
            mass_all[c] = s;
        }
    }
    __syncthreads();
    for (int c = tid; c < M; c += kThreads) {
        const double mc = mass[c];
        int rank = 0;
        for (int j = 0; j < M; ++j) {
            const double mj = mass[j];
            rank += (mj > mc || (mj == mc && j < c)) ? 1 : 0;
        }
        if (rank < found) {
            ids_out[rank] = c;
            if (mass_out) mass_out[rank] = mc;
        }
    }
}

int query_blocks(long long n_rows) {
    const long long b = (n_rows + kQThreads - 1) / kQThreads;
    return (int)(b < 1 ? 1 : (b > 1024 ? 1024 : b));
}

}  // namespace

extern "C" size_t wk_score_chunks_query_workspace_bytes(int32_t M, int64_t n_rows) {
    if (M < 0 || M > WK_QUERY_MAX_CHUNKS || n_rows < 1) return 0;
    const size_t m = (size_t)(M > 0 ? M : 1);
    return wk::align_up(m * sizeof(double), 256) + wk::align_up((size_t)query_blocks(n_rows) * m * sizeof(double), 256);
}

extern "C" wk_status wk_score_chunks_query(const float *lse, int32_t M, int64_t n_rows, int32_t R, int32_t *ids_out,
                                           double *mass_out, int32_t *n_found, void *workspace,
                                           size_t workspace_bytes, void *hip_stream) {
    if (M < 0 || R < 0 || n_rows < 1 || !n_found) return WK_ERR_INVALID_ARG;
    if (M > 0 && !lse) return WK_ERR_INVALID_ARG;
    if (R > 0 && !ids_out) return WK_ERR_INVALID_ARG;
    if (M > WK_QUERY_MAX_CHUNKS) return WK_ERR_UNSUPPORTED;
    const size_t need = wk_score_chunks_query_workspace_bytes(M, n_rows);
    if (!workspace || workspace_bytes < need || reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return WK_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    double *mass_all = reinterpret_cast<double *>(workspace);
    double *partial = reinterpret_cast<double *>(reinterpret_cast<char *>(workspace) +
                                                 wk::align_up((size_t)(M > 0 ? M : 1) * sizeof(double), 256));
    const int nb = query_blocks(n_rows);
    if (M > 0) {
        hipLaunchKernelGGL(k_query_mass_partial, dim3(nb), dim3(kQThreads), 0, st, lse, (int)M, (long long)n_rows,
                           partial);
        WK_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_query_topk, dim3(1), dim3(kThreads), 0, st, partial, nb, (int)M, (long long)n_rows, (int)R,
                       mass_all, ids_out, mass_out, n_found);
    WK_LAUNCH_CHECK();
    return WK_OK;
}

extern "C" wk_status wk_accumulate_actions(const int32_t *labels, int32_t n, float step, float dangle,
                                           float pitch_limit, float *poses_out) {
    if (n < 0 || (n > 0 && (!labels || !poses_out))) return WK_ERR_INVALID_ARG;
    for (int i = 0; i < n; ++i)
        if (labels[i] < 0 || labels[i] > 7) return WK_ERR_INVALID_ARG;
    // state in double; the table of per-label increments keeps the loop branch-free
    double pos[3] = {0, 0, 0}, yaw = 0, pitch = 0;
    const double st = step, da = dangle, lim = pitch_limit;
    static const double fwd_c[8] = {1, 0, -1, 0, 0, 0, 0, 0};    // along the heading
    static const double right_c[8] = {0, -1, 0, 1, 0, 0, 0, 0};  // along the right vector
    static const double yaw_c[8] = {0, 0, 0, 0, -1, 1, 0, 0};
    static const double pitch_c[8] = {0, 0, 0, 0, 0, 0, -1, 1};
    for (int i = 0; i < n; ++i) {
        const int a = labels[i];
        const double sy = std::sin(yaw), cy = std::cos(yaw);
        pos[0] += st * (fwd_c[a] * sy + right_c[a] * cy);
        pos[2] += st * (fwd_c[a] * cy - right_c[a] * sy);
        yaw += da * yaw_c[a];
        pitch = std::fmin(lim, std::fmax(-lim, pitch + da * pitch_c[a]));
        float *o = poses_out + (size_t)i * 5;
        o[0] = (float)pos[0]; o[1] = (float)pos[1]; o[2] = (float)pos[2];
        o[3] = (float)yaw; o[4] = (float)pitch;
    }
    return WK_OK;
}
