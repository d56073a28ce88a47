// diag.hip -- rank-1 friction diagnostic on gfx950.
//
// Section 4 of the paper ("How Close is xi~ to the Best Rank-1 Friction?")
// runs iKFAD0 while updating R-iKFAD's factors R, C as shadow states fed by
// the same P^(1), then compares the full friction xi with the rank-1
// xi~ = R C^T / (1^T R + eps) against the Eckart-Young floor
// sqrt(1 - sigma_1^2 / |xi|_F^2), and reports the stable rank
// |xi|_F^2 / sigma_1^2.  Both xi and the shadow factors obey the same
// linear filter driven by [P^(1)]^2, so from R = C = xi = 0 the shadows are
// exactly R = xi 1 and C = xi^T 1: this file computes them from xi directly.
//
// Every quantity is a deterministic reduction (fixed partition, fixed
// order): row sums in a wave (or the waves of a workgroup that share the row),
// column sums per workgroup down its rows (row stripes for n > 16384) then
// folded in their order, squared norms per workgroup then folded in order.
// sigma_1 comes from power iteration on xi^T xi started at C / |C| (xi >= 0,
// so the leading singular vectors are non-negative), normalised on the GPU:
// the column fold also writes per-workgroup squared-norm partials, from
// which every wave of the next pass derives the same scale.  For
// n <= 16384 every pass reads xi once (u = xi v and xi^T u together).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <mutex>
#include <string>

#include "../../include/rikfad.h"
#include "kernels.hpp"
#include "lanes.hpp"

namespace {

using rk::add_half32;
using rk::add_row16;
using rk::dpp;
using rk::kQuadXor1;
using rk::kQuadXor2;
using rk::kRor4;
using rk::kRor8;

constexpr int kT = 256;            // threads per workgroup
constexpr int kStatChunk = 4096;   // elements per workgroup of the vector statistics
constexpr int kErrRows = 16;       // rows per workgroup of the error pass
constexpr int kFoldCols = 16;                       // columns per workgroup of the column fold
constexpr int kFoldGroups = kT / kFoldCols;         // partial-sum groups per column

#define DG __attribute__((address_space(1)))
template <typename T> __device__ __forceinline__ const DG T *gp(const T *q) { return (const DG T *)q; }
template <typename T> __device__ __forceinline__ DG T *gp(T *q) { return (DG T *)q; }

// Wave-level sum in a fixed butterfly order (every lane gets the same bits).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o);
    return v;
}

// t where c holds, else +0.  A bitwise mask rather than a select: a select
// between a loaded value and 0 is compiled into a branch around the load.
__device__ __forceinline__ float keep_if(bool c, float t)
{
    return __uint_as_float(__float_as_uint(t) & (c ? 0xffffffffu : 0u));
}
__device__ __forceinline__ double keep_if(bool c, double t)
{
    return __longlong_as_double(__double_as_longlong(t) & (c ? ~0ll : 0ll));
}

// sum_q parts[2 q] in a fixed order (lanes stride over the partials, 8 loads
// in flight, then the butterfly); every wave that calls it gets the same
// bits.
__device__ __forceinline__ double sum_parts(const double *__restrict__ parts, int nparts)
{
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    for (int q0 = lane; q0 < nparts; q0 += 64 * 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int q = q0 + 64 * u;
            v[u] = keep_if(q < nparts, gp(parts)[2 * static_cast<int64_t>(min(q, nparts - 1))]);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    return wave_sum(s);
}

// Scale of a vector from its fold partials: 1 / norm, 0 for a zero vector.
__device__ __forceinline__ double inv_norm(const double *__restrict__ parts, int nparts)
{
    const double s = sum_parts(parts, nparts);
    return s > 0.0 ? 1.0 / sqrt(s) : 0.0;
}

// out[i] = sum_j xi[i, j] * (w ? w[j] * scale : 1) with scale = inv_norm of
// w's fold partials: one wave per row, lanes stride over the columns, fp64
// accumulation.
__global__ __launch_bounds__(kT) void row_reduce_kernel(const float *__restrict__ xi, int64_t m,
                                                        int64_t n, const double *__restrict__ w,
                                                        const double *__restrict__ wparts,
                                                        int nwparts, double *__restrict__ out)
{
    const int64_t row = static_cast<int64_t>(blockIdx.x) * (kT / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= m) return;
    const double scale = w ? inv_norm(wparts, nwparts) : 1.0;
    const DG float *xr = gp(xi) + row * n;
    double s = 0.0;
    // Eight loads in flight per lane; additions in column order.
    for (int64_t j0 = lane; j0 < n; j0 += 64 * 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t j = j0 + 64 * u;
            const int64_t jc = j < n ? j : n - 1;         // in the row; masked below
            v[u] = keep_if(j < n, static_cast<double>(xr[jc]) * (w ? gp(w)[jc] : 1.0));
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    s = wave_sum(s);
    if (lane == 0) gp(out)[row] = w ? s * scale : s;
}

// ------------------------------------------------- wave-level sums in VALU
//
// A butterfly through __shfl_xor would be a chain of LDS-crossbar round trips,
// which the one-pass kernels cannot hide.

// Lane 0's value, as a scalar.
__device__ __forceinline__ double first_lane(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// The sum of v over the 64 lanes, as a scalar.
__device__ __forceinline__ double wave_sum_valu(double v)
{
    v += dpp<kQuadXor1>(v);
    v += dpp<kQuadXor2>(v);
    v += dpp<kRor8>(v);
    v += dpp<kRor4>(v);
    return first_lane(add_half32(add_row16(v)));
}

// Sum over the W waves of a row of their partial sums, lane l holding that of
// wave l mod W, as a scalar.
template <int W>
__device__ __forceinline__ double sum_waves(double v)
{
    static_assert(W == 4 || W == 8 || W == 16, "waves per row");
    if (W == 16) v += dpp<kRor8>(v);
    if (W >= 8) v += dpp<kRor4>(v);
    v += dpp<kQuadXor2>(v);
    v += dpp<kQuadXor1>(v);
    return first_lane(v);
}

// ---------------------------------------------------------- one-pass kernels
//
// One pass over xi for n <= 16384, reading it once.  WPR of a workgroup's 16
// waves cover a row with K 16-byte loads per lane (V = 4; V = 1, one 4-byte
// load, for rows of fewer than 4 columns), so 16 / WPR groups of waves work on
// consecutive shares of the workgroup's rows.  A lane keeps its V K columns'
// weights and column sums in registers; for each row it
// forms its share of the weighted sum s_i = sum_j xi[i, j] w_j, the sum is
// completed in the wave (across WPR waves through LDS), and xi[i, j] s_i is
// added to the column sums, rows in order.  The next row's loads go out
// before the current one is summed.  The groups' column sums are added in
// order into the workgroup's row of part (folded by col_fold_kernel).  MODE:
//   kPassSums      part holds column sums of xi (C); no weights
//   kPassPower     w = v / |v| (scale from v's fold partials): s = u, and
//                  part holds xi^T u
//   kPassPowerErr  the same from v = C, not normalised, plus spart =
//                  (sum xi^2, sum (xi - xi~)^2) with xi~_ij = R_i C_j /
//                  (1^T R + eps) (0 if that is 0), R_i the row's own sum and
//                  1^T R the sum of C's fold partials
//   kPassNorm      w as kPassPower; spart[0] = sum s_i^2, no column sums
//
// What bounds it: reading xi (7.2 TB/s at best here, from the memory-side
// cache or from HBM alike), plus a prologue, an epilogue and a fold launch
// of a few us each per pass.  One 16-wave workgroup per compute unit and at
// most 256 of them fill the chip in one round and bound the partial sums to
// 256 rows.  Report with 30 iterations, against one wave per row of up to
// 1024 columns with 4-byte loads and LDS-crossbar sums, and two passes per
// iteration above (same box): 50257 x 768 1080 -> 1000 us, 40000 x 1000
// 1250 -> 1075, 768 x 768 864 -> 340, 20000 x 1500 1870 -> 1015,
// 4096 x 11008 3020 -> 1390.  Two or four rows per batch measured within 2%
// of one (50257 x 768: 1070 with two), and with spilled registers far
// slower (4096 x 11008 with two rows: 1790; 40000 x 1000: 1970).
enum : int { kPassSums = 0, kPassPower = 1, kPassPowerErr = 2, kPassNorm = 3 };

// Rows of xi start at any 4-byte boundary when n is not a multiple of 4.
typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x1 __attribute__((ext_vector_type(1)));
template <int V> struct RowAccess { typedef f32x4a4 type; };
template <> struct RowAccess<1> { typedef f32x1 type; };

typedef double f64x2 __attribute__((ext_vector_type(2)));

struct OnePass {
    const float *xi;
    int64_t m, n;
    int rows;                       // rows per workgroup
    int nvparts;
    const double *v, *vparts;
    double eps;
    double *part, *spart;
    int64_t stride;                 // doubles per row of part (n rounded up to 4)
};

constexpr int kPassWaves = 16;

template <int K, int WPR, int MODE, int V = 4>
__global__ __launch_bounds__(64 * kPassWaves) void onepass_kernel(OnePass a)
{
    static_assert(V == 4 || (V == 1 && K == 1 && WPR == 1), "one column per lane: one wave per row");
    constexpr bool kWeighted = MODE != kPassSums;
    constexpr bool kErr = MODE == kPassPowerErr;
    constexpr bool kCols = MODE != kPassNorm;
    constexpr int NW = kPassWaves, LT = 64 * WPR, NG = NW / WPR;
    __shared__ double lds[NG > 1 ? NG * V * K * LT : 1];
    __shared__ double rowsum[2][WPR > 1 ? NG : 1][WPR], rowsum1[2][WPR > 1 ? NG : 1][WPR];
    __shared__ double ls[NW][2];
    const int lane = threadIdx.x & 63;
    // Scalar, so that row addresses are computed once per wave, not per lane
    // (768 x 768: 375 -> 353 us per report, 200000 x 256 1379 -> 1292,
    // 50257 x 768 1051 -> 1023).
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = wave % WPR, grp = wave / WPR;
    const int lt = sub * 64 + lane;
    const int n = static_cast<int>(a.n);

    // Columns V (lt + k LT) .. + V - 1.  Only the last load can pass the row's
    // end: it then reads the row's last V elements and masks the ones
    // that another lane owns (all of them where none is left).
    int lc[K];
    uint32_t keep[V];
#pragma unroll
    for (int k = 0; k < K; ++k) lc[k] = min(V * (lt + k * LT), n - V);
    const int skip = min(V * (lt + (K - 1) * LT) - lc[K - 1], V);
#pragma unroll
    for (int i = 0; i < V; ++i) keep[i] = i >= skip ? 0xffffffffu : 0u;

    const int64_t wg0 = static_cast<int64_t>(blockIdx.x) * a.rows;
    const int share = (a.rows + NG - 1) / NG;
    const int64_t r0 = wg0 + static_cast<int64_t>(grp) * share;
    const int64_t rend = min(min(r0 + share, wg0 + a.rows), a.m);
    const int nr = static_cast<int>(max<int64_t>(0, rend - r0));
    const int64_t rlast = nr > 0 ? rend - 1 : a.m - 1;  // a row of xi

    // Row q of the group's share; past its last, the last again.
    typedef typename RowAccess<V>::type access;
    auto load = [&](int q, access (&x)[K]) {
        const DG float *xr = gp(a.xi) + min(r0 + q, rlast) * a.n;
#pragma unroll
        for (int k = 0; k < K; ++k) x[k] = *reinterpret_cast<const DG access *>(xr + lc[k]);
    };

    // The first row goes out ahead of the weights' loads, so that the two
    // chains overlap.
    access nx[K];
    load(0, nx);

    double w[K][V], acc[K][V];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < V; ++i) {
            w[k][i] = kWeighted ? gp(a.v)[lc[k] + i] : 1.0;
            acc[k][i] = 0.0;
        }
    if (kWeighted && !kErr) {
        const double scale = inv_norm(a.vparts, a.nvparts);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < V; ++i) w[k][i] *= scale;
    }
    double inv = 0.0;
    if (kErr) {
        const double denom = sum_parts(a.vparts + 1, a.nvparts) + a.eps;
        inv = denom == 0.0 ? 0.0 : 1.0 / denom;
    }

    double sa = 0.0, sb = 0.0;
    for (int q = 0; q < share; ++q) {           // the same count in every group
        float x[K][V];
        const uint32_t ok = q < nr ? 0xffffffffu : 0u;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < V; ++i)
                x[k][i] = __uint_as_float(__float_as_uint(nx[k][i]) &
                                          (k == K - 1 ? ok & keep[i] : ok));
        load(q + 1, nx);
        double s = 0.0, s1 = 0.0;
        if (kWeighted) {
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    s += static_cast<double>(x[k][i]) * w[k][i];
                    if (kErr) s1 += static_cast<double>(x[k][i]);
                }
            s = wave_sum_valu(s);
            if (kErr) s1 = wave_sum_valu(s1);
            if constexpr (WPR > 1) {
                const int slot = q & 1;         // two slots: one barrier per row
                if (lane == 0) {
                    rowsum[slot][grp][sub] = s;
                    if (kErr) rowsum1[slot][grp][sub] = s1;
                }
                __syncthreads();
                s = sum_waves<WPR>(rowsum[slot][grp][lane & (WPR - 1)]);
                if (kErr) s1 = sum_waves<WPR>(rowsum1[slot][grp][lane & (WPR - 1)]);
            }
        }
        if (MODE == kPassNorm) sa += s * s;
        const double ri = kErr ? s1 * inv : 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const double xv = x[k][i];
                if (kCols) acc[k][i] += kWeighted ? xv * s : xv;
                if (kErr) {
                    // masked columns hold xi = 0: their model value goes too
                    const bool own = k < K - 1 || keep[i] != 0u;
                    const double e = own ? xv - ri * w[k][i] : 0.0;
                    sa += xv * xv;
                    sb += e * e;
                }
            }
    }

    if (kCols) {
        double *out = a.part + static_cast<int64_t>(blockIdx.x) * a.stride;
        if (NG > 1) {
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < V; ++i) lds[(grp * K + k) * V * LT + V * lt + i] = acc[k][i];
            __syncthreads();
            for (int j = threadIdx.x; j < V * K * LT; j += 64 * NW) {
                double t = lds[j];
#pragma unroll
                for (int g = 1; g < NG; ++g) t += lds[g * K * V * LT + j];
                // slot j is element i of the lane whose first column is j - i
                const int i = j & (V - 1), c0 = j - i, d = min(c0 - min(c0, n - V), V);
                if (i >= d) gp(out)[c0 - d + i] = t;
            }
        } else if constexpr (V == 4) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k < K - 1 || skip == 0) {       // whole groups of 4: 32-byte aligned
                    DG f64x2 *q = reinterpret_cast<DG f64x2 *>(gp(out) + lc[k]);
                    q[0] = f64x2{acc[k][0], acc[k][1]};
                    q[1] = f64x2{acc[k][2], acc[k][3]};
                } else {
#pragma unroll
                    for (int i = 0; i < V; ++i)
                        if (keep[i] != 0u) gp(out)[lc[k] + i] = acc[k][i];
                }
            }
        }
    }
    if (kErr || MODE == kPassNorm) {
        if (kErr) {
            sa = wave_sum(sa);
            sb = wave_sum(sb);
        }
        if (lane == 0) {
            ls[wave][0] = sa;
            ls[wave][1] = sb;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            // of kPassNorm's s_i^2 every wave of a row's group holds the same sum
            double x2 = 0.0, e2 = 0.0;
            for (int t = 0; t < NW; t += MODE == kPassNorm ? WPR : 1) {
                x2 += ls[t][0];
                e2 += ls[t][1];
            }
            gp(a.spart)[2 * blockIdx.x] = x2;
            gp(a.spart)[2 * blockIdx.x + 1] = e2;
        }
    }
}

// part[s, j] = sum over rows i of stripe s of xi[i, j] * (w ? w[i] : 1).
__global__ __launch_bounds__(kT) void col_partial_kernel(const float *__restrict__ xi, int64_t m,
                                                         int64_t n, int64_t stripe,
                                                         const double *__restrict__ w,
                                                         double *__restrict__ part)
{
    const int64_t j = static_cast<int64_t>(blockIdx.x) * kT + threadIdx.x;
    const int64_t s = blockIdx.y;
    if (j >= n) return;
    const int64_t i0 = s * stripe;
    const int64_t i1 = i0 + stripe < m ? i0 + stripe : m;
    double acc = 0.0;
    // Sixteen rows in flight per thread; additions in row order.
    for (int64_t ib = i0; ib < i1; ib += 16) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int64_t i = ib + u;
            const int64_t ic = i < i1 ? i : i1 - 1;       // in the stripe; masked below
            v[u] = keep_if(i < i1, static_cast<double>(gp(xi)[ic * n + j]) * (w ? gp(w)[ic] : 1.0));
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += v[u];
    }
    gp(part)[s * n + j] = acc;
}

// out[j] = sum_s part[s * stride + j] for j < n: a workgroup takes kFoldCols
// columns; each of its kFoldGroups groups of 16 threads sums a consecutive
// range of the partial sums in order (16 loads in flight, addresses clamped
// and values masked), the groups of a wave are added by a butterfly and the
// waves in order.  The workgroup also writes parts[2 b] = sum of out[j]^2 and
// parts[2 b + 1] = sum of out[j] over its columns, the partials inv_norm and
// the statistics use.  Latency-bound (1.6 MB of partial sums for 768
// columns): with 64 groups added one by one through LDS by a few threads it
// took 4.8 us, of which that chain of LDS reads was about half.
__global__ __launch_bounds__(kT) void col_fold_kernel(const double *__restrict__ part,
                                                      int64_t stride, int64_t n, int nparts,
                                                      double *__restrict__ out,
                                                      double *__restrict__ parts)
{
    static_assert(kFoldCols == 16 && kT == 256, "4 groups per wave, 4 waves");
    __shared__ double l[kT / 64][kFoldCols];
    const int c = threadIdx.x & (kFoldCols - 1), g = threadIdx.x >> 4;
    const int wave = threadIdx.x >> 6;
    const int64_t j = static_cast<int64_t>(blockIdx.x) * kFoldCols + c;
    const int64_t jc = j < n ? j : n - 1;
    const int per = (nparts + kFoldGroups - 1) / kFoldGroups;
    const int s0 = min(g * per, nparts), s1 = min(s0 + per, nparts);
    double acc = 0.0;
    for (int b = s0; b < s1; b += 16) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int q = min(b + u, s1 - 1);
            v[u] = keep_if(b + u < s1 && j < n, gp(part)[q * stride + jc]);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += v[u];
    }
    acc += __shfl_xor(acc, 16);
    acc += __shfl_xor(acc, 32);
    if ((threadIdx.x & 63) < kFoldCols) l[wave][c] = acc;
    __syncthreads();
    if (threadIdx.x < kFoldCols) {
        double v = l[0][c];
#pragma unroll
        for (int w = 1; w < kT / 64; ++w) v += l[w][c];
        if (j < n) gp(out)[j] = v;
        double q2 = v * v, q1 = v;         // 0 past the last column
#pragma unroll
        for (int o = 1; o < kFoldCols; o <<= 1) {
            q2 += __shfl_xor(q2, o);
            q1 += __shfl_xor(q1, o);
        }
        if (threadIdx.x == 0) {
            gp(parts)[2 * blockIdx.x] = q2;
            gp(parts)[2 * blockIdx.x + 1] = q1;
        }
    }
}

// Workgroup b: part[2 b] = sum of v[k]^2 and part[2 b + 1] = sum of v[k]
// over its chunk of kStatChunk elements (fixed order).
__global__ __launch_bounds__(kT) void vec_stats_kernel(const double *__restrict__ v, int64_t k,
                                                       double *__restrict__ part)
{
    __shared__ double l2[kT / 64], l1[kT / 64];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kStatChunk;
    double s2 = 0.0, s1 = 0.0;
#pragma unroll
    for (int u = 0; u < kStatChunk / kT; ++u) {
        const int64_t i = base + u * kT + threadIdx.x;
        const double x = i < k ? gp(v)[i] : 0.0;
        s2 += x * x;
        s1 += x;
    }
    s2 = wave_sum(s2);
    s1 = wave_sum(s1);
    if ((threadIdx.x & 63) == 0) {
        l2[threadIdx.x >> 6] = s2;
        l1[threadIdx.x >> 6] = s1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int q = 0; q < kT / 64; ++q) {
            a += l2[q];
            b += l1[q];
        }
        gp(part)[2 * blockIdx.x] = a;
        gp(part)[2 * blockIdx.x + 1] = b;
    }
}

// res = the chunk statistics folded in chunk order.
__global__ void stats_fold_kernel(const double *__restrict__ part, int64_t nchunks,
                                  double *__restrict__ res)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int64_t q = 0; q < nchunks; ++q) {
            a += gp(part)[2 * q];
            b += gp(part)[2 * q + 1];
        }
        gp(res)[0] = a;
        gp(res)[1] = b;
    }
}

// Per workgroup of kErrRows rows: sum xi^2 and sum (xi - R_i C_j / (S + eps))^2
// with S = stats_r[1] (the sum of R) and xi~ = 0 when S + eps == 0.  A
// thread takes columns j = t, t + 256, ...; for each it loads the column's
// kErrRows entries together (rows clamped into the tensor and masked) and
// adds them in row order.
__global__ __launch_bounds__(kT) void err_partial_kernel(const float *__restrict__ xi, int64_t m,
                                                         int64_t n, const double *__restrict__ r,
                                                         const double *__restrict__ c,
                                                         const double *__restrict__ stats_r,
                                                         double eps, double *__restrict__ part)
{
    __shared__ double la[kT / 64], lb[kT / 64];
    const double denom = gp(stats_r)[1] + eps;
    const double inv = denom == 0.0 ? 0.0 : 1.0 / denom;
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kErrRows;
    const int64_t i1 = i0 + kErrRows < m ? i0 + kErrRows : m;
    double ri[kErrRows];
    int64_t ic[kErrRows];
#pragma unroll
    for (int u = 0; u < kErrRows; ++u) {
        ic[u] = i0 + u < i1 ? i0 + u : i1 - 1;
        ri[u] = keep_if(i0 + u < i1, gp(r)[ic[u]] * inv);
    }
    double sa = 0.0, sb = 0.0;
    for (int64_t j = threadIdx.x; j < n; j += kT) {
        const double cj = gp(c)[j];
        float v[kErrRows];
#pragma unroll
        for (int u = 0; u < kErrRows; ++u) v[u] = keep_if(i0 + u < i1, gp(xi)[ic[u] * n + j]);
#pragma unroll
        for (int u = 0; u < kErrRows; ++u) {
            const double x = v[u];
            const double e = x - ri[u] * cj;
            sa += x * x;
            sb += e * e;
        }
    }
    sa = wave_sum(sa);
    sb = wave_sum(sb);
    if ((threadIdx.x & 63) == 0) {
        la[threadIdx.x >> 6] = sa;
        lb[threadIdx.x >> 6] = sb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int q = 0; q < kT / 64; ++q) {
            a += la[q];
            b += lb[q];
        }
        gp(part)[2 * blockIdx.x] = a;
        gp(part)[2 * blockIdx.x + 1] = b;
    }
}

// res[0] = sum of part[2 k], res[1] = sum of part[2 k + 1]: thread t sums
// k = t, t + 256, ... in order, then the threads are combined in a fixed
// order (butterfly in each wave, waves in order).
__global__ __launch_bounds__(kT) void err_fold_kernel(const double *__restrict__ part, int64_t nblk,
                                                      double *__restrict__ res)
{
    __shared__ double la[kT / 64], lb[kT / 64];
    double a = 0.0, b = 0.0;
    for (int64_t q = threadIdx.x; q < nblk; q += kT) {
        a += gp(part)[2 * q];
        b += gp(part)[2 * q + 1];
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if ((threadIdx.x & 63) == 0) {
        la[threadIdx.x >> 6] = a;
        lb[threadIdx.x >> 6] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double x = la[0], y = lb[0];
        for (int w = 1; w < kT / 64; ++w) {
            x += la[w];
            y += lb[w];
        }
        gp(res)[0] = x;
        gp(res)[1] = y;
    }
}

// The one-pass report's numbers in one launch, each summed in a fixed order:
// res = (0, 1^T R = 1^T C from C's fold partials, |xi v|^2, 0, |xi|_F^2,
// |xi - xi~|_F^2).
__global__ __launch_bounds__(kT) void finish_kernel(const double *__restrict__ cfold, int nfold,
                                                    const double *__restrict__ upart,
                                                    const double *__restrict__ epart, int nblk,
                                                    double *__restrict__ res)
{
    __shared__ double l[kT / 64][4];
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int q = threadIdx.x; q < nfold; q += kT) t[0] += gp(cfold)[2 * q + 1];
    for (int q = threadIdx.x; q < nblk; q += kT) {
        t[1] += gp(upart)[2 * q];
        t[2] += gp(epart)[2 * q];
        t[3] += gp(epart)[2 * q + 1];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        t[k] = wave_sum(t[k]);
        if ((threadIdx.x & 63) == 0) l[threadIdx.x >> 6][k] = t[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            t[k] = l[0][k];
            for (int w = 1; w < kT / 64; ++w) t[k] += l[w][k];
        }
        gp(res)[0] = 0.0;
        gp(res)[1] = t[0];
        gp(res)[2] = t[1];
        gp(res)[3] = 0.0;
        gp(res)[4] = t[2];
        gp(res)[5] = t[3];
    }
}

struct DevBuf {
    void *p = nullptr;
    ~DevBuf()
    {
        if (p) (void)hipFree(p);
    }
};

constexpr int64_t kScratchWords = int64_t(1) << 21;    // static workspace: 16 MiB of doubles
constexpr int64_t kOnePassMaxCols = 16384;  // 16 waves x 4 16-byte loads per lane
constexpr int kOnePassMaxBlocks = 256;      // compute units: one round of 16-wave workgroups

// Launch geometry of one report and its workspace: words doubles, and the
// place of every buffer in it, so that the size cannot differ from the layout.
struct ReportShape {
    int64_t stripe, nstripes, ncb, nerr, nfold, nstat, words;
    // one-pass report: row length of the partial sums, workgroups and rows
    // per workgroup (nblk 0: two passes per iteration)
    int64_t stride;
    int nblk, rows;
    // Buffers: R and u (two-pass form only), C, v, column partial sums, fold
    // partials of C and of v, error partials, norm partials (vector statistics
    // in the two-pass form), the six results
    int64_t r, u, c, v, cpart, cfold, vfold, epart, spart, res;
};

ReportShape report_shape(int64_t m, int64_t n)
{
    ReportShape s;
    // Stripe height: the largest power of two in [16, 1024] that still gives
    // the column pass about eight workgroups per compute unit, raised if the
    // stripe count would pass the grid's y limit.
    s.ncb = (n + kT - 1) / kT;
    s.stripe = 1024;
    while (s.stripe > 16 && s.ncb * ((m + s.stripe - 1) / s.stripe) < 2048) s.stripe >>= 1;
    while ((m + s.stripe - 1) / s.stripe > 65535) s.stripe <<= 1;
    s.nstripes = (m + s.stripe - 1) / s.stripe;
    s.nerr = (m + kErrRows - 1) / kErrRows;
    s.nfold = (n + kFoldCols - 1) / kFoldCols;
    const int64_t mk = m > n ? m : n;
    s.nstat = (mk + kStatChunk - 1) / kStatChunk;
    int64_t end = 0;
    auto take = [&end](int64_t count) {
        const int64_t at = end;
        end += count;
        return at;
    };
    s.stride = (n + 3) / 4 * 4;
    s.nblk = s.rows = 0;
    if (n <= kOnePassMaxCols) {
        // The rest of the static workspace bounds the partial sums (only
        // above 8000 columns: 187 workgroups for 4096 x 11008).
        const int64_t fixed = 2 * s.stride + 4 * s.nfold + 6 + 16;
        int64_t most = (kScratchWords - fixed) / (s.stride + 4);
        if (most > kOnePassMaxBlocks) most = kOnePassMaxBlocks;
        // Small tensors: one row per wave up to 1024 columns, beyond that about
        // 128 KB of xi per workgroup, so that there is less to fold (768 x
        // 3072, 30 iterations: 555 us with 4 rows each, 514 with 8, 487 with
        // 12).
        int64_t least = n <= 1024 ? 16 : (32768 + n - 1) / n;
        least = least > 16 ? 16 : least < 4 ? 4 : least;
        int64_t rows = (m + most - 1) / most;
        if (rows < least) rows = least;
        s.rows = static_cast<int>(rows);
        s.nblk = static_cast<int>((m + rows - 1) / rows);
        s.r = s.u = -1;
        s.c = take(s.stride);
        s.v = take(s.stride);
        s.cpart = take(s.nblk * s.stride);
        s.cfold = take(2 * s.nfold);
        s.vfold = take(2 * s.nfold);
        s.epart = take(2 * s.nblk);
        s.spart = take(2 * s.nblk);
    } else {
        s.r = take(m);
        s.c = take(n);
        s.u = take(m);
        s.v = take(n);
        s.cpart = take(s.nstripes * n);
        s.epart = take(2 * s.nerr);
        s.cfold = take(2 * s.nfold);
        s.vfold = take(2 * s.nfold);
        s.spart = take(2 * s.nstat);
    }
    s.res = take(6);
    // Callers plan with one size rule for both forms: r, u of m, c, v of n,
    // column partials (one row per 256 rows of xi up to 1024 columns, one per
    // stripe above), error partials, fold partials of 4 columns each, vector
    // statistics, results.  Whether a tensor fits the static workspace does
    // not depend on the form.
    const int64_t nparts = n <= 1024 ? (m + 255) / 256 : s.nstripes;
    s.words = m + n + m + n + nparts * n + 2 * s.nerr + 4 * ((n + 3) / 4) + 2 * s.nstat + 6;
    if (end > s.words) s.words = end;
    return s;
}

rikfad_status check_report_args(const float *xi, int64_t m, int64_t n, double eps_stab,
                                int32_t power_iters, const rikfad_friction_stats *out)
{
    if (!xi || !out || m < 1 || n < 1 || m >= (int64_t(1) << 31) || n >= (int64_t(1) << 31) ||
        power_iters < 1 || power_iters > 10000 || !(eps_stab >= 0.0) || !std::isfinite(eps_stab)) {
        rk::set_last_error("friction_report: NULL pointer, m or n outside [1, 2^31), "
                           "power_iters outside [1, 10000] or eps_stab negative / not finite");
        return RIKFAD_EINVAL;
    }
    if (reinterpret_cast<uintptr_t>(xi) % 4 != 0) {
        rk::set_last_error("friction_report: xi is not 4-byte aligned");
        return RIKFAD_EALIGN;
    }
    return RIKFAD_OK;
}

// The fewest waves per row whose registers hold it (4 K columns' weights and
// sums in 128 registers: K <= 4 within a wave), K = 2 where several waves
// share a row, up to all 16 waves; K = 3 and 4 only where they must.  The error
// pass, which runs once a report, spills at K = 4 (24 bytes a lane, 76 where 16
// waves share a row).
template <int MODE>
void launch_onepass(const OnePass &a, int nblk, hipStream_t st)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(nblk)), dim3(64 * kPassWaves), 0, st,
                           a);
    };
    if (a.n < 4) go(onepass_kernel<1, 1, MODE, 1>);
    else if (a.n <= 256) go(onepass_kernel<1, 1, MODE>);
    else if (a.n <= 512) go(onepass_kernel<2, 1, MODE>);
    else if (a.n <= 768) go(onepass_kernel<3, 1, MODE>);
    else if (a.n <= 1024) go(onepass_kernel<4, 1, MODE>);
    else if (a.n <= 2048) go(onepass_kernel<2, 4, MODE>);
    else if (a.n <= 4096) go(onepass_kernel<2, 8, MODE>);
    else if (a.n <= 8192) go(onepass_kernel<2, 16, MODE>);
    else if (a.n <= 12288) go(onepass_kernel<3, 16, MODE>);
    else go(onepass_kernel<4, 16, MODE>);
}

// The report itself on a workspace of sh.words doubles at buf (device
// memory).  Every word of the workspace that a kernel reads was written
// earlier in the same call, so its previous contents do not matter.
rikfad_status report_on(const float *xi, int64_t m, int64_t n, double eps_stab,
                        int32_t power_iters, hipStream_t st, const ReportShape &sh, double *buf,
                        rikfad_friction_stats *out)
{
    double *c = buf + sh.c, *v = buf + sh.v, *cpart = buf + sh.cpart;
    double *cfold = buf + sh.cfold, *vfold = buf + sh.vfold, *epart = buf + sh.epart;
    double *stats_r = buf + sh.res;         // results: R (2), u (2), errors (2)
    const int nfold = static_cast<int>(sh.nfold);
    const dim3 fold_grid(static_cast<uint32_t>(nfold));
    if (sh.nblk) {
        // power_iters + 2 passes over xi.  The first forms C = xi^T 1; the
        // first power iteration (from v = C) also sums |xi|_F^2 and
        // |xi - xi~|_F^2; the last pass forms |xi v| for the final unit
        // vector v.
        double *upart = buf + sh.spart;
        OnePass a{xi, m, n, sh.rows, nfold, nullptr, nullptr, eps_stab, cpart, epart, sh.stride};
        auto fold = [&](double *out, double *parts) {
            hipLaunchKernelGGL(col_fold_kernel, fold_grid, dim3(kT), 0, st, cpart, sh.stride, n,
                               sh.nblk, out, parts);
        };
        launch_onepass<kPassSums>(a, sh.nblk, st);
        fold(c, cfold);
        a.v = c;
        a.vparts = cfold;
        launch_onepass<kPassPowerErr>(a, sh.nblk, st);
        fold(v, vfold);
        a.v = v;
        a.vparts = vfold;
        for (int it = 1; it < power_iters; ++it) {
            launch_onepass<kPassPower>(a, sh.nblk, st);
            fold(v, vfold);
        }
        a.spart = upart;
        launch_onepass<kPassNorm>(a, sh.nblk, st);
        hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(kT), 0, st, cfold, nfold, upart, epart,
                           sh.nblk, stats_r);
    } else {
        const int64_t stripe = sh.stripe, nerr = sh.nerr;
        const int nstripes = static_cast<int>(sh.nstripes);
        double *r = buf + sh.r, *u = buf + sh.u, *spart = buf + sh.spart;
        double *stats_u = stats_r + 2, *err = stats_u + 2;
        const dim3 rows_grid(static_cast<uint32_t>((m + kT / 64 - 1) / (kT / 64)));
        const dim3 cols_grid(static_cast<uint32_t>(sh.ncb), static_cast<uint32_t>(nstripes));
        auto stats = [&](const double *vec, int64_t k, double *res) {
            const int64_t nch = (k + kStatChunk - 1) / kStatChunk;
            hipLaunchKernelGGL(vec_stats_kernel, dim3(static_cast<uint32_t>(nch)), dim3(kT), 0, st,
                               vec, k, spart);
            hipLaunchKernelGGL(stats_fold_kernel, dim3(1), dim3(1), 0, st, spart, nch, res);
        };
        // Shadow factors R = xi 1, C = xi^T 1 and the sum of R.
        hipLaunchKernelGGL(row_reduce_kernel, rows_grid, dim3(kT), 0, st, xi, m, n, nullptr,
                           nullptr, 0, r);
        hipLaunchKernelGGL(col_partial_kernel, cols_grid, dim3(kT), 0, st, xi, m, n, stripe,
                           nullptr, cpart);
        hipLaunchKernelGGL(col_fold_kernel, fold_grid, dim3(kT), 0, st, cpart, n, n, nstripes, c,
                           cfold);
        stats(r, m, stats_r);
        // |xi|_F^2 and |xi - xi~|_F^2
        hipLaunchKernelGGL(err_partial_kernel, dim3(static_cast<uint32_t>(nerr)), dim3(kT), 0, st,
                           xi, m, n, r, c, stats_r, eps_stab, epart);
        hipLaunchKernelGGL(err_fold_kernel, dim3(1), dim3(kT), 0, st, epart, nerr, err);
        // Power iteration on xi^T xi from v = C / |C|: u = xi v / |v|,
        // v <- xi^T u; each row pass normalises its input from the fold
        // partials of the last column pass.
        const double *vin = c, *vin_fold = cfold;
        for (int it = 0; it < power_iters; ++it) {
            hipLaunchKernelGGL(row_reduce_kernel, rows_grid, dim3(kT), 0, st, xi, m, n, vin,
                               vin_fold, nfold, u);
            hipLaunchKernelGGL(col_partial_kernel, cols_grid, dim3(kT), 0, st, xi, m, n, stripe,
                               u, cpart);
            hipLaunchKernelGGL(col_fold_kernel, fold_grid, dim3(kT), 0, st, cpart, n, n, nstripes,
                               v, vfold);
            vin = v;
            vin_fold = vfold;
        }
        // sigma_1 = |xi v| for the final unit vector v.
        hipLaunchKernelGGL(row_reduce_kernel, rows_grid, dim3(kT), 0, st, xi, m, n, vin,
                           vin_fold, nfold, u);
        stats(u, m, stats_u);
    }
    // The six results are adjacent: one copy brings them back (host[] keeps
    // the order R, errors, u).
    hipError_t e = hipGetLastError();
    double res[6];
    if (e == hipSuccess) e = hipMemcpyAsync(res, stats_r, sizeof(res), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    const double host[6] = {res[0], res[1], res[4], res[5], res[2], res[3]};
    if (e != hipSuccess) {
        rk::set_last_error((std::string("friction_report: ") + hipGetErrorString(e)).c_str());
        return RIKFAD_EHIP;
    }
    const double fro2 = host[2], err2 = host[3], sigma1_sq = host[4];
    out->xi_fro2 = fro2;
    out->err_fro2 = err2;
    out->sum_r = host[1];
    out->sigma1 = std::sqrt(sigma1_sq);
    out->rel_err = fro2 > 0.0 ? std::sqrt(err2 / fro2) : 0.0;
    const double ratio = fro2 > 0.0 ? sigma1_sq / fro2 : 1.0;
    out->eckart_young_floor = std::sqrt(ratio < 1.0 ? 1.0 - ratio : 0.0);
    out->stable_rank = sigma1_sq > 0.0 ? fro2 / sigma1_sq : 0.0;
    out->power_iters = power_iters;
    out->reserved = 0;
    return RIKFAD_OK;
}

// ------------------------------------------------ report without allocation
//
// A file-scope device array is the workspace of rikfad_friction_report_noalloc.
// Each device holds its own copy at its own address, which host code must
// obtain with hipGetSymbolAddress (the array's name in host code is only a
// stand-in for the symbol, not a device address).  The address is looked up
// once per device, with that device current, on the first call there.

}  // namespace

static __device__ __align__(256) double scratch[kScratchWords];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};

rikfad_status scratch_of_current_device(double **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        rk::set_last_error((std::string("friction_report_noalloc: hipGetDevice: ") +
                            hipGetErrorString(e)).c_str());
        return RIKFAD_EHIP;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        rk::set_last_error("friction_report_noalloc: device index beyond 63");
        return RIKFAD_EINVAL;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            rk::set_last_error((std::string("friction_report_noalloc: hipGetSymbolAddress: ") +
                                hipGetErrorString(e)).c_str());
            return RIKFAD_EHIP;
        }
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return RIKFAD_OK;
}

}  // namespace

extern "C" rikfad_status rikfad_friction_report(const float *xi, int64_t m, int64_t n,
                                                double eps_stab, int32_t power_iters,
                                                void *stream_, rikfad_friction_stats *out)
{
    rikfad_status s = check_report_args(xi, m, n, eps_stab, power_iters, out);
    if (s != RIKFAD_OK) return s;
    const ReportShape sh = report_shape(m, n);
    DevBuf buf;
    if (hipMalloc(&buf.p, sizeof(double) * static_cast<size_t>(sh.words)) != hipSuccess) {
        rk::set_last_error("friction_report: hipMalloc of the workspace failed");
        return RIKFAD_ENOMEM;
    }
    return report_on(xi, m, n, eps_stab, power_iters, static_cast<hipStream_t>(stream_), sh,
                     static_cast<double *>(buf.p), out);
}

extern "C" int64_t rikfad_friction_report_noalloc_max_bytes(void)
{
    return kScratchWords * static_cast<int64_t>(sizeof(double));
}

extern "C" int64_t rikfad_friction_report_workspace_bytes(int64_t m, int64_t n)
{
    if (m < 1 || n < 1 || m >= (int64_t(1) << 31) || n >= (int64_t(1) << 31)) return -1;
    return report_shape(m, n).words * static_cast<int64_t>(sizeof(double));
}

extern "C" rikfad_status rikfad_friction_report_noalloc(const float *xi, int64_t m, int64_t n,
                                                        double eps_stab, int32_t power_iters,
                                                        void *stream_,
                                                        rikfad_friction_stats *out)
{
    rikfad_status s = check_report_args(xi, m, n, eps_stab, power_iters, out);
    if (s != RIKFAD_OK) return s;
    const ReportShape sh = report_shape(m, n);
    if (sh.words > kScratchWords) {
        rk::set_last_error(("friction_report_noalloc: an " + std::to_string(m) + " x " +
                            std::to_string(n) + " tensor needs " +
                            std::to_string(sh.words * 8) + " bytes of workspace, more than the " +
                            std::to_string(kScratchWords * 8) + "-byte static scratch")
                               .c_str());
        return RIKFAD_EINVAL;
    }
    double *ws = nullptr;
    if ((s = scratch_of_current_device(&ws)) != RIKFAD_OK) return s;
    return report_on(xi, m, n, eps_stab, power_iters, static_cast<hipStream_t>(stream_), sh, ws,
                     out);
}
