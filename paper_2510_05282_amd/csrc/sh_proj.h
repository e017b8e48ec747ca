// sh_proj.h -- per-point projector evaluation shared by the projector and
// serving kernels: spline lookup of R_l(r) and the product R_l(r) * R_l^m(d).
//
// Radial table layout (one table): [n_r][ch] of (y_i, M_i) -- knot i of every
// channel is adjacent, so the interval [i, i+1] of all channels of a point is
// 2 ch consecutive double2 (one 128-byte line for ch = 4) instead of ch lines
// n_r * 16 bytes apart.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sh_core.h"
#include "sh_fwd.h"
#include "sh_internal.h"

namespace shk {

struct SplineGrid {
    int n_r;
    double h, inv_h, r_max, h2_over_6;
};

// R_0 .. R_{NL-1} at r >= 0 from a table with ch >= NL channels: interval
// i = floor(r/h) clamped to [0, n_r-2], t = r/h - i, A = 1 - t, B = t,
//     S = A y_i + B y_{i+1} + ((A^3 - A) M_i + (B^3 - B) M_{i+1}) h^2/6;
// 0 beyond r_max; a NaN r gives NaN.  spline_eval, below, is the one to call; its steps:
// spline_knots loads the pairs of knots i and i+1 (r <= r_max), spline_from evaluates the
// cubic from them (any r; the pairs are not used beyond r_max or for NaN).
__host__ __device__ __forceinline__ int spline_interval(double r, const SplineGrid& g)
{
    const double q = r <= g.r_max ? r * g.inv_h : 0.0;
    const int i = int(q);
    return i > g.n_r - 2 ? g.n_r - 2 : i;
}

template <int NL, typename KN>
__host__ __device__ __forceinline__ void spline_knots(const KN* __restrict__ tab, int ch, const SplineGrid& g,
                                                      double r, KN (&a)[NL], KN (&b)[NL])
{
    const KN* k0 = tab + int64_t(spline_interval(r, g)) * ch;
    static_for<0, NL>([&](auto lc) {
        constexpr int L = decltype(lc)::value;
        a[L] = k0[L];
        b[L] = k0[ch + L];
    });
}

template <int NL, typename TIO>
__host__ __device__ __forceinline__ void spline_from(const double2 (&a)[NL], const double2 (&b)[NL],
                                                     const SplineGrid& g, double r, TIO (&R)[NL])
{
    if (!(r <= g.r_max)) {
        const double v = r != r ? r : 0.0;
        static_for<0, NL>([&](auto lc) { R[decltype(lc)::value] = TIO(v); });
        return;
    }
    const double q = r * g.inv_h;
    const double t = q - double(spline_interval(r, g));
    const double A = 1.0 - t, B = t;
    static_for<0, NL>([&](auto lc) {
        constexpr int L = decltype(lc)::value;
        R[L] = TIO(A * a[L].x + B * b[L].x + ((A * A * A - A) * a[L].y + (B * B * B - B) * b[L].y) * g.h2_over_6);
    });
}

// The same from float pairs, for the FP32 kernels: the interval i and t = r/h - i
// in FP64 (near r_max, r/h is ~n_r, and float would leave t only a few bits), the
// cubic in FP32.  Table values rounded to float and the FP32 cubic put at most a
// few 1e-7 (of max|R|) into R, well inside the FP32 tolerance.
template <int NL, typename TIO>
__host__ __device__ __forceinline__ void spline_from(const float2 (&a)[NL], const float2 (&b)[NL],
                                                     const SplineGrid& g, double r, TIO (&R)[NL])
{
    static_assert(sizeof(TIO) == 4, "float tables serve the FP32 kernels");
    if (!(r <= g.r_max)) {
        const float v = r != r ? float(r) : 0.0f;
        static_for<0, NL>([&](auto lc) { R[decltype(lc)::value] = v; });
        return;
    }
    const double q = r * g.inv_h;
    const float t = float(q - double(spline_interval(r, g)));
    const float A = 1.0f - t, B = t, h26 = float(g.h2_over_6);
    static_for<0, NL>([&](auto lc) {
        constexpr int L = decltype(lc)::value;
        R[L] = A * a[L].x + B * b[L].x + ((A * A * A - A) * a[L].y + (B * B * B - B) * b[L].y) * h26;
    });
}

// Both steps for one point; nothing is loaded beyond r_max.
template <int NL, typename TIO, typename KN>
__host__ __device__ __forceinline__ void spline_eval(const KN* __restrict__ tab, int ch, const SplineGrid& g,
                                                     double r, TIO (&R)[NL])
{
    KN a[NL], b[NL];
    if (r <= g.r_max) spline_knots<NL>(tab, ch, g, r, a, b);
    spline_from<NL, TIO>(a, b, g, r, R);
}

// Natural cubic spline on a uniform grid for one channel.  With knot spacing h
// the second derivatives solve, for k = 1 .. n_r-2,
//     M_{k-1} + 4 M_k + M_{k+1} = 6 (y_{k+1} - 2 y_k + y_{k-1}) / h^2,
// M_0 = M_{n_r-1} = 0, by forward elimination and back substitution (cc holds
// the eliminated super-diagonal).  Knot k's pair (y_k, M_k) goes to
// tc[k * stride], so the channels of a table can be interleaved.
__host__ __device__ inline void spline_solve(const double* __restrict__ yc, double2* __restrict__ tc, int64_t stride,
                                             double* __restrict__ cc, int n_r, double six_over_h2)
{
    for (int k = 0; k < n_r; ++k) tc[k * stride] = make_double2(yc[k], 0.0);
    double cprev = 0.0, dprev = 0.0;  // forward elimination over k = 1 .. n_r-2 (dp kept in .y)
    for (int k = 1; k <= n_r - 2; ++k) {
        const double rhs = six_over_h2 * (yc[k + 1] - 2.0 * yc[k] + yc[k - 1]);
        const double den = 4.0 - cprev;
        cprev = 1.0 / den;
        dprev = (rhs - dprev) / den;
        cc[k] = cprev;
        tc[k * stride].y = dprev;
    }
    for (int k = n_r - 3; k >= 1; --k) tc[k * stride].y -= cc[k] * tc[(k + 1) * stride].y;  // M_{n_r-1} = 0
}

__host__ __device__ constexpr int l_of_row(int r)
{
    int l = 0;
    while ((l + 1) * (l + 1) <= r) ++l;
    return l;
}

// All projector values of one point p (coordinates already loaded): d = p - c,
// R_l(|d|) from the table `tab` with `ch` channels, harmonics of d; the value of
// row f goes to out[f * stride].
template <int LMAX, typename TIO>
__device__ __forceinline__ void proj_point(double px, double py, double pz, const double c[3],
                                           const knot_t<TIO>* __restrict__ tab, int ch, const SplineGrid& g,
                                           TIO* __restrict__ out, int64_t stride)
{
    const double dx = px - c[0], dy = py - c[1], dz = pz - c[2];
    double xb, yb, zb, keep;
    normalize(dx, dy, dz, xb, yb, zb, keep);
    const double r = sqrt(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)));
    TIO R[LMAX + 1];
    spline_eval<LMAX + 1, TIO>(tab, ch, g, r, R);
    eval_unit<LMAX, TIO>(TIO(xb), TIO(yb), TIO(zb), TIO(keep),
                         [&](int f, TIO v) { out[int64_t(f) * stride] = R[l_of_row(f)] * v; });
}

// The first nvalid of the PPL values of o (adjacent points) to dst: 16-byte stores at
// any element alignment where all of them are wanted, else one by one.
template <typename TIO, int PPL, typename V>
__device__ __forceinline__ void store_run(TIO* __restrict__ dst, V o, int nvalid)
{
    constexpr int UNIT = 16 / int(sizeof(TIO)) < PPL ? 16 / int(sizeof(TIO)) : PPL;
    if (nvalid < PPL) {
#pragma unroll
        for (int q = 0; q < PPL; ++q)
            if (q < nvalid) dst[q] = lane<V, PPL>(o, q);
        return;
    }
    static_for<0, PPL / UNIT>([&](auto kc) {
        constexpr int i0 = decltype(kc)::value * UNIT;
        typename uvec_of<TIO, UNIT>::type w;
        static_for<0, UNIT>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            w[u] = lane<V, PPL>(o, i0 + u);
        });
        *reinterpret_cast<typename uvec_of<TIO, UNIT>::type*>(dst + i0) = w;
    });
}

// The same for PPL adjacent points of one table and centre, evaluated together
// (the polynomials on PPL-wide vectors, which keeps more independent work in each
// lane): point q's coordinates are (px[q], py[q], pz[q]) and row f of point q goes
// to out[f * stride + q], for the first nvalid points only (the others are computed
// and dropped, so a tail lane runs the same code).
template <int LMAX, typename TIO, int PPL>
__device__ __forceinline__ void proj_points(const double (&px)[PPL], const double (&py)[PPL], const double (&pz)[PPL],
                                            const double c[3], const knot_t<TIO>* __restrict__ tab, int ch,
                                            const SplineGrid& g, TIO* __restrict__ out, int64_t stride,
                                            int nvalid = PPL)
{
    using V = typename vec_of<TIO, PPL>::type;
    V x, y, z, k;
    TIO R[PPL][LMAX + 1];
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        const double dx = px[q] - c[0], dy = py[q] - c[1], dz = pz[q] - c[2];
        double xb, yb, zb, keep;
        normalize(dx, dy, dz, xb, yb, zb, keep);
        spline_eval<LMAX + 1, TIO>(tab, ch, g, sqrt(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz))), R[q]);
        lane<V, PPL>(x, q) = TIO(xb);
        lane<V, PPL>(y, q) = TIO(yb);
        lane<V, PPL>(z, q) = TIO(zb);
        lane<V, PPL>(k, q) = TIO(keep);
    }
    eval_unit<LMAX, V>(x, y, z, k, [&](int f, V v) {
        const int l = l_of_row(f);
        V r;
#pragma unroll
        for (int q = 0; q < PPL; ++q) lane<V, PPL>(r, q) = R[q][l];
        store_run<TIO, PPL>(out + int64_t(f) * stride, r * v, nvalid);
    });
}

// Points per lane of a projector build that fills the GPU many times over: 16 bytes' worth.
// (FP64 4 points at lmax 1 141 us against 2 points 144, at lmax >= 2 4-20% slower; FP32 2
// points equal at lmax 6, 8 and 9 and up to 30% slower elsewhere; builds of 64 atoms.)
template <typename TIO> constexpr int kProjPpl = 16 / int(sizeof(TIO));

// Builds of at least this many points, or bytes written, take several points per lane
// (launch_proj_l in sh_proj.hip): below, a launch lasts its workgroups' chain of work, which
// wider lanes lengthen, and what it writes stays in the memory-side cache.  us, one point
// against several: FP64 lmax 6, 24 x 4189 points (41 MB) 10.7 / 14.6; lmax 1, 64 x 14137 (50
// MB) 13.0 / 18.0; FP32 lmax 3 (68 MB) 14.6 / 22.5; FP64 lmax 3, 904673 points (116 MB) into
// one output 24.4 / 30.7, three outputs in turn 27.0 / 31.8, inputs and outputs out of the
// caches 42.2 / 38.5; lmax 4 (181 MB) 32 / 38, 41 / 43; lmax 6 (355 MB) 118 / 98, 117 / 97.
constexpr int64_t kProjVecPoints = int64_t(1) << 20, kProjVecBytes = int64_t(1) << 28;

// LDS reserved (not used) by proj_kernel with several points per lane: at most 2 resident
// workgroups per CU, or 1.  Fewer waves at once keep each row's concurrent writes in a
// smaller window and let the partial lines of neighbouring waves merge in the L2 (an atom
// has any number of points, so its rows start anywhere); more hide the latency of the
// spline lookups, which matters where a row count is small or the tables of many atoms
// outgrow the L2.  us, uncapped / 2 / 1 workgroups, 64 atoms of about 4 to 10 MB a row:
// FP64 lmax 0 78 / 107 / 154, lmax 3 156 / 132 / 160, lmax 4 217 / 179 / 197, lmax 5 285 /
// 254 / 243, lmax 6 313 / 297 / 272, lmax 7 340 / 321 / 290, lmax 9 384 / 388 / 348; FP32
// lmax 3 127 / 114 / -, lmax 4 190 / 154 / -, lmax 5 238 / 217 / 212, lmax 6 254 / 244 /
// 228, lmax 8 266 / 254 / 236, lmax 9 329 / 314 / 285.  200 atoms, 2 / 1: FP64 lmax 5 268 /
// 287, lmax 6 280 / 293, lmax 7 255 / 237; FP32 lmax 6 201 / 218, lmax 8 182 / 175.  The
// offsets are on the device; a total that deals every atom the same whole number of 128-byte
// lines is taken for rows on lines: 64 x 150000, FP64 lmax 5 601 / 616, lmax 6 791 / 812.
template <typename TIO, int LMAX>
inline size_t proj_cap_lds(int n_atoms, int64_t n_points)
{
    constexpr bool f64 = sizeof(TIO) == 8;
    if (f64 ? LMAX == 0 : LMAX <= 1) return 0;
    if (LMAX <= 4) return kCapLds2;
    if (LMAX >= (f64 ? 7 : 8)) return kCapLds1;
    const bool lines = n_atoms > 0 && n_points % (int64_t(n_atoms) * (128 / int64_t(sizeof(TIO)))) == 0;
    return n_atoms > 64 || (f64 && lines) ? kCapLds2 : kCapLds1;
}

// Builds that hold tables in LDS (proj_lds_kernel): one workgroup of 1024 lanes per CU, or two
// of 512 where the table is small (FP32 lmax <= 1: 65 us against 74 at lmax 1, 64 x 150k points).
constexpr int64_t kLdsPerCu = 160 * 1024;
constexpr int64_t kProjLoadCost = 256;  // a table load's worth in points, and one more per 256 bytes
template <typename TIO, int LMAX> constexpr int kProjLdsBlock = sizeof(TIO) == 4 && LMAX <= 1 ? 512 : 1024;
template <typename TIO> constexpr int kProjLdsMax = sizeof(TIO) == 8 ? 3 : 4;  // highest lmax that uses it

template <typename TIO, int LMAX>
constexpr int64_t proj_lds_bytes(int n_r)
{
    return (int64_t(n_r) * (LMAX + 1) * int64_t(sizeof(knot_t<TIO>)) + 15) / 16 * 16;
}

// Whether a large build does: the table has the build's channels (a handle keeps such copies)
// and fits, an atom has enough points on average for its load, and over few atoms, whose
// tables stay in the L2, there are points enough or the launch without LDS is the slower one.
// us without / with, tables of 2000 knots: FP32 lmax 1, 64 x 17187 11.8 / 13.5, 8 x 137500 11.3 /
// 13.2, 8 x 300000 17.0 / 18.7, 64 x 62500 36.0 / 29.9, 128 x 8593 15.7 / 14.0; FP64 lmax 0, 64 x
// 25000 12.4 / 13.4, 64 x 62500 37.1 / 30.1, 128 x 8593 13.2 / 11.2; FP64 lmax 2, 8 x 1200000
// 196 / 227, 64 x 150000 207 / 209, 128 x 12500 45.3 / 40.7; FP64 lmax 3, 300 x 3666 47.2 / 58.2,
// 300 x 5333 65.9 / 64.9; FP32 lmax 3, 64 x 62500 72.2 / 70.9, 300 x 5333 41.1 / 40.3.
template <typename TIO, int LMAX>
inline bool use_proj_lds(int n_atoms, int64_t n_points, int tab_ch, int n_r)
{
    constexpr bool f64 = sizeof(TIO) == 8;
    if (LMAX > kProjLdsMax<TIO> || tab_ch != LMAX + 1) return false;
    if (proj_lds_bytes<TIO, LMAX>(n_r) * (1024 / kProjLdsBlock<TIO, LMAX>) > kLdsPerCu) return false;
    if (n_points < kProjVecPoints || n_points / (f64 && LMAX == 3 ? 4096 : 2048) < n_atoms) return false;
    if (LMAX == (f64 ? 1 : 2)) return true;
    if (LMAX == 0 || (!f64 && LMAX == 1)) return n_atoms > 64 || n_points >= int64_t(3) << 20;
    return n_atoms > (f64 && LMAX == 3 ? 128 : 64);
}

// How many workgroups go side by side through consecutive points there: 1, or the 32 CUs of an
// XCD where the write path is what counts and the points are enough for 32 loads of a table.
// us with 1 / 32: FP32 lmax 0, 64 x 150000 37.7 / 39.2; lmax 1, 64 x 62500 29.9 / 32.7, 64 x
// 150000 into one output 66.8 / 63.3, 128 x 18750 18.9 / 24.7; lmax 2, 64 x 37500 32.5 / 38.5, 64 x
// 150000 116 / 109; lmax 3, 300 x 3666 30.7 / 37.8, 300 x 5333 36.6 / 40.1, 128 x 31250 82.1 /
// 70.8; FP64 lmax 0, 8 x 1200000 68.1 / 63.3, 64 x 150000 69.1 / 66.6, 128 x 75000 67.7 / 83.2;
// lmax 1, 8 x 137500 15.4 / 16.5, 64 x 150000 128 / 122, 128 x 75000 128 / 143; lmax 2, 128 x
// 12500 40.7 / 41.5, 300 x 3666 37.1 / 42.5; lmax 3, 300 x 13333 168 / 159.
template <typename TIO, int LMAX>
inline int proj_lds_group(int n_atoms, int64_t n_points)
{
    constexpr bool f64 = sizeof(TIO) == 8;
    constexpr int kAtoms = LMAX > 2 ? 1 << 30 : (!f64 && LMAX == 2 ? 128 : 64);  // at most, for 32
    constexpr int kLog = LMAX == (f64 ? 0 : 1) ? 23 : (f64 ? 21 : (LMAX == 2 ? 22 : 21));
    if (LMAX == (f64 ? 2 : 0)) return 1;
    return n_atoms <= kAtoms && ((f64 && LMAX == 3) || n_points >= int64_t(1) << kLog) ? 32 : 1;
}

// Wave-wide searches, N at once over the same n sorted keys: at[i] = the last k in [0, n)
// with key(k) <= x[i], or -1 if there is none.  Every lane must be active and pass the same
// x; each round the 64 lanes probe 64 evenly spaced keys and a ballot keeps the bracket, so
// n keys take ceil(log64 n) dependent loads.  Keys that are not sorted still give some k
// in [0, n) or -1 (callers check what they use).
template <int N, typename Key>
__device__ __forceinline__ void wave_searches(int n, Key&& key, const int64_t (&x)[N], int (&at)[N])
{
    const int lane = threadIdx.x & 63;
    int lo[N], hi[N];  // the answers lie in [lo, hi)
    bool none[N];
#pragma unroll
    for (int i = 0; i < N; ++i) lo[i] = 0, hi[i] = n, none[i] = false;
    for (int width = n, first = 1; width > 1 || first; first = 0) {
        width = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int step = (hi[i] - lo[i] + 63) / 64;
            const int k = lo[i] + lane * step;
            const bool pred = k < hi[i] && key(k) <= x[i];
            const int c = __popcll(__ballot(pred));  // lanes 0 .. c-1 probe keys <= x
            none[i] = none[i] || c == 0;
            lo[i] += c > 0 ? (c - 1) * step : 0;
            hi[i] = c > 0 ? min(lo[i] + step, hi[i]) : lo[i];
            width = max(width, hi[i] - lo[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) at[i] = none[i] ? -1 : lo[i];
}

// One of them over an array.
__device__ __forceinline__ int wave_search(const int64_t* __restrict__ keys, int n, int64_t x)
{
    const int64_t xs[1] = {x};
    int at[1];
    wave_searches<1>(n, [&](int k) { return keys[k]; }, xs, at);
    return at[0];
}

// The value v holds in lane k of the wave; k must be the same in every lane (one
// scalar read per 32 bits, no memory access).
template <typename T>
__device__ __forceinline__ T lane_value(T v, int k)
{
    static_assert(sizeof(T) % 4 == 0, "32-bit words");
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int q = 0; q < int(sizeof(T) / 4); ++q) w[q] = __builtin_amdgcn_readlane(w[q], k);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// The same for one lane (binary search): the last k in [0, n) with keys[k] <= x, or 0.
__device__ __forceinline__ int lane_search(const int64_t* __restrict__ keys, int n, int64_t x)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (keys[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace shk
