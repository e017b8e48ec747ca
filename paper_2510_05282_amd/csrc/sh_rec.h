// sh_rec.h -- real harmonics of any l <= shc::kRecLmax by the normalised
// associated-Legendre recurrence (sh_rec.hip states the formulas; the
// coefficients are the generated tables of sh_rec_constants.h).  Host and device.
#pragma once

#include <hip/hip_runtime.h>

#include "sh_core.h"
#include "sh_fwd.h"
#include "sh_rec_constants.h"

namespace shk {

// The recurrence's coefficients in the order the loops take them, in the arithmetic
// type S (rounded once from double): for every m the pairs (a, b) of l = m, m + 1, ...
// with Yb_l = a (z Yb_{l-1} - b Yb_{l-2}).  l = m + 1 is kRecE with b = 0; at l = m,
// Yb_{m-1} = 0 and Yb_{m-2} = -1 make it d_m = d_m (z 0 - 1 (-1)).  Rows are padded so
// that a block of up to 8 pairs from any l <= kRecLmax stays inside: a wave reads a
// block's pairs in one or two scalar loads.
constexpr int kRecRow = (shc::kRecLmax + 1 + 8 + 7) / 8 * 8;
template <typename S>
struct alignas(64) RecTable {
    S ab[shc::kRecLmax + 1][kRecRow][2];
    constexpr RecTable() : ab{}
    {
        for (int m = 0; m <= shc::kRecLmax; ++m)
            for (int l = m; l <= shc::kRecLmax; ++l) {
                ab[m][l - m][0] = S(l == m ? shc::kRecD[m] : l == m + 1 ? shc::kRecE[m] : shc::kRecA[l][m]);
                ab[m][l - m][1] = S(l == m ? 1.0 : l == m + 1 ? 0.0 : shc::kRecB[l][m]);
            }
    }
};
template <typename S> constexpr RecTable<S> kRecTable{};

// All (lmax+1)^2 values at the unit vector (x, y, z); store(l, m, value), and for
// m > 0 the value of +m comes just before that of -m.  keep
// masks the m = 0 rows of l > 0 at the origin, as in eval_unit.  T is double, float
// or a clang vector of them (that many points at once).  The loops run over the
// runtime lmax, UNROLL degrees at a time (8 at most), and over m = part, part + parts, ... only:
// the values do not depend on how many parts a point is dealt to.
template <typename T, int UNROLL = 4, typename Store>
__host__ __device__ __forceinline__ void eval_unit_rec(T x, T y, T z, T keep, int lmax, Store&& store, int part = 0,
                                                       int parts = 1)
{
    static_assert(UNROLL <= 8, "the table's rows are padded for 8");
    using S = scalar_t<T>;
    T c = T(S(1)), s = T(S(0));  // C_m + i S_m = (x + i y)^m
    auto step = [&] {
        const T cn = x * c - y * s;
        s = x * s + y * c;
        c = cn;
    };
    for (int m = 0; m < part; ++m) step();
    for (int m = part; m <= lmax; m += parts) {
        const auto& row_m = kRecTable<S>.ab[m];
        auto put = [&](int l, T yl) {
            if (m == 0) {
                store(l, 0, l > 0 ? yl * keep : yl);
            } else {
                store(l, m, yl * c);
                store(l, -m, yl * s);
            }
        };
        T y2 = T(S(0)), y1 = T(row_m[0][0]);  // Yb_{l-2}^m, Yb_{l-1}^m
        put(m, y1);
        for (int l0 = m + 1; l0 <= lmax; l0 += UNROLL) {
            S a[UNROLL], b[UNROLL];
#pragma unroll
            for (int i = 0; i < UNROLL; ++i) a[i] = row_m[l0 - m + i][0], b[i] = row_m[l0 - m + i][1];
#pragma unroll
            for (int i = 0; i < UNROLL; ++i) {
                if (l0 + i > lmax) break;
                const T yl = a[i] * (z * y1 - b[i] * y2);
                y2 = y1;
                y1 = yl;
                put(l0 + i, yl);
            }
        }
        for (int k = 0; k < parts; ++k) step();
    }
}

// v = sum over rows of G[row] grad_u P_row at the unit vector u = (x, y, z), for
// 0 <= lmax <= kRecLmax, where P is the off-sphere extension the recurrence
// evaluates: P_l^0 = Pb_l^0(z), P_l^m = Pb_l^m(z) C_m(x, y), P_l^-m = Pb_l^m(z) S_m(x, y)
// with C_m + i S_m = (x + i y)^m.  Its partials are
//     d(Pb C_m) = (m Pb C_{m-1}, -m Pb S_{m-1}, Pb' C_m),
//     d(Pb S_m) = (m Pb S_{m-1},  m Pb C_{m-1}, Pb' S_m),
// so per m only four sums over l are needed: a = sum G Pb and b = sum G Pb' for the
// cosine (+m) and sine (-m) rows.  Pb' follows from differentiating the recurrence:
// Pb_l' = A_l (Pb_{l-1} + z Pb_{l-1}' - B_l Pb_{l-2}').  The m are dealt to kRecParts
// parts, m = part, part + kRecParts, ..., which one lane each can take at the same time
// (their rows are then read by as many waves); grad_unit_rec_sum adds them up, always in
// the same order.  g(row) returns G[row], asked for a block of UNROLL degrees before the
// first is used, so that many reads are under way at once; T is double, float or a
// clang vector of them.
constexpr int kRecParts = 4;
template <typename T, int UNROLL, typename GAt>
__host__ __device__ __forceinline__ void grad_unit_rec_part(T x, T y, T z, int lmax, int part, GAt&& g, T& vx, T& vy,
                                                            T& vz)
{
    static_assert(UNROLL <= 8, "the table's rows are padded for 8");
    using S = scalar_t<T>;
    const T zero = T(S(0));
    vx = zero;
    vy = zero;
    vz = zero;
    T c = T(S(1)), s = zero, cp = zero, sp = zero;  // C_m, S_m, C_{m-1}, S_{m-1}
    auto step = [&] {
        cp = c;
        sp = s;
        c = x * cp - y * sp;
        s = x * sp + y * cp;
    };
    for (int m = 0; m < part; ++m) step();
    for (int m = part; m <= lmax; m += kRecParts) {
        const auto& row_m = kRecTable<S>.ab[m];
        T y1 = zero, dy1 = zero, y2 = T(S(-1)), dy2 = zero;  // Pb_{l-1}, Pb'_{l-1}, Pb_{l-2}, Pb'_{l-2}
        T ac = zero, bc = zero, as = zero, bs = zero;
        for (int l0 = m; l0 <= lmax; l0 += UNROLL) {
            S a[UNROLL], b[UNROLL];
            T gc[UNROLL], gs[UNROLL];
#pragma unroll
            for (int i = 0; i < UNROLL; ++i) {
                // beyond lmax the last row again, as 0: a branch around each read would
                // have it waited for before the next is issued
                const int l = l0 + i <= lmax ? l0 + i : lmax;
                a[i] = row_m[l0 - m + i][0], b[i] = row_m[l0 - m + i][1];
                gc[i] = g(row(l, m));
                // m = 0 has no sine rows: read as more of the cosine's, or not at all
                gs[i] = std::is_arithmetic_v<T> && UNROLL == 1 && m == 0 ? zero : g(row(l, -m));
            }
#ifdef __HIP_DEVICE_COMPILE__
            __builtin_amdgcn_sched_barrier(0);  // the reads stay ahead of the arithmetic
#endif
#pragma unroll
            for (int i = 0; i < UNROLL; ++i) {
                const T yl = a[i] * (z * y1 - b[i] * y2);
                const T dl = a[i] * (y1 + z * dy1 - b[i] * dy2);
                y2 = y1;
                dy2 = dy1;
                y1 = yl;
                dy1 = dl;
                const T c_l = l0 + i <= lmax ? gc[i] : zero, s_l = l0 + i <= lmax ? gs[i] : zero;
                ac += c_l * yl;
                bc += c_l * dl;
                as += s_l * yl;
                bs += s_l * dl;
            }
        }
        if (m == 0) {
            vz += bc;
        } else {
            const S fm = S(m);
            vx += fm * (ac * cp + as * sp);
            vy += fm * (as * cp - ac * sp);
            vz += bc * c + bs * s;
        }
        for (int k = 0; k < kRecParts; ++k) step();
    }
}

// The sum of the parts, from v(part).
template <typename GetPart>
__host__ __device__ __forceinline__ auto grad_unit_rec_sum(GetPart&& v)
{
    static_assert(kRecParts == 4, "two pairs");
    return (v(0) + v(1)) + (v(2) + v(3));
}

// All of v by one lane: the same sum, a pair at a time.
template <typename T, int UNROLL = 2, typename GAt>
__host__ __device__ __forceinline__ void grad_unit_rec(T x, T y, T z, int lmax, GAt&& g, T& vx, T& vy, T& vz)
{
#pragma unroll 1
    for (int p = 0; p < kRecParts; p += 2) {
        T ax, ay, az, bx, by, bz;
        grad_unit_rec_part<T, UNROLL>(x, y, z, lmax, p, g, ax, ay, az);
        grad_unit_rec_part<T, UNROLL>(x, y, z, lmax, p + 1, g, bx, by, bz);
        vx = p == 0 ? ax + bx : vx + (ax + bx);
        vy = p == 0 ? ay + by : vy + (ay + by);
        vz = p == 0 ? az + bz : vz + (az + bz);
    }
}

// Complex harmonics (Condon-Shortley phase) from the recurrence's real values, as
// complex_unit does for the explicit ones: Y_l^0 = R_l^0, and for m > 0
//     Y_l^m = (-1)^m (R_l^m + i R_l^-m) / sqrt(2),   Y_l^-m = (R_l^m - i R_l^-m) / sqrt(2);
// sink(l, m, re, im).
template <typename T, int UNROLL = 4, typename Sink>
__host__ __device__ __forceinline__ void complex_unit_rec(T x, T y, T z, T keep, int lmax, Sink&& sink)
{
    using S = scalar_t<T>;
    const T h = T(S(0.70710678118654752440));  // 1/sqrt(2)
    T cos_part = T(S(0));
    eval_unit_rec<T, UNROLL>(x, y, z, keep, lmax, [&](int l, int m, T v) {
        if (m == 0) {
            sink(l, 0, v, T(S(0)));
        } else if (m > 0) {
            cos_part = v;  // R_l^m arrives just before R_l^-m
        } else {
            const T re = h * cos_part, im = h * v;
            if (-m & 1) sink(l, -m, -re, -im);
            else sink(l, -m, re, im);
            sink(l, m, re, -im);
        }
    });
}

// Spinor harmonics (eq. spinorial) from complex_unit_rec, with the coefficient
// table of sh_rec_constants.h; sink(k, c, re, im) as for spinor_unit.
template <typename T, int UNROLL = 4, typename Sink>
__host__ __device__ __forceinline__ void spinor_unit_rec(T x, T y, T z, T keep, int lmax, Sink&& sink)
{
    complex_unit_rec<T, UNROLL>(x, y, z, keep, lmax, [&](int l, int m, T re, T im) {
        spinor_spread(l, m, re, im, [](int ll, int q) { return shc::kSpinP[ll][q]; }, sink);
    });
}

// How a forward launch by recurrence is shaped.
struct RecShape {
    bool wide;   // 16 bytes of adjacent points per lane and row, else one point
    bool split;  // the m of a point dealt to four waves
    int unroll;  // degrees at a time: 1, 4 or 8
    size_t lds;  // reserved
};
constexpr int64_t kRecSplitPoints = int64_t(1) << 16, kRecCapPoints = int64_t(1) << 19;
constexpr int64_t kRecThrottleBytes = int64_t(23) << 24;
inline size_t rec_lds(int64_t n, bool lines) { return !lines && n >= kRecCapPoints ? kCapLds1 : kCapLds2; }

// Real harmonics of n points, `bytes` written (us, points per lane / KiB of LDS reserved):
//   below 2^16 points  the m dealt to four waves, whatever is written: such a launch is one chain
//                      of work long: 10001 points, lmax 16 FP64 26.9 -> 8.6, FP32 25.3 -> 7.4; 60000,
//                      lmax 16 FP64 27.9 against 2/54 35.6, 30000, lmax 24 30.2 / 62.5, FP32 60000 32.3
//                      / 64.2
//   then one point     FP64 up to 5 x 2^14 points, FP32 to 2^17 (where several leave CUs idle):
//                      lmax 20, 65537 44.6 / 2/54 49.7, FP32 lmax 24, 100000 51.2 / 4/54 65.1; and
//                      below 2^27 bytes, FP32 from 3 x 2^16 points below 3 x 2^25: lmax 10, 262144 26.7 /
//                      4/54 23.0, 170001 16.8 / 19.5, lmax 12, 170001 22.0 / 23.6
//   wide               200001 points, lmax 16 FP64 2/54 88, 2/84 114 (one workgroup per CU
//                      leaves a short last round); FP32 4/54 47; 4000000 FP64 2/54 1730,
//                      2/84 1761; off the lines from 2^19 points 2/84: 1000001 points, lmax 16 FP64 485,
//                      2/54 500, 1/0 598; FP32, 2000001 4/84 473, 4/54 515
//   FP64, 23 x 2^24    resident all at once, the waves meet in the write path: four degrees at a
//   bytes and more     time are slower than one.  Up to 33 x 2^12 points eight with one point per lane:
//                      lmax 24, 106001 2/54 x 4 144, 1/0 x 8 110, lmax 20, 131072 104 / 84; to 3 x 2^16 one
//                      with two: lmax 20, 163840 119 / 112, 188001 127 / 121; then four: 204801 132, one 146
template <typename TIO>
inline RecShape rec_shape(int64_t n, int64_t bytes, bool lines)
{
    constexpr bool f64 = sizeof(TIO) == 8;
    if (n < kRecSplitPoints) return {false, true, 4, 0};
    if (f64 && bytes >= kRecThrottleBytes && n <= int64_t(3) << 16)
        return n < int64_t(33) << 12 ? RecShape{false, false, 8, 0} : RecShape{true, false, 1, kCapLds2};
    const bool wide = f64 ? n > int64_t(5) << 14 && bytes >= kWideBytes
                          : (n > int64_t(1) << 17 && bytes >= kWideBytes) ||
                                (n >= int64_t(3) << 16 && bytes >= 3 * (kWideBytes >> 2));
    return wide ? RecShape{true, false, 4, rec_lds(n, lines)} : RecShape{false, false, 4, 0};
}

// Complex and spinor harmonics.  FP32 takes several points from 2^16 on, where the CUs no longer
// hold one per lane in one round (spinor lmax 16, 14514 points 90.6 against 102; complex lmax 24, 30000
// 58.4 / 67.5; lmax 20, 80001 66.5 / 55.7).  FP64 (one point, 16 bytes) unrolls as the real harmonics:
// complex lmax 24, 57001 points x 4 154, x 8 120, 90001 x 4 175, x 1 162, 106001 x 4 201, x 1 216; spinor
// lmax 24, 30001 x 4 302, x 8 285, lmax 16, 65537 x 4 247, x 8 272.
template <typename TIO, bool SPINOR>
inline RecShape rec_cplx_shape(int64_t n, int64_t bytes, bool lines)
{
    if (bytes < kWideBytes) return {false, false, 4, 0};
    if (sizeof(TIO) == 4 && n <= kRecSplitPoints) return {false, false, 4, 0};
    int unroll = 4;
    if (sizeof(TIO) == 8 && bytes >= kRecThrottleBytes) {
        if (n <= (SPINOR ? kRecSplitPoints : int64_t(5) << 14)) unroll = 8;
        else if (!SPINOR && n <= int64_t(3) << 15) unroll = 1;
    }
    return {true, false, unroll, rec_lds(n, lines)};
}

// How a backward launch by recurrence is shaped.
struct GradRecShape {
    int ppl;     // adjacent points per lane
    bool split;  // the m of a point dealt to four waves
    int unroll;  // degrees whose reads are issued together
};
constexpr int64_t kGradRecNarrow = int64_t(1) << 16;

// Bound by the reads of G (us, SPLIT or whole, points per lane x degrees):
//   below 2^16 points  10001, lmax 16: FP64 split 1 x 8 11.0, 1 x 2 16.6, 2 x 2 18.9; FP32 10.1, 15.0, 17.7
//   then, split 2 x 2  lmax 16, 130001 FP64 50.9 / whole 1 x 2 69; FP32 24.6 / 40.7; 800001 FP32 178 / whole
//                      4 x 2 204
//   FP64 from 2^18     lmax 16, 400001 whole 2 x 1 153, 1 x 1 155, 2 x 2 170-175, 1 x 2 182; 2000001, lmax 10 340 /
//                      347 / 364 / 405 (held to 128 registers, four waves a SIMD; 238 against 208 at 130
//                      registers); up to 5 x 2^16, where all lanes are resident with one point each, whole 1 x 2:
//                      lmax 9, 270001 42.0, 2 x 1 44.5.  Few rows, 1 x 1: lmax 1, 4000001 54.5, 2 x 1 69,
//                      2 x 2 67-75, lmax 4 174 / 180 / 192, lmax 7, 400001 37.5 / 38.9 / 43
//   FP32 from 2^20     lmax 16, 2000001 whole 4 x 2 389, 2 x 2 433, 1 x 2 463.  Up to lmax 3 from 2^19 whole
//                      1 x 2: lmax 1, 1000001 9.2 / split 12.5, 4000001 27.5 / 4 x 2 32.9; lmax 4, 4000001
//                      102 / 101
template <typename TIO>
inline GradRecShape grad_rec_shape(int lmax, int64_t n)
{
    if (n < kGradRecNarrow) return {1, true, 8};
    if constexpr (sizeof(TIO) == 8) {
        if (n < int64_t(1) << 18) return {2, true, 2};
        if (lmax < 8) return {1, false, 1};
        return n < int64_t(5) << 16 ? GradRecShape{1, false, 2} : GradRecShape{2, false, 1};
    } else {
        if (n < int64_t(1) << (lmax < 4 ? 19 : 20)) return {2, true, 2};
        return lmax < 4 ? GradRecShape{1, false, 2} : GradRecShape{4, false, 2};
    }
}

}  // namespace shk
