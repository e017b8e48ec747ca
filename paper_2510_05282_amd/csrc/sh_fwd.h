// sh_fwd.h -- the forward kernel template (all real Y_lm of a batch of points).
//
// Each lane evaluates PPL adjacent points at once (the formula core runs on a
// PPL-wide clang vector), so every (l, m) row gets one PPL * sizeof(T) byte
// store per lane and one contiguous 64 * PPL * sizeof(T) byte run per wave.
// Points are normalised in FP64 whatever the output type.
//
// Work distribution is XCD-aware: the hardware deals consecutive workgroups
// round-robin to the 8 XCDs, so workgroup b is remapped to the logical tile
// start(b % 8) + b / 8, giving each XCD one contiguous range of points.  The
// points that are being written at any moment then stay within a few compact
// windows of every output row, which the HBM write path rewards measurably.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sh_core.h"

namespace shk {

constexpr int kFwdBlock = 256;
constexpr int kCus = 256;  // of the GPU

template <typename S, int N> struct vec_of { typedef S type __attribute__((ext_vector_type(N))); };
template <typename S> struct vec_of<S, 1> { typedef S type; };

// The same aligned only as its elements: a 16-byte access of it is one instruction at any
// element address.
template <typename S, int N> struct uvec_of { typedef S type __attribute__((ext_vector_type(N), aligned(sizeof(S)))); };
template <typename S> struct uvec_of<S, 1> { typedef S type; };

template <typename V, int PPL>
__device__ __forceinline__ auto& lane(V& v, int k)
{
    if constexpr (PPL == 1) return v;
    else return reinterpret_cast<scalar_t<V>*>(&v)[k];
}

// How a launch that stores rows of values is shaped, from what it writes.
struct StoreShape {
    bool wide;   // 16 bytes (or more) of adjacent points per lane and row, else one point
    size_t lds;  // LDS reserved (not used) per 256-thread workgroup
};

// LDS reservations out of a CU's 160 KiB: at most 4, 2 or 1 resident workgroups.
constexpr size_t kCapLds4 = 40 * 1024, kCapLds2 = 54 * 1024, kCapLds1 = 84 * 1024;

// Whether rows that start at p and lie row_bytes apart all start on a 128-byte line.
inline bool on_lines(const void* p, int64_t row_bytes)
{
    return row_bytes % 128 == 0 && reinterpret_cast<uintptr_t>(p) % 128 == 0;
}

// The shape of a launch over n points that writes ROWS rows of `value` bytes a point, for the
// real, complex and spinor harmonics and the Jacobian; in_bytes a point are read (0: not
// counted).  Small outputs stay in the caches on their way out, and such a launch lasts its
// workgroups' chain of work, which wide lanes lengthen; large ones are bound by the HBM write
// path, which rewards wide stores and, from 16 rows on, few waves at once: the writes under way
// to each row then lie in a smaller window, and the partial lines that neighbouring waves write
// where rows do not start on lines merge in the L2.  Measured in us as points per lane / KiB
// reserved, two or three outputs in turn, "odd" where rows lie off the lines:
//  one round           a launch of one point per lane that the CUs hold in one round halves
//                      its workgroups with two: Jacobian lmax 9, 42368 points 1/0 27.8, 2/0 28.7,
//                      60032 37.1 / 38.3, odd 45001 31.5 / 31.8, 66048 46.4 / 41.3; FP32 spinor lmax
//                      8, 56064 28.0 / 29.5
//  1 row               FP32 15M points 4/0 10.3, 4/54 12.4, 1/0 16.6, 25M 16.2, 18.2, 25.1, 4M 6.9,
//                      6.9, 7.4; FP64 7.5M 2/0 10.3, 1/0 11.0
//  4 rows              2^25 points FP64 1/40 307, 1/0 328, 2/54 321; FP32 1/0 156, 4/54
//                      184; complex 8000001 FP64 1/40 126, 1/54 155, FP32 1/0 67, 2/54 86
//  below 2^27 bytes    FP64 lmax 6, 255000 points (100 MB) 1/0 19.1, 2/54 19.6; FP32 lmax 5,
//                      798592 (115 MB) 24.4, 24.8; lmax 9, 2^17 9.7, 10.8; complex FP64 lmax 9,
//                      50001 1/0 13.7, 2/0 21.6
//  read and written    on lines it is what is read and written that leaves the caches: 9 rows
//                      FP64 115 MB written 1/0 30.6, 2/54 29.7, 133 MB 38.5, 37.1, 100 MB 20.1, 20.9; 16
//                      rows FP64 133 MB 1/0 33.9, 2/0 29.5, FP32 34.2, 4/54 32.0; 25 rows FP32 133 MB
//                      30.0, 4/54 26.2; 36 rows FP64 133 MB 24.8, 22.9; Jacobian lmax 2 133 MB 23.6, 22.6
//  9 rows              2^25 points FP64 2/54 563, 2/0 608, 2/84 582; FP32 4/54 283, 4/84
//                      324; complex 8000001 FP32 2/54 127, 1/0 141, 2/84 156
//  on lines,           below 2^29 bytes: FP64 lmax 9, 2^19 2/0 77.2, 2/84 80.4; FP32 lmax
//  16 rows and more    5, 2^21 4/0 61.3, 4/84 63.6; complex FP64 lmax 6, 250000 1/0 38.0,
//                      1/54 39.3, but FP32 lmax 3, 180 MB 4/0 43.5, 4/54 42.2, into one output 33.8,
//                      32.2.  Above: 16 rows FP64 800 MB 2/84 178, 2/54 184, FP32 173, 183, complex
//                      lmax 3 FP32 164, 173, FP64 168, 172, spinor lmax 1 165, 173 and 168, 171, Jacobian
//                      lmax 1 180, 183; FP64 lmax 4, 2^25 points 1386, 1375, lmax 9 at 2^26 68.4% of
//                      8 TB/s against 67.8%, but complex FP64 lmax 9, 560 MB 111, 108, FP32 equal
//  off the lines,      below 5 x 2^25 bytes: FP64 lmax 7, 137 MB 1/0 23.4, 2/0 23.9, 2/84 26.0, lmax
//  16 rows and more    5, 150 MB 37.8, 32.6, 36.5; FP32 lmax 7 137 MB 24.6, 24.7, 27.5; complex FP64
//                      lmax 3, 137 MB 1/0 25.9, 1/84 30.9; FP32 spinor lmax 1 28.6, 27.2, 30.3; but
//                      FP64 lmax 3, 150 MB 42.0, 39.1, 38.8, of three outputs 41.5, 41.4, 37.0, FP32
//                      lmax 3 43.9, 39.4, 4/54 39.6, of one 27.1, 29.0, 4/54 27.3.  Above: FP64 lmax
//                      3, 220 MB 2/84 50.0, 2/0 57.5, lmax 9, 2^22 + 1 points 661, 783, 2/54 748;
//                      FP32 lmax 8, 2^23 + 3 4/84 532, 4/54 594, 1/0 820; complex lmax 9, 1000001
//                      FP64 1/84 328, 1/54 337, FP32 2/84 166, 1/0 191; Jacobian lmax 9, 1000001
//                      2/84 651, 2/54 708, 1/0 813
// A caller that writes one output again and again, below 220 MB, is served by the memory-side
// cache, where off the lines one point per lane stays ahead by 1 to 5% (FP64 lmax 3, 150 MB
// 26.6 / 27.4, FP32 lmax 4 25.4 / 26.7); the lines are drawn for two outputs in turn, as
// a new output for every call makes them.
constexpr int64_t kWideBytes = int64_t(1) << 27, kOffBytes = int64_t(5) << 25, kCapBytes = int64_t(1) << 29;
constexpr int64_t kOneRound = int64_t(kCus) * kFwdBlock;

template <int ROWS, typename TIO>
inline StoreShape store_shape(int64_t n, int value, int in_bytes, bool lines)
{
    const int64_t bytes = n * ROWS * value;
    if (ROWS == 1) return {bytes >= kWideBytes / 16, 0};
    if (ROWS <= 4) return {false, sizeof(TIO) == 8 && bytes >= kWideBytes ? kCapLds4 : 0};
    if (n <= kOneRound || bytes + (lines && ROWS <= 49 ? n * in_bytes : 0) < kWideBytes) return {false, 0};
    if (ROWS <= 9) return {true, kCapLds2};
    const bool real = value == int(sizeof(TIO)), one16 = ROWS == 16 && real && sizeof(TIO) == 8;
    if (bytes < (lines ? kCapBytes : (one16 ? 0 : kOffBytes))) {
        const bool two = real && sizeof(TIO) == 4 && (ROWS == 16 || (ROWS == 25 && lines && bytes < kWideBytes));
        return {true, two ? kCapLds2 : 0};
    }
    return {true, !lines || ROWS == 16 || (ROWS > 64 && ROWS <= 100 && value == 8 && sizeof(TIO) == 8) ? kCapLds1
                                                                                                      : kCapLds2};
}

// How the explicit backward kernel reads G and orders its workgroups (one point per lane: two,
// or four in FP32, are equal or up to 25% slower below 400 MB of G and within 5% above).
//  kCached   small: loads that keep lines, XCD-contiguous order, no cap.  G, which a caller has
//            usually just written, is then in the memory-side cache, with what else a step
//            touches.  us for a forward call, G = 2 y and the backward call, against kStream,
//            FP64: lmax 9, 100 MB of G 62.7 / 63.6, 130 MB 82.5 / 87.6, 160 MB 114.7 / 110.2,
//            195 MB 144 / 131; lmax 3, 133 MB 101 / 94; lmax 2, 92 MB 67.5 / 69.1, 133 MB 119 / 103;
//            lmax 1, 85 MB 79.2 / 81.2, 105 MB 106 / 100; lmax 0, 60 MB 103 / 99; FP32 lmax 2, 125 MB
//            93.8 / 98.4, lmax 1, 195 MB 194 / 222.  (One G read over and over, and little else, is
//            15-25% faster as kCached up to 190 MB.)
//  kStream   larger: non-temporal loads, plain order, at most 4 resident workgroups per CU.
//            us, rows on 128-byte lines, FP64 lmax 6, 2000000 147 against 158 with loads that
//            keep lines and 167 as kCached; FP32 145 / 156 / 167
//  kShared   from kGradSharedBytes and lmax 3, rows off the lines: as kStream with loads that keep
//            lines, as neighbouring waves read parts of the same ones.  FP64 lmax 6, 4194301 331
//            against 364 streaming, lmax 8, 2000001 250 / 260; FP32 lmax 8, 4000001 247 /
//            270; but FP64 lmax 2, 8000001 153 / 149, lmax 5, 1000001 (288 MB) 61 / 58
enum class GRead { kCached, kStream, kShared };
constexpr int64_t kGradSharedBytes = int64_t(1) << 29;

template <int LMAX, typename TIO>
inline GRead grad_read(int64_t n, bool lines)
{
    constexpr int64_t f64_lines[] = {int64_t(3) << 24, int64_t(11) << 23, int64_t(3) << 25, int64_t(15) << 23};
    constexpr int64_t f32_lines[] = {int64_t(3) << 26, int64_t(3) << 26, int64_t(15) << 23, int64_t(15) << 23};
    constexpr int64_t cached = LMAX >= 4 ? int64_t(1) << 27 : (sizeof(TIO) == 8 ? f64_lines : f32_lines)[LMAX];
    const int64_t bytes = n * nfun(LMAX) * int64_t(sizeof(TIO));
    if (bytes < cached) return GRead::kCached;
    return LMAX >= 3 && bytes >= kGradSharedBytes && !lines ? GRead::kShared : GRead::kStream;
}

// First point of lane `t` of a launch whose lanes take PPL adjacent points of n >= PPL
// (t * PPL < n): where PPL does not divide n the last lane takes the last PPL points,
// some of which the lane before it takes too, and both store the same bits.
template <int PPL>
__device__ __forceinline__ uint32_t first_point(uint32_t t, uint32_t n)
{
    return t * PPL + PPL <= n ? t * PPL : n - PPL;
}

// The paper's three input interfaces (Section 2): Cartesian points (normalised
// here), points already on the unit sphere, and the angles (theta, phi).
enum class In { kXyz, kUnit, kAngles };

// Unit vector (in FP64) and origin mask of point i of the input.
template <In MODE, typename TIO>
__device__ __forceinline__ void load_unit(const TIO* __restrict__ a, const TIO* __restrict__ b, uint32_t i,
                                          double& xb, double& yb, double& zb, double& kb)
{
    if constexpr (MODE == In::kXyz) {
        const TIO* p = a + 3 * size_t(i);
        normalize(double(p[0]), double(p[1]), double(p[2]), xb, yb, zb, kb);
    } else if constexpr (MODE == In::kUnit) {
        const TIO* p = a + 3 * size_t(i);
        xb = double(p[0]);
        yb = double(p[1]);
        zb = double(p[2]);
        kb = 1.0;
    } else {
        double st, ct, sp, cp;
        sincos(double(a[i]), &st, &ct);
        sincos(double(b[i]), &sp, &cp);
        xb = st * cp;
        yb = st * sp;
        zb = ct;
        kb = 1.0;
    }
}

// out is [F][ld]; the input is xyz [n][3] (kXyz, kUnit) or theta = xyz[n],
// phi = in1[n] (kAngles); n * sizeof(TIO) < 2^31 so per-row byte offsets
// fit 32 bits (the host splits larger batches).  With PPL > 1 the host
// guarantees n >= PPL; ld and out need no alignment beyond the element's (first_point).
template <int LMAX, typename TIO, int PPL, In MODE = In::kXyz>
__global__ __launch_bounds__(kFwdBlock) void fwd_kernel(const TIO* __restrict__ xyz, TIO* __restrict__ out,
                                                        uint32_t n, int64_t ld, const TIO* __restrict__ in1)
{
    using V = typename vec_of<TIO, PPL>::type;
    const uint32_t b = xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t t = b * kFwdBlock + threadIdx.x;  // vector index
    if (t * PPL >= n) return;
    const uint32_t i0 = first_point<PPL>(t, n);
    V x, y, z, k;
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        double xb, yb, zb, kb;
        load_unit<MODE, TIO>(xyz, in1, i0 + q, xb, yb, zb, kb);
        lane<V, PPL>(x, q) = TIO(xb);
        lane<V, PPL>(y, q) = TIO(yb);
        lane<V, PPL>(z, q) = TIO(zb);
        lane<V, PPL>(k, q) = TIO(kb);
    }
    const uint32_t boff = i0 * uint32_t(sizeof(TIO));
    eval_unit<LMAX, V>(x, y, z, k, [&](int r, V v) {
        *reinterpret_cast<typename uvec_of<TIO, PPL>::type*>(reinterpret_cast<char*>(out + int64_t(r) * ld) + boff) = v;
    });
}

// Loads PPL adjacent points (from point i0) as unit vectors in V lanes; the input
// interface is chosen at run time (the same for the whole launch).
template <typename TIO, int PPL, typename V>
__device__ __forceinline__ void load_points(const TIO* __restrict__ in0, const TIO* __restrict__ in1, In mode,
                                            uint32_t i0, V& x, V& y, V& z, V& k)
{
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        double xb, yb, zb, kb;
        if (mode == In::kXyz) load_unit<In::kXyz, TIO>(in0, in1, i0 + q, xb, yb, zb, kb);
        else if (mode == In::kUnit) load_unit<In::kUnit, TIO>(in0, in1, i0 + q, xb, yb, zb, kb);
        else load_unit<In::kAngles, TIO>(in0, in1, i0 + q, xb, yb, zb, kb);
        lane<V, PPL>(x, q) = TIO(xb);
        lane<V, PPL>(y, q) = TIO(yb);
        lane<V, PPL>(z, q) = TIO(zb);
        lane<V, PPL>(k, q) = TIO(kb);
    }
}

// PPL complex values (re, im interleaved, PPL adjacent points) as one vector.
template <typename TIO, int PPL, typename V>
__device__ __forceinline__ typename vec_of<TIO, 2 * PPL>::type interleave(V re, V im)
{
    typename vec_of<TIO, 2 * PPL>::type w;
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        w[2 * q] = lane<V, PPL>(re, q);
        w[2 * q + 1] = lane<V, PPL>(im, q);
    }
    return w;
}

// Complex harmonics from the real ones (Section 3, complex_unit): out[row][i] as
// (re, im) pairs, [F][ld] complex.  Each lane evaluates PPL adjacent points and
// stores their PPL complex values of a row at once: 16 bytes per lane and row for
// FP64 with PPL = 1 and FP32 with PPL = 2.  With PPL > 1 the host guarantees n >= PPL
// (first_point); ld and out need only the element's alignment.  Inputs as for fwd_kernel:
// in0 = xyz [n][3] (kXyz, kUnit) or theta[n] and in1 = phi[n] (kAngles).
template <int LMAX, typename TIO, int PPL>
__global__ __launch_bounds__(kFwdBlock) void fwd_complex_kernel(const TIO* __restrict__ in0,
                                                                TIO* __restrict__ out, uint32_t n, int64_t ld,
                                                                const TIO* __restrict__ in1, In mode)
{
    using V = typename vec_of<TIO, PPL>::type;
    using W = typename uvec_of<TIO, 2 * PPL>::type;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x) * kFwdBlock + threadIdx.x;
    if (t * PPL >= n) return;
    const uint32_t i0 = first_point<PPL>(t, n);
    V x, y, z, k;
    load_points<TIO, PPL>(in0, in1, mode, i0, x, y, z, k);
    const uint32_t boff = i0 * uint32_t(2 * sizeof(TIO));
    complex_unit<LMAX, V>(x, y, z, k, [&](int l, int m, V re, V im) {
        *reinterpret_cast<W*>(reinterpret_cast<char*>(out + 2 * int64_t(row(l, m)) * ld) + boff) =
            interleave<TIO, PPL>(re, im);
    });
}

// Spinor harmonics (eq. spinorial): spinor_unit's values, stored as they come to
// out[(2 s + c) ld + i] as (re, im) pairs (c = 0 for the upper component), with
// the same lanes as the complex kernel.
template <int LMAX, typename TIO, int PPL>
__global__ __launch_bounds__(kFwdBlock) void fwd_spinor_kernel(const TIO* __restrict__ in0,
                                                               TIO* __restrict__ out, uint32_t n, int64_t ld,
                                                               const TIO* __restrict__ in1, In mode)
{
    using V = typename vec_of<TIO, PPL>::type;
    using W = typename uvec_of<TIO, 2 * PPL>::type;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x) * kFwdBlock + threadIdx.x;
    if (t * PPL >= n) return;
    const uint32_t i0 = first_point<PPL>(t, n);
    V x, y, z, k;
    load_points<TIO, PPL>(in0, in1, mode, i0, x, y, z, k);
    const uint32_t boff = i0 * uint32_t(2 * sizeof(TIO));
    spinor_unit<LMAX, V>(x, y, z, k, [&](int s, int c, V re, V im) {
        *reinterpret_cast<W*>(reinterpret_cast<char*>(out + 2 * int64_t(2 * s + c) * ld) + boff) =
            interleave<TIO, PPL>(re, im);
    });
}

}  // namespace shk
