// sh_rec.hip -- real harmonics beyond l = 9 by recurrence.
//
// The explicit formulas stop at l = 9; the paper's conclusion points to
// recurrence relations for higher orders.  On the unit vector u = (x, y, z),
//     R_l^0 = Yb_l^0(z),  R_l^{+m} = Yb_l^m(z) C_m(x, y),  R_l^{-m} = Yb_l^m(z) S_m(x, y),
// with C_m + i S_m = (x + i y)^m (built by repeated complex multiplication) and
// Yb_l^m(z) = sqrt(2)^[m>0] N_lm d^m P_l/dz^m, the normalised associated Legendre
// functions with the sin^m factor moved into C_m, S_m.  They follow the stable
// normalised recurrences
//     Yb_m^m     = d_m,  d_0 = 1/sqrt(4 pi),  d_m = d_{m-1} sqrt((2m+1)/(2m)) (x sqrt(2) at m = 1),
//     Yb_{m+1}^m = sqrt(2m+3) z Yb_m^m,
//     Yb_l^m     = a_lm (z Yb_{l-1}^m - b_lm Yb_{l-2}^m),
//     a_lm = sqrt((4l^2 - 1)/(l^2 - m^2)),  b_lm = sqrt(((l-1)^2 - m^2)/(4(l-1)^2 - 1)),
// whose coefficients are generated once (gen_rec_constants.py, 50-digit mpmath),
// so the kernel does no square roots or divisions.  Same normalisation, origin
// guard and [F][ld] layout as the explicit kernels, FP64 or FP32 (normalisation
// in FP64 either way), lmax up to SH_LMAX_REC.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/shmi.h"
#include "sh_core.h"
#include "sh_fwd.h"
#include "sh_internal.h"
#include "sh_rec.h"

namespace shk {

static_assert(shc::kRecLmax == SH_LMAX_REC, "recurrence tables and the public limit disagree");

constexpr int kRecBlock = 256;
constexpr int64_t kRecChunk = int64_t(1) << 28;

// TIO = double: up to 2 points per lane (PPL = 2); float: 4 (PPL = 4); both then store
// 16 bytes per lane and row.  Points are normalised in FP64 either way.  SPLIT: the
// workgroup takes 64 lanes' worth of points and deals their m to its four waves.
template <typename TIO, int PPL, bool SPLIT, int UNROLL>
__global__ __launch_bounds__(kRecBlock) void rec_kernel(const TIO* __restrict__ xyz, TIO* __restrict__ out,
                                                        uint32_t n, int64_t ld, int lmax)
{
    using V = typename vec_of<TIO, PPL>::type;
    using U = typename uvec_of<TIO, PPL>::type;
    constexpr int kLanes = SPLIT ? 64 : kRecBlock;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x) * kLanes + threadIdx.x % kLanes;
    if (t * PPL >= n) return;
    const uint32_t i0 = first_point<PPL>(t, n);
    V x, y, z, k;
    load_points<TIO, PPL>(xyz, nullptr, In::kXyz, i0, x, y, z, k);
    const uint32_t boff = i0 * uint32_t(sizeof(TIO));
    auto store = [&](int l, int m, V v) {
        *reinterpret_cast<U*>(reinterpret_cast<char*>(out + int64_t(row(l, m)) * ld) + boff) = v;
    };
    const int part = SPLIT ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    eval_unit_rec<V, UNROLL>(x, y, z, k, lmax, store, part, SPLIT ? kRecBlock / 64 : 1);
}

template <typename TIO, int PPL, bool SPLIT, int UNROLL>
static hipError_t launch_rec_one(int lmax, int64_t n, const TIO* xyz, TIO* out, int64_t ld, hipStream_t s, size_t lds)
{
    constexpr int kLanes = SPLIT ? 64 : kRecBlock;
    const unsigned grid = unsigned(((n + PPL - 1) / PPL + kLanes - 1) / kLanes);
    hipLaunchKernelGGL((rec_kernel<TIO, PPL, SPLIT, UNROLL>), dim3(grid), dim3(kRecBlock), lds, s, xyz, out,
                       uint32_t(n), ld, lmax);
    return hipGetLastError();
}

template <typename TIO>
hipError_t launch_rec(int lmax, int64_t n, const TIO* xyz, TIO* out, int64_t ld, hipStream_t s)
{
    constexpr int kVec = 16 / sizeof(TIO);
    const RecShape f = rec_shape<TIO>(n, n * nfun(lmax) * int64_t(sizeof(TIO)), on_lines(out, ld * sizeof(TIO)));
    for (int64_t c0 = 0; c0 < n; c0 += kRecChunk) {
        const int64_t nc = n - c0 < kRecChunk ? n - c0 : kRecChunk;
        const TIO* x = xyz + 3 * c0;
        TIO* o = out + c0;
        const hipError_t e =
            f.split                  ? launch_rec_one<TIO, 1, true, 4>(lmax, nc, x, o, ld, s, f.lds)
            : !f.wide || nc < kVec
                ? (f.unroll == 8 ? launch_rec_one<TIO, 1, false, 8>(lmax, nc, x, o, ld, s, f.lds)
                                 : launch_rec_one<TIO, 1, false, 4>(lmax, nc, x, o, ld, s, f.lds))
            : f.unroll == 1          ? launch_rec_one<TIO, kVec, false, 1>(lmax, nc, x, o, ld, s, f.lds)
                                     : launch_rec_one<TIO, kVec, false, 4>(lmax, nc, x, o, ld, s, f.lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template hipError_t launch_rec<double>(int, int64_t, const double*, double*, int64_t, hipStream_t);
template hipError_t launch_rec<float>(int, int64_t, const float*, float*, int64_t, hipStream_t);

// Backward pass by recurrence: the vector-Jacobian product of sh_eval_rec,
//     g = (1/r) (v - u (u . v)),   v = sum_rows G[row] grad_u P_row(u),
// as the explicit backward kernel, with v from grad_unit_rec (the recurrence
// differentiated in z, the xy factors by their closed-form partials).  PPL adjacent
// points per lane, whose values of a row of G are one read at any alignment; UNROLL
// degrees' reads issued together; workgroups in XCD-contiguous order; the normalisation
// and 1/r in FP64.  SPLIT: a workgroup takes 64 lanes' worth of points, its four waves a
// quarter of the m each, and one wave adds the four sums up; otherwise a lane goes
// through the quarters itself.  The sums are the same either way.
// Bound by the reads of G, and by their latency wherever few waves have few reads under
// way: with every read waited for before the next and no split, 200001 points at lmax 16
// took 124 us in FP64 (3.8 TB/s) and 110 in FP32 (2.1), 10001 points 84 and 75; now 81
// (5.8 TB/s), 47 (5.0), 11 and 10.  grad_rec_shape says which launch.  FP32's split launches are
// held to 72 registers, seven waves a SIMD: 400001 points at lmax 9 26.3 us, 28.6 at six waves.
template <typename TIO, bool SPLIT>
constexpr int kGradRecWaves = sizeof(TIO) == 8 ? (SPLIT ? 1 : 4) : (SPLIT ? 7 : 1);  // a SIMD, at least

template <typename TIO, int PPL, bool SPLIT, int UNROLL, bool NT>
__global__ __launch_bounds__(kRecBlock, (kGradRecWaves<TIO, SPLIT>)) void grad_rec_kernel(
    const TIO* __restrict__ xyz, const TIO* __restrict__ G, TIO* __restrict__ gxyz, uint32_t n, int64_t ldg, int lmax)
{
    using V = typename vec_of<TIO, PPL>::type;
    using U = typename uvec_of<TIO, PPL>::type;
    static_assert(kRecBlock == 64 * kRecParts, "one wave per part");
    constexpr int kLanes = SPLIT ? 64 : kRecBlock;  // lanes' worth of points per workgroup
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x) * kLanes + threadIdx.x % kLanes;
    const bool live = t * PPL < n;
    if (!SPLIT && !live) return;
    const uint32_t i0 = live ? first_point<PPL>(t, n) : 0;
    double xb[PPL], yb[PPL], zb[PPL], rinv[PPL];
    V x, y, z;
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        const TIO* p = xyz + 3 * size_t(i0 + q);
        double keep;  // not needed: rinv = 0 at the origin, so the gradient is 0 there
        normalize(double(p[0]), double(p[1]), double(p[2]), xb[q], yb[q], zb[q], keep, rinv[q]);
        lane<V, PPL>(x, q) = TIO(xb[q]);
        lane<V, PPL>(y, q) = TIO(yb[q]);
        lane<V, PPL>(z, q) = TIO(zb[q]);
    }
    const uint32_t boff = i0 * uint32_t(sizeof(TIO));
    auto g_at = [&](int r) {
        const U* g = reinterpret_cast<const U*>(reinterpret_cast<const char*>(G + int64_t(r) * ldg) + boff);
        return NT ? V(__builtin_nontemporal_load(g)) : V(*g);
    };
    V v[3];
    if constexpr (SPLIT) {
        __shared__ V parts[kRecParts][3][64];
        const int wl = threadIdx.x & 63, part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        grad_unit_rec_part<V, UNROLL>(x, y, z, lmax, part, g_at, v[0], v[1], v[2]);
#pragma unroll
        for (int k = 0; k < 3; ++k) parts[part][k][wl] = v[k];
        __syncthreads();
        if (part != 0 || !live) return;
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = grad_unit_rec_sum([&](int p) { return p == 0 ? v[k] : parts[p][k][wl]; });
    } else {
        grad_unit_rec<V, UNROLL>(x, y, z, lmax, g_at, v[0], v[1], v[2]);
    }
    // gxyz may be xyz: a last lane that read its neighbour's points too, which may be
    // gradients by then, stores only its own (only there is i0 no multiple of PPL)
    TIO* o = gxyz + 3 * size_t(i0);
    const int first = int(-i0 % PPL);
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        if (q < PPL - 1 && q < first) continue;
        const double gx = double(lane<V, PPL>(v[0], q)), gy = double(lane<V, PPL>(v[1], q)),
                     gz = double(lane<V, PPL>(v[2], q));
        const double uv = xb[q] * gx + yb[q] * gy + zb[q] * gz;
        o[3 * q + 0] = TIO(rinv[q] * (gx - xb[q] * uv));
        o[3 * q + 1] = TIO(rinv[q] * (gy - yb[q] * uv));
        o[3 * q + 2] = TIO(rinv[q] * (gz - zb[q] * uv));
    }
}

template <typename TIO, int PPL, bool SPLIT, int UNROLL, bool NT>
static hipError_t launch_grad_rec_one(int lmax, int64_t n, const TIO* xyz, const TIO* G, int64_t ldg, TIO* gxyz,
                                      hipStream_t s)
{
    constexpr int kLanes = SPLIT ? 64 : kRecBlock;
    const unsigned grid = unsigned(((n + PPL - 1) / PPL + kLanes - 1) / kLanes);
    hipLaunchKernelGGL((grad_rec_kernel<TIO, PPL, SPLIT, UNROLL, NT>), dim3(grid), dim3(kRecBlock), 0, s, xyz, G, gxyz,
                       uint32_t(n), ldg, lmax);
    return hipGetLastError();
}

template <typename TIO, bool NT>
static hipError_t launch_grad_rec_nt(int lmax, int64_t n, const TIO* xyz, const TIO* G, int64_t ldg, TIO* gxyz,
                                     hipStream_t s)
{
    constexpr int kVec = 16 / sizeof(TIO);
    const GradRecShape f = grad_rec_shape<TIO>(lmax, n);
    for (int64_t c0 = 0; c0 < n; c0 += kRecChunk) {
        const int64_t nc = n - c0 < kRecChunk ? n - c0 : kRecChunk;
        const TIO *x = xyz + 3 * c0, *g = G + c0;
        TIO* o = gxyz + 3 * c0;
        hipError_t e;
        if (f.unroll == 8 || nc < kVec) e = launch_grad_rec_one<TIO, 1, true, 8, NT>(lmax, nc, x, g, ldg, o, s);
        else if (f.split) e = launch_grad_rec_one<TIO, 2, true, 2, NT>(lmax, nc, x, g, ldg, o, s);
        else if (f.ppl == 1 && f.unroll == 2) e = launch_grad_rec_one<TIO, 1, false, 2, NT>(lmax, nc, x, g, ldg, o, s);
        else if constexpr (kVec == 4) e = launch_grad_rec_one<TIO, 4, false, 2, NT>(lmax, nc, x, g, ldg, o, s);
        else if (f.ppl == 1) e = launch_grad_rec_one<TIO, 1, false, 1, NT>(lmax, nc, x, g, ldg, o, s);
        else e = launch_grad_rec_one<TIO, 2, false, 1, NT>(lmax, nc, x, g, ldg, o, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// NT (non-temporal reads of G) from kReadCachedBytes on: lmax 16, 60001 points FP64 26.4 us
// without, 29.5 with, FP32 100000 20.9 / 24.5; 200000 FP64 (462 MB) 88.5 / 78.0, FP32
// 400000 89 / 79.
template <typename TIO>
hipError_t launch_grad_rec(int lmax, int64_t n, const TIO* xyz, const TIO* G, int64_t ldg, TIO* gxyz, hipStream_t s)
{
    return n * nfun(lmax) * int64_t(sizeof(TIO)) < kReadCachedBytes
               ? launch_grad_rec_nt<TIO, false>(lmax, n, xyz, G, ldg, gxyz, s)
               : launch_grad_rec_nt<TIO, true>(lmax, n, xyz, G, ldg, gxyz, s);
}

template hipError_t launch_grad_rec<double>(int, int64_t, const double*, const double*, int64_t, double*,
                                            hipStream_t);
template hipError_t launch_grad_rec<float>(int, int64_t, const float*, const float*, int64_t, float*, hipStream_t);

// Complex (SPINOR = false) or spinor harmonics by recurrence, any input interface:
// the lanes and layout of fwd_complex_kernel / fwd_spinor_kernel, lmax at run time.
template <typename TIO, int PPL, bool SPINOR, int UNROLL>
__global__ __launch_bounds__(kRecBlock) void rec_cplx_kernel(const TIO* __restrict__ in0, TIO* __restrict__ out,
                                                             uint32_t n, int64_t ld, const TIO* __restrict__ in1,
                                                             In mode, int lmax)
{
    using V = typename vec_of<TIO, PPL>::type;
    using W = typename uvec_of<TIO, 2 * PPL>::type;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x) * kRecBlock + threadIdx.x;
    if (t * PPL >= n) return;
    const uint32_t i0 = first_point<PPL>(t, n);
    V x, y, z, k;
    load_points<TIO, PPL>(in0, in1, mode, i0, x, y, z, k);
    const uint32_t boff = i0 * uint32_t(2 * sizeof(TIO));
    auto put = [&](int64_t r, V re, V im) {
        *reinterpret_cast<W*>(reinterpret_cast<char*>(out + 2 * r * ld) + boff) = interleave<TIO, PPL>(re, im);
    };
    if constexpr (SPINOR)
        spinor_unit_rec<V, UNROLL>(x, y, z, k, lmax, [&](int s, int c, V re, V im) { put(2 * s + c, re, im); });
    else
        complex_unit_rec<V, UNROLL>(x, y, z, k, lmax, [&](int l, int m, V re, V im) { put(row(l, m), re, im); });
}

template <typename TIO, int PPL, bool SPINOR, int UNROLL>
static hipError_t launch_rec_cplx_one(int lmax, int64_t n, In mode, const TIO* a, const TIO* b, TIO* out,
                                      int64_t ld, hipStream_t s, size_t lds)
{
    const unsigned grid = unsigned(((n + PPL - 1) / PPL + kRecBlock - 1) / kRecBlock);
    hipLaunchKernelGGL((rec_cplx_kernel<TIO, PPL, SPINOR, UNROLL>), dim3(grid), dim3(kRecBlock), lds, s, a, out,
                       uint32_t(n), ld, b, mode, lmax);
    return hipGetLastError();
}

template <typename TIO, bool SPINOR>
static hipError_t launch_rec_cplx(int lmax, int64_t n, int input, const TIO* in0, const TIO* in1, TIO* out,
                                  int64_t ld, hipStream_t s)
{
    constexpr int kVec = sizeof(TIO) == 4 ? 2 : 1;
    constexpr int64_t kValue = 2 * sizeof(TIO);
    const In mode = In(input);
    const int64_t stride = mode == In::kAngles ? 1 : 3;
    const RecShape f = rec_cplx_shape<TIO, SPINOR>(n, n * nfun(lmax) * (SPINOR ? 4 : 1) * kValue,
                                                   on_lines(out, ld * kValue));
    for (int64_t c0 = 0; c0 < n; c0 += kRecChunk) {
        const int64_t nc = n - c0 < kRecChunk ? n - c0 : kRecChunk;
        const TIO *a = in0 + stride * c0, *b = mode == In::kAngles ? in1 + c0 : in1;
        TIO* o = out + 2 * c0;
        hipError_t e = hipErrorInvalidValue;
        if (kVec > 1 && (!f.wide || nc < kVec))
            e = launch_rec_cplx_one<TIO, 1, SPINOR, 4>(lmax, nc, mode, a, b, o, ld, s, f.lds);
        else if (f.unroll == 4)
            e = launch_rec_cplx_one<TIO, kVec, SPINOR, 4>(lmax, nc, mode, a, b, o, ld, s, f.lds);
        else if constexpr (sizeof(TIO) == 8)  // the others are FP64's
            e = f.unroll == 8 || SPINOR ? launch_rec_cplx_one<TIO, 1, SPINOR, 8>(lmax, nc, mode, a, b, o, ld, s, f.lds)
                                        : launch_rec_cplx_one<TIO, 1, SPINOR, 1>(lmax, nc, mode, a, b, o, ld, s, f.lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename TIO>
hipError_t launch_rec_complex(int lmax, int64_t n, int input, const TIO* in0, const TIO* in1, TIO* out, int64_t ld,
                              hipStream_t s)
{
    return launch_rec_cplx<TIO, false>(lmax, n, input, in0, in1, out, ld, s);
}

template <typename TIO>
hipError_t launch_rec_spinor(int lmax, int64_t n, int input, const TIO* in0, const TIO* in1, TIO* out, int64_t ld,
                             hipStream_t s)
{
    return launch_rec_cplx<TIO, true>(lmax, n, input, in0, in1, out, ld, s);
}

template hipError_t launch_rec_complex<double>(int, int64_t, int, const double*, const double*, double*, int64_t,
                                               hipStream_t);
template hipError_t launch_rec_complex<float>(int, int64_t, int, const float*, const float*, float*, int64_t,
                                              hipStream_t);
template hipError_t launch_rec_spinor<double>(int, int64_t, int, const double*, const double*, double*, int64_t,
                                              hipStream_t);
template hipError_t launch_rec_spinor<float>(int, int64_t, int, const float*, const float*, float*, int64_t,
                                             hipStream_t);

}  // namespace shk
