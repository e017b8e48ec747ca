// sh_eval.hip -- launchers of the forward kernels (all real Y_lm, l <= lmax).
//
// The kernel (sh_fwd.h) normalises each point in FP64, evaluates the factorised
// formulas and writes every (l, m) value to its row of the [F][ld] output.  The
// path moves 3s + F s bytes per point (s = element size) against a few hundred
// flops, so it is bound by HBM stores.  Launch choices, all measured on MI355X:
//  - Each lane evaluates 16 bytes' worth of adjacent points (two in FP64, four
//    in FP32) and stores 16 bytes per row, at any element alignment: one contiguous
//    1 KiB run per wave and row.  Outputs that stay in the caches on the way out, and
//    launches of few workgroups, take one point per lane: what they last is their
//    workgroups' chain of work, which the wider lanes lengthen.
//  - Workgroups are remapped so each XCD walks one contiguous range of points.
//  - The kernels of large outputs reserve LDS they do not use, which caps the
//    resident workgroups per CU.  Fewer points in flight keep the concurrent writes of
//    each row in a smaller window, which the HBM write path rewards, and most where
//    the rows do not start on cache lines: there neighbouring waves write parts of the
//    same lines, which merge in the L2 only while both are at work (store_shape).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sh_fwd.h"
#include "sh_internal.h"

namespace shk {

// Points per launch: keeps every per-row byte offset of a launch below 2^31 so
// the store address is a scalar row base plus a 32-bit per-lane offset.
constexpr int64_t kChunk = int64_t(1) << 28;

// Input pointers of a launch that starts at point c0.
template <In MODE, typename TIO>
struct Inputs {
    const TIO* a;
    const TIO* b;
    Inputs at(int64_t c0) const
    {
        if constexpr (MODE == In::kAngles) return {a + c0, b + c0};
        else return {a + 3 * c0, b};
    }
    // whether the angles of n points share memory with out[0 .. len)
    bool shares(const TIO* out, int64_t n, int64_t len) const
    {
        auto meets = [&](const TIO* p) {
            return uintptr_t(p) < uintptr_t(out + len) && uintptr_t(out) < uintptr_t(p + n);
        };
        return MODE == In::kAngles && (meets(a) || meets(b));
    }
};

template <int LMAX, typename TIO, int PPL, In MODE>
static hipError_t launch_one(Inputs<MODE, TIO> in, TIO* out, int64_t n, int64_t ld, hipStream_t s, size_t lds)
{
    const int64_t nvec = (n + PPL - 1) / PPL;
    const unsigned grid = unsigned((nvec + kFwdBlock - 1) / kFwdBlock);
    hipLaunchKernelGGL((fwd_kernel<LMAX, TIO, PPL, MODE>), dim3(grid), dim3(kFwdBlock), lds, s,
                       in.a, out, uint32_t(n), ld, in.b);
    return hipGetLastError();
}

template <int LMAX, typename TIO, In MODE>
static hipError_t launch_fwd_l(int64_t n, Inputs<MODE, TIO> in, TIO* out, int64_t ld, hipStream_t s)
{
    // store_shape never asks lmax 1 for more than one point per lane
    constexpr bool kBusy = MODE == In::kAngles && LMAX <= 6;
    constexpr int kVec = LMAX == 1 && !kBusy ? 1 : 16 / sizeof(TIO);
    const int64_t bytes = n * nfun(LMAX) * int64_t(sizeof(TIO));
    const bool lines = on_lines(out, ld * sizeof(TIO));
    StoreShape f = store_shape<nfun(LMAX), TIO>(n, sizeof(TIO), MODE == In::kAngles ? 0 : 3 * sizeof(TIO), lines);
    // angles take two FP64 sines and cosines per point, which at few rows need every wave
    // (us, wide uncapped / capped / one point: FP64 lmax 2, 8000000 points 137 / 180 / 135; lmax 3,
    // 1500000 43.4 / 48.0 / 45.6; FP32 lmax 1, 9000001 64 / 86 / 94; lmax 6, 1000001 43.4 /
    // 45.9 / 52.4), and at more rows until the output is far from the caches (FP32 lmax 7, 585857
    // points 31.1 / 35.4 / 30.5, 859265 48.9 / 51.1 / 56.5, 1562497 89.9 / 87.7 / 117; FP64 lmax 9,
    // 187392 28.9 / 30.0 / 28.2)
    if (kBusy && bytes >= kWideBytes) f = {LMAX != 2 || sizeof(TIO) == 4, 0};
    if (MODE == In::kAngles && LMAX > 6 && bytes < 2 * kWideBytes && (!lines || bytes < kOffBytes))
        f = {bytes >= kOffBytes, 0};
    // angles may be rows of out, as every point's are read before its values are written:
    // then no lane reads a neighbour's, and a remainder takes one point per lane
    const bool in_place = in.shares(out, n, (nfun(LMAX) - 1) * ld + n);
    for (int64_t c0 = 0; c0 < n; c0 += kChunk) {
        const int64_t nc = n - c0 < kChunk ? n - c0 : kChunk;
        const int64_t nw = !f.wide || nc < kVec ? 0 : in_place ? nc / kVec * kVec : nc;
        hipError_t e = nw ? launch_one<LMAX, TIO, kVec, MODE>(in.at(c0), out + c0, nw, ld, s, f.lds) : hipSuccess;
        if (e == hipSuccess && nw < nc)
            e = launch_one<LMAX, TIO, 1, MODE>(in.at(c0 + nw), out + c0 + nw, nc - nw, ld, s, f.lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename TIO, In MODE>
static hipError_t dispatch(int lmax, int64_t n, Inputs<MODE, TIO> in, TIO* out, int64_t ld, hipStream_t s)
{
    switch (lmax) {
    case 0: return launch_fwd_l<0, TIO, MODE>(n, in, out, ld, s);
    case 1: return launch_fwd_l<1, TIO, MODE>(n, in, out, ld, s);
    case 2: return launch_fwd_l<2, TIO, MODE>(n, in, out, ld, s);
    case 3: return launch_fwd_l<3, TIO, MODE>(n, in, out, ld, s);
    case 4: return launch_fwd_l<4, TIO, MODE>(n, in, out, ld, s);
    case 5: return launch_fwd_l<5, TIO, MODE>(n, in, out, ld, s);
    case 6: return launch_fwd_l<6, TIO, MODE>(n, in, out, ld, s);
    case 7: return launch_fwd_l<7, TIO, MODE>(n, in, out, ld, s);
    case 8: return launch_fwd_l<8, TIO, MODE>(n, in, out, ld, s);
    case 9: return launch_fwd_l<9, TIO, MODE>(n, in, out, ld, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename TIO>
hipError_t launch_fwd(int lmax, int64_t n, const TIO* xyz, TIO* out, int64_t ld, hipStream_t s)
{
    return dispatch<TIO, In::kXyz>(lmax, n, {xyz, nullptr}, out, ld, s);
}

template <typename TIO>
hipError_t launch_fwd_unit(int lmax, int64_t n, const TIO* xyz, TIO* out, int64_t ld, hipStream_t s)
{
    return dispatch<TIO, In::kUnit>(lmax, n, {xyz, nullptr}, out, ld, s);
}

template <typename TIO>
hipError_t launch_fwd_angles(int lmax, int64_t n, const TIO* theta, const TIO* phi, TIO* out, int64_t ld,
                             hipStream_t s)
{
    return dispatch<TIO, In::kAngles>(lmax, n, {theta, phi}, out, ld, s);
}

// Complex and spinor kernels: 16 bytes per lane and row (one FP64 complex, or two FP32
// complex values of adjacent points) or one point per lane, and the LDS reservation,
// as store_shape says.
// Inputs of a complex or spinor launch: in0 (+ in1 for angles) and their kind.
template <typename TIO>
struct AnyInputs {
    const TIO* a;
    const TIO* b;
    In mode;
    AnyInputs at(int64_t c0) const
    {
        if (mode == In::kAngles) return {a + c0, b + c0, mode};
        return {a + 3 * c0, b, mode};
    }
};

template <bool SPINOR, int LMAX, typename TIO, int PPL>
static hipError_t launch_complex_one(int64_t n, AnyInputs<TIO> in, TIO* out, int64_t ld, hipStream_t s, size_t lds)
{
    const auto kernel = SPINOR ? fwd_spinor_kernel<LMAX, TIO, PPL> : fwd_complex_kernel<LMAX, TIO, PPL>;
    const unsigned grid = unsigned(((n + PPL - 1) / PPL + kFwdBlock - 1) / kFwdBlock);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kFwdBlock), lds, s, in.a, out, uint32_t(n), ld, in.b, in.mode);
    return hipGetLastError();
}

// out holds rows of ld complex values; a launch starting at point c0 writes from
// out + 2 c0 (in TIO units).
template <bool SPINOR, int LMAX, typename TIO>
static hipError_t launch_complex_l(int64_t n, AnyInputs<TIO> in, TIO* out, int64_t ld, hipStream_t s)
{
    constexpr int kRows = (SPINOR ? 4 : 1) * nfun(LMAX);
    constexpr int kVec = sizeof(TIO) == 4 && kRows != 4 ? 2 : 1;  // store_shape never asks 4 rows for more
    constexpr int kValue = 2 * sizeof(TIO);
    StoreShape f = store_shape<kRows, TIO>(n, kValue, 0, on_lines(out, ld * kValue));
    // angles need every wave, as for the real harmonics: below 2^29 bytes at any number of rows
    // (us, uncapped / one workgroup per CU: FP64 lmax 4, 374913 points 28.5 / 32.7, lmax 7, 214785
    // 47.8 / 50.2; FP32 lmax 4, 1000001 42.5 / 48.5), above at few; but FP64 at 16 and 25 rows from
    // 5 x 2^26 bytes on two workgroups per CU (spinor lmax 1, 1562497 uncapped 93.6, so 90.2, 2343681
    // 147 / 134; lmax 4, 1499905 135 / 130)
    if (in.mode == In::kAngles && (kRows <= 25 || n * kRows * kValue < kCapBytes))
        f.lds = kRows >= 16 && kRows <= 25 && sizeof(TIO) == 8 && n * kRows * kValue >= 2 * kOffBytes ? kCapLds2 : 0;
    for (int64_t c0 = 0; c0 < n; c0 += kChunk) {
        const int64_t nc = n - c0 < kChunk ? n - c0 : kChunk;
        const hipError_t e = f.wide && nc >= kVec
                                 ? launch_complex_one<SPINOR, LMAX, TIO, kVec>(nc, in.at(c0), out + 2 * c0, ld, s, f.lds)
                                 : launch_complex_one<SPINOR, LMAX, TIO, 1>(nc, in.at(c0), out + 2 * c0, ld, s, f.lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool SPINOR, typename TIO>
static hipError_t dispatch_complex(int lmax, int64_t n, AnyInputs<TIO> xyz, TIO* out, int64_t ld, hipStream_t s)
{
    switch (lmax) {
    case 0: return launch_complex_l<SPINOR, 0, TIO>(n, xyz, out, ld, s);
    case 1: return launch_complex_l<SPINOR, 1, TIO>(n, xyz, out, ld, s);
    case 2: return launch_complex_l<SPINOR, 2, TIO>(n, xyz, out, ld, s);
    case 3: return launch_complex_l<SPINOR, 3, TIO>(n, xyz, out, ld, s);
    case 4: return launch_complex_l<SPINOR, 4, TIO>(n, xyz, out, ld, s);
    case 5: return launch_complex_l<SPINOR, 5, TIO>(n, xyz, out, ld, s);
    case 6: return launch_complex_l<SPINOR, 6, TIO>(n, xyz, out, ld, s);
    case 7: return launch_complex_l<SPINOR, 7, TIO>(n, xyz, out, ld, s);
    case 8: return launch_complex_l<SPINOR, 8, TIO>(n, xyz, out, ld, s);
    case 9: return launch_complex_l<SPINOR, 9, TIO>(n, xyz, out, ld, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename TIO>
hipError_t launch_fwd_complex(int lmax, int64_t n, int input, const TIO* in0, const TIO* in1, TIO* out, int64_t ld,
                              hipStream_t s)
{
    return dispatch_complex<false, TIO>(lmax, n, {in0, in1, In(input)}, out, ld, s);
}

template <typename TIO>
hipError_t launch_fwd_spinor(int lmax, int64_t n, int input, const TIO* in0, const TIO* in1, TIO* out, int64_t ld,
                             hipStream_t s)
{
    return dispatch_complex<true, TIO>(lmax, n, {in0, in1, In(input)}, out, ld, s);
}

template hipError_t launch_fwd_spinor<double>(int, int64_t, int, const double*, const double*, double*, int64_t,
                                             hipStream_t);
template hipError_t launch_fwd_spinor<float>(int, int64_t, int, const float*, const float*, float*, int64_t,
                                             hipStream_t);
template hipError_t launch_fwd<double>(int, int64_t, const double*, double*, int64_t, hipStream_t);
template hipError_t launch_fwd<float>(int, int64_t, const float*, float*, int64_t, hipStream_t);
template hipError_t launch_fwd_unit<double>(int, int64_t, const double*, double*, int64_t, hipStream_t);
template hipError_t launch_fwd_unit<float>(int, int64_t, const float*, float*, int64_t, hipStream_t);
template hipError_t launch_fwd_angles<double>(int, int64_t, const double*, const double*, double*, int64_t,
                                              hipStream_t);
template hipError_t launch_fwd_angles<float>(int, int64_t, const float*, const float*, float*, int64_t,
                                             hipStream_t);
template hipError_t launch_fwd_complex<double>(int, int64_t, int, const double*, const double*, double*, int64_t,
                                             hipStream_t);
template hipError_t launch_fwd_complex<float>(int, int64_t, int, const float*, const float*, float*, int64_t,
                                             hipStream_t);

}  // namespace shk
