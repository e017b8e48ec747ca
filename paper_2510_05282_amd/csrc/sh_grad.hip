// sh_grad.hip -- backward kernel: vector-Jacobian product of the forward pass.
//
// For an upstream gradient G[F][n] the kernel returns, per point,
//     g = sum_{l,m} G_lm grad_r R_l^m(r) = (1/r) (v - u (u . v)),
//     v = sum_{l,m} G_lm grad_u P_lm(u),   u = r / |r|,
// where P_lm is the factorised polynomial the forward kernel evaluates.  Any
// smooth extension of R_l^m off the unit sphere gives the same tangential part,
// so the projection makes the result exact whatever the extension.  The polynomial
// gradients come from running the same factorised forms on dual numbers
// (grad_unit in sh_dual.h).
// One thread per point; G is read row by row (coalesced across the wave), the
// three gradient components are written per point.  Memory traffic per point:
// 3s B in (xyz) + F s B (G) + 3s B out (s = element size); this path is bound by
// reading G.  The same file holds the fused value + Jacobian kernel.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sh_core.h"
#include "sh_dual.h"
#include "sh_fwd.h"
#include "sh_internal.h"

namespace shk {

constexpr int kGradBlock = 256;
constexpr int64_t kGradChunk = int64_t(1) << 28;

// TIO is the element type of xyz, G and the result; the normalisation and 1/r
// run in FP64, the polynomials and the contraction in TIO.
template <int LMAX, typename TIO, GRead READ>
__global__ __launch_bounds__(kGradBlock) void grad_kernel(const TIO* __restrict__ xyz, const TIO* __restrict__ G,
                                                          TIO* __restrict__ gxyz, uint32_t n, int64_t ldg)
{
    const uint32_t b = READ == GRead::kCached ? xcd_tile(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t i = b * kGradBlock + threadIdx.x;
    if (i >= n) return;
    const TIO* p = xyz + 3 * size_t(i);
    double xb, yb, zb, keep, rinv;
    normalize(double(p[0]), double(p[1]), double(p[2]), xb, yb, zb, keep, rinv);
    const uint32_t boff = i * uint32_t(sizeof(TIO));
    auto g_at = [&](int r) {
        const TIO* g = reinterpret_cast<const TIO*>(reinterpret_cast<const char*>(G + int64_t(r) * ldg) + boff);
        return READ == GRead::kStream ? __builtin_nontemporal_load(g) : *g;
    };
    (void)keep;  // the origin needs no mask here: rinv = 0 there, so the gradient is 0
    TIO vx, vy, vz;
    const TIO x = TIO(xb), y = TIO(yb), z = TIO(zb);
    grad_unit<LMAX, TIO>(x, y, z, g_at, vx, vy, vz);
    const double uv = xb * double(vx) + yb * double(vy) + zb * double(vz);
    TIO* o = gxyz + 3 * size_t(i);
    o[0] = TIO(rinv * (double(vx) - xb * uv));
    o[1] = TIO(rinv * (double(vy) - yb * uv));
    o[2] = TIO(rinv * (double(vz) - zb * uv));
}

template <int LMAX, typename TIO, GRead READ>
static hipError_t launch_grad_one(int64_t n, const TIO* xyz, const TIO* G, int64_t ldg, TIO* gxyz, hipStream_t s)
{
    for (int64_t c0 = 0; c0 < n; c0 += kGradChunk) {
        const int64_t nc = n - c0 < kGradChunk ? n - c0 : kGradChunk;
        const unsigned grid = unsigned((nc + kGradBlock - 1) / kGradBlock);
        hipLaunchKernelGGL((grad_kernel<LMAX, TIO, READ>), dim3(grid), dim3(kGradBlock),
                           READ == GRead::kCached ? 0 : kCapLds4, s, xyz + 3 * c0, G + c0, gxyz + 3 * c0, uint32_t(nc),
                           ldg);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int LMAX, typename TIO>
static hipError_t launch_grad_l(int64_t n, const TIO* xyz, const TIO* G, int64_t ldg, TIO* gxyz, hipStream_t s)
{
    switch (grad_read<LMAX, TIO>(n, on_lines(G, ldg * sizeof(TIO)))) {
    case GRead::kCached: return launch_grad_one<LMAX, TIO, GRead::kCached>(n, xyz, G, ldg, gxyz, s);
    case GRead::kShared:
        if constexpr (LMAX >= 3) return launch_grad_one<LMAX, TIO, GRead::kShared>(n, xyz, G, ldg, gxyz, s);
        [[fallthrough]];
    default: return launch_grad_one<LMAX, TIO, GRead::kStream>(n, xyz, G, ldg, gxyz, s);
    }
}

template <typename TIO>
hipError_t launch_grad(int lmax, int64_t n, const TIO* xyz, const TIO* G, int64_t ldg, TIO* gxyz, hipStream_t s)
{
    switch (lmax) {
    case 0: return launch_grad_l<0, TIO>(n, xyz, G, ldg, gxyz, s);
    case 1: return launch_grad_l<1, TIO>(n, xyz, G, ldg, gxyz, s);
    case 2: return launch_grad_l<2, TIO>(n, xyz, G, ldg, gxyz, s);
    case 3: return launch_grad_l<3, TIO>(n, xyz, G, ldg, gxyz, s);
    case 4: return launch_grad_l<4, TIO>(n, xyz, G, ldg, gxyz, s);
    case 5: return launch_grad_l<5, TIO>(n, xyz, G, ldg, gxyz, s);
    case 6: return launch_grad_l<6, TIO>(n, xyz, G, ldg, gxyz, s);
    case 7: return launch_grad_l<7, TIO>(n, xyz, G, ldg, gxyz, s);
    case 8: return launch_grad_l<8, TIO>(n, xyz, G, ldg, gxyz, s);
    case 9: return launch_grad_l<9, TIO>(n, xyz, G, ldg, gxyz, s);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_grad<double>(int, int64_t, const double*, const double*, int64_t, double*,
                                        hipStream_t);
template hipError_t launch_grad<float>(int, int64_t, const float*, const float*, int64_t, float*, hipStream_t);

// ---------------------------------------------------------------- fused value + Jacobian

// Values out[F][ld] and the Jacobian jac[3][F][ld] (d R_f / d x_k at
// jac[(k F + f) ld + i]) in one pass: the dual-number core gives P and grad_u P,
// which is projected with (1/r)(I - u u^T).  The launch follows the forward
// kernel's (4F + 3 doubles per point, all but 3 of them row stores): PPL = 2
// adjacent points per lane with 16-byte row stores at any alignment or one point per
// lane, and the LDS reservation, as store_shape says for 4F rows; workgroups in
// XCD-contiguous order.

template <int LMAX, int PPL>
__global__ __launch_bounds__(kGradBlock) void jac_kernel(const double* __restrict__ xyz, double* __restrict__ out,
                                                         double* __restrict__ jac, uint32_t n, int64_t ld)
{
    constexpr int F = nfun(LMAX);
    using V = std::conditional_t<PPL == 1, double, double2_t>;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x) * kGradBlock + threadIdx.x;
    if (t * PPL >= n) return;
    const uint32_t i0 = first_point<PPL>(t, n);
    V x, y, z, k, ri;
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        const double* p = xyz + 3 * size_t(i0 + q);
        double xb, yb, zb, kb, rb;
        normalize(p[0], p[1], p[2], xb, yb, zb, kb, rb);
        if constexpr (PPL == 1) {
            x = xb, y = yb, z = zb, k = kb, ri = rb;
        } else {
            x[q] = xb, y[q] = yb, z[q] = zb, k[q] = kb, ri[q] = rb;
        }
    }
    const uint32_t boff = i0 * uint32_t(sizeof(double));
    auto at = [&](double* base, int64_t r) {
        return reinterpret_cast<typename uvec_of<double, PPL>::type*>(reinterpret_cast<char*>(base + r * ld) + boff);
    };
    eval_unit_jac<LMAX, V>(x, y, z, k, [&](int f, V v, V gx, V gy, V gz) {
        const V ug = x * gx + y * gy + z * gz;
        *at(out, f) = v;
        *at(jac, f) = ri * (gx - x * ug);
        *at(jac, F + f) = ri * (gy - y * ug);
        *at(jac, 2 * F + f) = ri * (gz - z * ug);
    });
}

template <int LMAX, int PPL>
static hipError_t launch_jac_one(int64_t n, const double* xyz, double* out, double* jac, int64_t ld, hipStream_t s,
                                 size_t lds)
{
    const unsigned grid = unsigned(((n + PPL - 1) / PPL + kGradBlock - 1) / kGradBlock);
    hipLaunchKernelGGL((jac_kernel<LMAX, PPL>), dim3(grid), dim3(kGradBlock), lds, s, xyz, out, jac, uint32_t(n), ld);
    return hipGetLastError();
}

template <int LMAX>
static hipError_t launch_jac_l(int64_t n, const double* xyz, double* out, double* jac, int64_t ld, hipStream_t s)
{
    constexpr int kRows = 4 * nfun(LMAX);
    constexpr int kVec = kRows == 4 ? 1 : 2;  // store_shape never asks 4 rows for more
    const StoreShape f = store_shape<kRows, double>(n, sizeof(double), 3 * sizeof(double),
                                                    on_lines(out, ld * 8) && on_lines(jac, ld * 8));
    for (int64_t c0 = 0; c0 < n; c0 += kGradChunk) {
        const int64_t nc = n - c0 < kGradChunk ? n - c0 : kGradChunk;
        const hipError_t e = f.wide && nc >= kVec
                                 ? launch_jac_one<LMAX, kVec>(nc, xyz + 3 * c0, out + c0, jac + c0, ld, s, f.lds)
                                 : launch_jac_one<LMAX, 1>(nc, xyz + 3 * c0, out + c0, jac + c0, ld, s, f.lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_jac(int lmax, int64_t n, const double* xyz, double* out, double* jac, int64_t ld, hipStream_t s)
{
    switch (lmax) {
    case 0: return launch_jac_l<0>(n, xyz, out, jac, ld, s);
    case 1: return launch_jac_l<1>(n, xyz, out, jac, ld, s);
    case 2: return launch_jac_l<2>(n, xyz, out, jac, ld, s);
    case 3: return launch_jac_l<3>(n, xyz, out, jac, ld, s);
    case 4: return launch_jac_l<4>(n, xyz, out, jac, ld, s);
    case 5: return launch_jac_l<5>(n, xyz, out, jac, ld, s);
    case 6: return launch_jac_l<6>(n, xyz, out, jac, ld, s);
    case 7: return launch_jac_l<7>(n, xyz, out, jac, ld, s);
    case 8: return launch_jac_l<8>(n, xyz, out, jac, ld, s);
    case 9: return launch_jac_l<9>(n, xyz, out, jac, ld, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace shk
