// sh_proj.hip -- radial spline tables and the fused projector build.
//
// A projector value for atom a at grid point p is R_l(|d|) * R_l^m(d / |d|) with
// d = p - c_a (the role the harmonics play in the paper's introduction).  R_l is
// a natural cubic spline through values tabulated on a uniform radial grid; it is
// 0 beyond the table's last knot.  One pass per point computes d, r, every R_l(r)
// for l <= lmax, the harmonics, and stores their products; nothing is
// materialised in between.
//
// Device table layout of a radial handle: [n_tables][n_r][channels] of double2
// (y_i, M_i), M the spline's second derivatives: the knots i and i+1 of all
// channels of a table are 2 * channels adjacent pairs, so one point's spline
// lookups touch one or two cache lines.
//
// Launch (measured on MI355X, 64 atoms / 0.9M points / lmax 3: 43 us -> 30 us):
// workgroups remapped so each XCD works through one contiguous range of atoms
// (their tables then stay in that XCD's L2); the atom of a wave found by one
// wave-wide search; plain stores; one point per lane, or, for builds of at least
// kProjVecPoints points, kProjPpl adjacent points per lane evaluated together, with
// at most 2 resident workgroups per CU (kProjCapLds); those builds run
// proj_vec_kernel where kProjVecKernel or kProjVecWindow is set.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sh_core.h"
#include "sh_internal.h"
#include "sh_proj.h"

namespace shk {

// ---------------------------------------------------------------- spline set-up

// The eliminated super-diagonal c_k = 1 / (4 - c_{k-1}), c_0 = 0, of spline_solve: the
// same for every channel, and from k = kSplineCs - 1 on a fixed point in double
// (c -> 1 / (4 - c) contracts by 0.07 near 2 - sqrt(3)).
constexpr int kSplineCs = 24;
struct SplineC {
    double c[kSplineCs];
    constexpr SplineC() : c{}
    {
        for (int k = 1; k < kSplineCs; ++k) c[k] = 1.0 / (4.0 - c[k - 1]);
    }
};
constexpr SplineC kSplineC;
static_assert(1.0 / (4.0 - kSplineC.c[kSplineCs - 1]) == kSplineC.c[kSplineCs - 1], "c_k has not settled");
__device__ constexpr SplineC kSplineCDev;

__device__ __forceinline__ double spline_c(int k)
{
    constexpr double last = kSplineC.c[kSplineCs - 1];
    return k < kSplineCs ? kSplineCDev.c[k] : last;
}

constexpr int kSplineBlock = 256;                        // threads per channel
constexpr int kSplinePer = 8;                            // adjacent knots per thread
constexpr int kSplineTile = kSplineBlock * kSplinePer;   // knots per pass of a workgroup
// LDS slot of knot j of a tile: one slot of padding per kSplinePer, so that lanes
// reading kSplinePer knots apart spread over the banks.
__device__ __forceinline__ constexpr int spline_slot(int j) { return j + j / kSplinePer; }

// Composition of affine maps v -> a v + b over the workgroup: on entry each thread's
// own map, on return the map of all threads before it (REV: after it), in their order
// of application.  Every thread must call it; tot holds one map per wave.
struct Affine {
    double a, b;
};
template <bool REV>
__device__ __forceinline__ Affine block_before(Affine own, Affine* tot)
{
    const int wl = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int s = 1; s < 64; s *= 2) {
        const double a = REV ? __shfl_down(own.a, s) : __shfl_up(own.a, s);
        const double b = REV ? __shfl_down(own.b, s) : __shfl_up(own.b, s);
        if (REV ? wl + s < 64 : wl >= s) {
            own.b = own.a * b + own.b;
            own.a = own.a * a;
        }
    }
    if (wl == (REV ? 0 : 63)) tot[wave] = own;
    Affine m{REV ? __shfl_down(own.a, 1) : __shfl_up(own.a, 1), REV ? __shfl_down(own.b, 1) : __shfl_up(own.b, 1)};
    if (wl == (REV ? 63 : 0)) m = Affine{1.0, 0.0};
    __syncthreads();
    constexpr int kWaves = kSplineBlock / 64;
#pragma unroll
    for (int q = 1; q < kWaves; ++q) {  // the waves before this one, nearest first
        const int w = REV ? wave + q : wave - q;
        if (w >= 0 && w < kWaves) {
            m.b = m.a * tot[w].b + m.b;
            m.a = m.a * tot[w].a;
        }
    }
    __syncthreads();
    return m;
}

// One workgroup per channel c = (table t = c / ch, channel l = c % ch): values y[c][n_r]
// in, pairs to table[t][k][l] and, rounded to float, to table_f32 (each if not null).
// The tridiagonal solve of spline_solve is a chain of n_r dependent steps each way,
//     d_k = (rhs_k - d_{k-1}) / (4 - c_{k-1}),   M_k = d_k - c_k M_{k+1},
// but every step is an affine map of the one before with |slope| < 0.27 and c_k is known
// beforehand, so each thread composes the maps of its kSplinePer knots, a scan over the
// workgroup gives the value its first knot starts from, and it then takes its own steps
// from there.  Channels longer than kSplineTile take several passes each way, carrying
// one value from pass to pass and d in cp[c][n_r].  Where a right-hand side is not finite
// (a value of y that is not) or near overflow, one thread runs spline_solve, so that
// infinities and NaN spread as there; `work` is where its pairs go when table is null.
// Bound by latency: with one thread per channel 168 channels of 2000 knots took 1.48 ms
// (0.74 us per knot, 168 lanes of the GPU busy); this takes 8 us.
__global__ __launch_bounds__(kSplineBlock) void spline_setup_kernel(const double* __restrict__ y,
                                                                    double2* __restrict__ table,
                                                                    float2* __restrict__ table_f32,
                                                                    double2* __restrict__ work,
                                                                    double* __restrict__ cp, int64_t c0, int ch,
                                                                    int n_r, double six_over_h2)
{
    __shared__ double ys[spline_slot(kSplineTile + 2) + 1], ms[spline_slot(kSplineTile) + 1];
    __shared__ Affine tot[kSplineBlock / 64];
    __shared__ double edge;
    const int tid = threadIdx.x;
    // the channels of a table on one XCD, whose L2 then merges the lines they share
    const int64_t c = c0 + xcd_tile(blockIdx.x, gridDim.x);
    const double* yc = y + c * n_r;
    double* dc = cp + c * n_r;
    const int64_t at0 = c / ch * n_r * ch + c % ch;
    const int nt = (n_r + kSplineTile - 1) / kSplineTile;
    auto interior = [&](int k) { return k >= 1 && k <= n_r - 2; };
    double d[kSplinePer];
    double carry = 0.0;
    for (int t = 0; t < nt; ++t) {
        const int base = t * kSplineTile;
        for (int j = tid; j < kSplineTile + 2; j += kSplineBlock) {  // slot j holds y[base - 1 + j]
            const int k = base - 1 + j;
            ys[spline_slot(j)] = k >= 0 && k < n_r ? yc[k] : 0.0;
        }
        __syncthreads();
        const int k0 = base + tid * kSplinePer;
        bool bad = false;
        Affine own{1.0, 0.0};
#pragma unroll
        for (int i = 0; i < kSplinePer; ++i) {
            const int j = tid * kSplinePer + i;
            const double rhs = six_over_h2 * (ys[spline_slot(j + 2)] - 2.0 * ys[spline_slot(j + 1)] + ys[spline_slot(j)]);
            d[i] = rhs;
            if (interior(k0 + i)) {
                const double ck = spline_c(k0 + i);
                own.b = (rhs - own.b) * ck;
                own.a = -own.a * ck;
                bad = bad || !(fabs(rhs) < 0x1p+1000);
            } else {
                own = Affine{0.0, 0.0};
            }
        }
        if (__syncthreads_or(bad)) {
            double2* tc = (table ? table : work) + at0;
            if (tid == 0) spline_solve(yc, tc, ch, dc, n_r, six_over_h2);
            __syncthreads();
            if (table_f32)
                for (int k = tid; k < n_r; k += kSplineBlock) {
                    const double2 v = tc[int64_t(k) * ch];
                    table_f32[at0 + int64_t(k) * ch] = make_float2(float(v.x), float(v.y));
                }
            return;
        }
        const Affine m = block_before<false>(own, tot);
        double v = m.a * carry + m.b;
#pragma unroll
        for (int i = 0; i < kSplinePer; ++i) {
            if (interior(k0 + i)) {
                // (rhs - v) / (4 - c_{k-1}) through the reciprocal c_k and one correction
                const double ck = spline_c(k0 + i), x = d[i] - v, den = 4.0 - spline_c(k0 + i - 1), q = x * ck;
                v = __builtin_fma(__builtin_fma(-q, den, x), ck, q);
            } else {
                v = 0.0;
            }
            d[i] = v;
            if (nt > 1 && k0 + i < n_r) dc[k0 + i] = v;
        }
        if (tid == kSplineBlock - 1) edge = v;
        __syncthreads();
        carry = edge;
    }
    carry = 0.0;
    for (int t = nt - 1; t >= 0; --t) {
        const int base = t * kSplineTile, k0 = base + tid * kSplinePer;
        Affine own{1.0, 0.0};
#pragma unroll
        for (int i = kSplinePer - 1; i >= 0; --i) {
            if (nt > 1) d[i] = k0 + i < n_r ? dc[k0 + i] : 0.0;
            if (interior(k0 + i)) {
                const double ck = spline_c(k0 + i);
                own.b = d[i] - ck * own.b;
                own.a = -ck * own.a;
            } else {
                own = Affine{0.0, 0.0};
            }
        }
        const Affine m = block_before<true>(own, tot);
        double v = m.a * carry + m.b;
#pragma unroll
        for (int i = kSplinePer - 1; i >= 0; --i) {
            v = interior(k0 + i) ? d[i] - spline_c(k0 + i) * v : 0.0;
            ms[spline_slot(tid * kSplinePer + i)] = v;
        }
        if (tid == 0) edge = v;
        __syncthreads();
        carry = edge;
        for (int j = tid; j < kSplineTile && base + j < n_r; j += kSplineBlock) {
            const double2 p = make_double2(nt > 1 ? yc[base + j] : ys[spline_slot(j + 1)], ms[spline_slot(j)]);
            const int64_t at = at0 + int64_t(base + j) * ch;
            if (table) table[at] = p;
            if (table_f32) table_f32[at] = make_float2(float(p.x), float(p.y));
        }
        __syncthreads();
    }
}

// The same with one thread per channel, for many short channels (launch_spline_setup).
__global__ __launch_bounds__(64) void spline_serial_kernel(const double* __restrict__ y, double2* __restrict__ table,
                                                           float2* __restrict__ table_f32,
                                                           double2* __restrict__ work, double* __restrict__ cp,
                                                           int64_t c0, int64_t n_ch, int ch, int n_r,
                                                           double six_over_h2)
{
    const int64_t c = c0 + int64_t(blockIdx.x) * 64 + threadIdx.x;
    if (c >= n_ch) return;
    const int64_t at0 = c / ch * n_r * ch + c % ch;
    double2* tc = (table ? table : work) + at0;
    spline_solve(y + c * n_r, tc, ch, cp + c * n_r, n_r, six_over_h2);
    if (table_f32)
        for (int64_t k = 0; k < n_r; ++k)
            table_f32[at0 + k * ch] = make_float2(float(tc[k * ch].x), float(tc[k * ch].y));
}

// Flat projector kernel over the concatenated atom point sets, PPL adjacent
// points per lane.  A lane whose PPL points lie in one atom evaluates them
// together (proj_points); a lane that straddles an atom boundary or the end of
// the points takes them one by one.  A point whose offsets are inconsistent
// (outside [offsets[a], offsets[a+1]) or beyond n_points) is skipped, so every
// store stays inside out[F * n_points].
//
// Finding a point's atom: with at most 64 atoms (SMALL), lane k loads atom k's
// offsets, centre and table index while the point loads are in flight; a ballot
// over the loaded offsets gives the wave's first atom aw, whose data (and that of
// aw + 1, where a wave crosses into the next atom) every lane reads from lanes aw
// and aw + 1.  That leaves one dependent step (the spline lookup) between the
// point loads and the arithmetic.  Otherwise, and for lanes past atom aw + 1, the
// wave's atom comes from a wave-wide search and a lane's from a binary search, and
// the atom's data is loaded after it.  Measured on the 64-atom lmax 3 build (one
// point per lane): 29.6-29.8 us -> 27.6-28.0 us.  In this kernel the launches with
// several points per lane keep the search: there the preload alone cost as much as
// the shorter chain saved (-6% to +5% across lmax and dtype on 64 x 150k-point
// builds); proj_vec_kernel combines it with loading every knot of a lane at once.
struct AtomRef {
    int64_t o0, o1;  // its point range
    double c[3];
    int t;           // its table
};

template <int LMAX, typename TIO, int PPL, bool SMALL>
__global__ __launch_bounds__(256) void proj_kernel(const TIO* __restrict__ centers,
                                                   const int64_t* __restrict__ offsets, int n_atoms,
                                                   const TIO* __restrict__ points, int64_t n_points,
                                                   const knot_t<TIO>* __restrict__ table, int tab_ch,
                                                   int n_tables, const int32_t* __restrict__ table_of_atom,
                                                   SplineGrid g, TIO* __restrict__ out, int64_t j0)
{
    constexpr int F = nfun(LMAX);
    // first point of this wave; the launch covers points j0 .. j0 + 256 PPL gridDim.x - 1
    const int64_t w0 = j0 + (int64_t(xcd_tile(blockIdx.x, gridDim.x)) * 256 + (threadIdx.x & ~63u)) * PPL;
    if (w0 >= n_points) return;
    const int lane = threadIdx.x & 63;
    const int64_t j = w0 + lane * PPL;
    const bool live = j < n_points;
    double px[PPL], py[PPL], pz[PPL];
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        const TIO* p = points + 3 * (live && j + q < n_points ? j + q : w0);
        px[q] = double(p[0]);
        py[q] = double(p[1]);
        pz[q] = double(p[2]);
    }
    auto clamp_table = [&](int t) { return t < 0 ? 0 : (t >= n_tables ? n_tables - 1 : t); };
    auto load_atom = [&](int a) {
        AtomRef r;
        r.o0 = offsets[a];
        r.o1 = offsets[a + 1];
        r.c[0] = double(centers[3 * a]);
        r.c[1] = double(centers[3 * a + 1]);
        r.c[2] = double(centers[3 * a + 2]);
        r.t = clamp_table(table_of_atom ? table_of_atom[a] : a);
        return r;
    };
    AtomRef A0, A1;  // atoms aw and aw + 1 (o0 = o1 = -1 if there is none)
    A0.o0 = A0.o1 = A1.o0 = A1.o1 = -1;
    int aw;
    if constexpr (SMALL) {
        AtomRef mine{};  // atom `lane`
        if (lane < n_atoms) mine = load_atom(lane);
        const int c = __popcll(__ballot(lane < n_atoms && mine.o0 <= w0));
        aw = c - 1;
        if (aw >= 0) {
            A0 = AtomRef{lane_value(mine.o0, aw), lane_value(mine.o1, aw),
                         {lane_value(mine.c[0], aw), lane_value(mine.c[1], aw), lane_value(mine.c[2], aw)},
                         lane_value(mine.t, aw)};
        }
        if (aw + 1 < n_atoms) {
            const int b = aw + 1;
            A1 = AtomRef{lane_value(mine.o0, b), lane_value(mine.o1, b),
                         {lane_value(mine.c[0], b), lane_value(mine.c[1], b), lane_value(mine.c[2], b)},
                         lane_value(mine.t, b)};
        }
    } else {
        aw = wave_search(offsets, n_atoms, w0);
        if (aw >= 0) A0.o1 = offsets[aw + 1];  // the rest of atom aw is loaded by the lanes that need it
    }
    if (!live) return;
    // atom of point jq and its data; ok = false if jq's range is inconsistent
    auto atom_of = [&](int64_t jq, AtomRef& r) {
        if (SMALL && A0.o0 <= jq && jq < A0.o1) {
            r = A0;
        } else if (SMALL && A1.o0 <= jq && jq < A1.o1) {
            r = A1;
        } else {
            r = load_atom(jq < A0.o1 ? aw : lane_search(offsets, n_atoms, jq));
        }
        return r.o0 >= 0 && r.o0 <= jq && jq < r.o1 && r.o1 <= n_points;
    };
    AtomRef A;
    const bool ok = atom_of(j, A);
    if constexpr (PPL == 1) {
        if (!ok) return;
        proj_point<LMAX, TIO>(px[0], py[0], pz[0], A.c, table + int64_t(A.t) * g.n_r * tab_ch, tab_ch, g,
                              out + F * A.o0 + (j - A.o0), A.o1 - A.o0);
    } else if (ok && j + PPL <= A.o1) {
        proj_points<LMAX, TIO, PPL>(px, py, pz, A.c, table + int64_t(A.t) * g.n_r * tab_ch, tab_ch, g,
                                    out + F * A.o0 + (j - A.o0), A.o1 - A.o0);
    } else {
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
            const int64_t jq = j + q;
            if (jq >= n_points) break;
            AtomRef B;
            if (!atom_of(jq, B)) continue;
            proj_point<LMAX, TIO>(px[q], py[q], pz[q], B.c, table + int64_t(B.t) * g.n_r * tab_ch, tab_ch, g,
                                  out + F * B.o0 + (jq - B.o0), B.o1 - B.o0);
        }
    }
}

// The launches with several points per lane, for the (dtype, lmax) where
// kProjVecKernel (at most 64 atoms) or kProjVecWindow (more) is set: lane k loads
// the offsets, centre and table of atom a0 + k with the points (a0 = 0 for at most
// 64 atoms, as the one-point SMALL path does; otherwise the wave's atom, from one
// wave-wide search), a ballot gives the wave's
// atom and the next, and a lane then issues the knot loads of all its points before
// it evaluates any spline (spline_knots, then spline_from), so the chain per lane is
// the point loads, one wave of knot loads and the stores.  Each lane's points lie
// in one of those two atoms unless the wave crosses more than one atom boundary;
// such lanes, and lanes that straddle a boundary, take their points one by one.
// The same arithmetic as proj_kernel, so the same bits.
template <int LMAX, typename TIO, int PPL>
__global__ __launch_bounds__(256) void proj_vec_kernel(const TIO* __restrict__ centers,
                                                       const int64_t* __restrict__ offsets, int n_atoms,
                                                       const TIO* __restrict__ points, int64_t n_points,
                                                       const knot_t<TIO>* __restrict__ table, int tab_ch,
                                                       int n_tables, const int32_t* __restrict__ table_of_atom,
                                                       SplineGrid g, TIO* __restrict__ out, int64_t j0)
{
    using V = typename vec_of<TIO, PPL>::type;
    constexpr int F = nfun(LMAX);
    const int64_t w0 = j0 + (int64_t(xcd_tile(blockIdx.x, gridDim.x)) * 256 + (threadIdx.x & ~63u)) * PPL;
    if (w0 >= n_points) return;
    const int wl = threadIdx.x & 63;  // lane in the wave
    auto load_atom = [&](int a) {
        AtomRef r;
        r.o0 = offsets[a];
        r.o1 = offsets[a + 1];
        r.c[0] = double(centers[3 * a]);
        r.c[1] = double(centers[3 * a + 1]);
        r.c[2] = double(centers[3 * a + 2]);
        const int t = table_of_atom ? table_of_atom[a] : a;
        r.t = t < 0 ? 0 : (t >= n_tables ? n_tables - 1 : t);
        return r;
    };
    int a0 = 0;  // first atom of the window held in the lanes
    if (n_atoms > 64) {
        a0 = wave_search(offsets, n_atoms, w0);
        a0 = a0 < 0 ? 0 : a0;
    }
    const int nw = n_atoms - a0 < 64 ? n_atoms - a0 : 64;
    AtomRef mine{};
    if (wl < nw) mine = load_atom(a0 + wl);
    const int64_t j = w0 + wl * PPL;
    double px[PPL], py[PPL], pz[PPL];
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        const TIO* p = points + 3 * (j + q < n_points ? j + q : w0);
        px[q] = double(p[0]);
        py[q] = double(p[1]);
        pz[q] = double(p[2]);
    }
    auto atom_at = [&](int a) {
        return AtomRef{lane_value(mine.o0, a), lane_value(mine.o1, a),
                       {lane_value(mine.c[0], a), lane_value(mine.c[1], a), lane_value(mine.c[2], a)},
                       lane_value(mine.t, a)};
    };
    const int aw = __popcll(__ballot(wl < nw && mine.o0 <= w0)) - 1;  // in the window
    AtomRef A0, A1;  // atoms a0 + aw and a0 + aw + 1 (o0 = o1 = -1 if there is none)
    A0.o0 = A0.o1 = A1.o0 = A1.o1 = -1;
    if (aw >= 0) A0 = atom_at(aw);
    if (aw + 1 < nw) A1 = atom_at(aw + 1);
    if (j >= n_points) return;
    const bool in0 = A0.o0 >= 0 && A0.o0 <= j && j + PPL <= A0.o1 && A0.o1 <= n_points;
    const bool in1 = A1.o0 >= 0 && A1.o0 <= j && j + PPL <= A1.o1 && A1.o1 <= n_points;
    if (!in0 && !in1) {
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
            const int64_t jq = j + q;
            if (jq >= n_points) break;
            const AtomRef B = load_atom(lane_search(offsets, n_atoms, jq));
            if (!(B.o0 >= 0 && B.o0 <= jq && jq < B.o1 && B.o1 <= n_points)) continue;
            proj_point<LMAX, TIO>(px[q], py[q], pz[q], B.c, table + int64_t(B.t) * g.n_r * tab_ch, tab_ch, g,
                                  out + F * B.o0 + (jq - B.o0), B.o1 - B.o0);
        }
        return;
    }
    const AtomRef& A = in0 ? A0 : A1;
    const knot_t<TIO>* tab = table + int64_t(A.t) * g.n_r * tab_ch;
    knot_t<TIO> ka[PPL][LMAX + 1], kb[PPL][LMAX + 1];
    double r[PPL];
    V x, y, z, k;
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        const double dx = px[q] - A.c[0], dy = py[q] - A.c[1], dz = pz[q] - A.c[2];
        double xb, yb, zb, keep;
        normalize(dx, dy, dz, xb, yb, zb, keep);
        r[q] = sqrt(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)));
        spline_knots<LMAX + 1>(tab, tab_ch, g, r[q], ka[q], kb[q]);
        lane<V, PPL>(x, q) = TIO(xb);
        lane<V, PPL>(y, q) = TIO(yb);
        lane<V, PPL>(z, q) = TIO(zb);
        lane<V, PPL>(k, q) = TIO(keep);
    }
    TIO R[PPL][LMAX + 1];
#pragma unroll
    for (int q = 0; q < PPL; ++q) spline_from<LMAX + 1, TIO>(ka[q], kb[q], g, r[q], R[q]);
    TIO* o = out + F * A.o0 + (j - A.o0);
    const int64_t stride = A.o1 - A.o0;
    eval_unit<LMAX, V>(x, y, z, k, [&](int f, V v) {
        const int l = l_of_row(f);
        V rl;
#pragma unroll
        for (int q = 0; q < PPL; ++q) lane<V, PPL>(rl, q) = R[q][l];
        store_run<TIO, PPL>(o + int64_t(f) * stride, rl * v, PPL);
    });
}

// Points per launch: keeps each grid well inside the 32-bit work-item count of a
// dispatch (a multiple of every lane width, so only the last launch has a tail).
constexpr int64_t kProjChunk = int64_t(1) << 28;

template <int LMAX, typename TIO, int P>
static void launch_vec(const ProjArgs<TIO>& A, const SplineGrid& g, dim3 grid, size_t lds, int64_t j0, hipStream_t s)
{
    if constexpr (P > 1 && (kProjVecKernel<TIO, LMAX> || kProjVecWindow<TIO, LMAX>))
        hipLaunchKernelGGL((proj_vec_kernel<LMAX, TIO, P>), grid, dim3(256), lds, s, A.centers, A.offsets,
                           A.n_atoms, A.points, A.n_points, A.table, A.tab_ch, A.n_tables, A.table_of_atom, g,
                           A.out, j0);
}

template <int LMAX, typename TIO, int P>
static hipError_t launch_proj_p(const ProjArgs<TIO>& A, hipStream_t s)
{
    const SplineGrid g{A.n_r, A.h, 1.0 / A.h, A.r_max, A.h * A.h / 6.0};
    const size_t lds = P > 1 ? kProjCapLds<TIO, LMAX> : 0;
    for (int64_t j0 = 0; j0 < A.n_points; j0 += kProjChunk) {
        const int64_t nc = A.n_points - j0 < kProjChunk ? A.n_points - j0 : kProjChunk;
        const dim3 grid = dim3(unsigned((nc + 256 * P - 1) / (256 * P))), block = dim3(256);
        const bool vec = P > 1 && (A.n_atoms <= 64 ? kProjVecKernel<TIO, LMAX> : kProjVecWindow<TIO, LMAX>);
        if (P == 1 && A.n_atoms <= 64)
            hipLaunchKernelGGL((proj_kernel<LMAX, TIO, P, P == 1>), grid, block, 0, s, A.centers, A.offsets,
                               A.n_atoms, A.points, A.n_points, A.table, A.tab_ch, A.n_tables, A.table_of_atom, g,
                               A.out, j0);
        else if (vec)
            launch_vec<LMAX, TIO, P>(A, g, grid, lds, j0, s);
        else
            hipLaunchKernelGGL((proj_kernel<LMAX, TIO, P, false>), grid, block, lds, s, A.centers, A.offsets,
                               A.n_atoms, A.points, A.n_points, A.table, A.tab_ch, A.n_tables, A.table_of_atom, g,
                               A.out, j0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int LMAX, typename TIO>
static hipError_t launch_proj_l(const ProjArgs<TIO>& A, hipStream_t s)
{
    return A.n_points >= kProjVecPoints ? launch_proj_p<LMAX, TIO, kProjPpl<TIO, LMAX>>(A, s)
                                        : launch_proj_p<LMAX, TIO, 1>(A, s);
}

template <typename TIO>
hipError_t launch_projectors(int lmax, const ProjArgs<TIO>& A, hipStream_t s)
{
    switch (lmax) {
    case 0: return launch_proj_l<0, TIO>(A, s);
    case 1: return launch_proj_l<1, TIO>(A, s);
    case 2: return launch_proj_l<2, TIO>(A, s);
    case 3: return launch_proj_l<3, TIO>(A, s);
    case 4: return launch_proj_l<4, TIO>(A, s);
    case 5: return launch_proj_l<5, TIO>(A, s);
    case 6: return launch_proj_l<6, TIO>(A, s);
    case 7: return launch_proj_l<7, TIO>(A, s);
    case 8: return launch_proj_l<8, TIO>(A, s);
    case 9: return launch_proj_l<9, TIO>(A, s);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_projectors<double>(int, const ProjArgs<double>&, hipStream_t);
template hipError_t launch_projectors<float>(int, const ProjArgs<float>&, hipStream_t);

// out[row][c] = in[row][c] for c < ch_out (rows of ch_in pairs in, ch_out out)
template <typename P>
__global__ void compact_tables_kernel(const P* __restrict__ in, P* __restrict__ out, int64_t rows, int ch_in,
                                      int ch_out)
{
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= rows * ch_out) return;
    const int64_t row = k / ch_out;
    out[k] = in[row * ch_in + (k - row * ch_out)];
}

template <typename P>
hipError_t launch_compact_tables(const P* in, P* out, int64_t rows, int ch_in, int ch_out, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    if (ch_out < 1 || ch_out > ch_in) return hipErrorInvalidValue;
    const int64_t n = rows * ch_out;
    hipLaunchKernelGGL((compact_tables_kernel<P>), dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, in, out, rows,
                       ch_in, ch_out);
    return hipGetLastError();
}

template hipError_t launch_compact_tables<double2>(const double2*, double2*, int64_t, int, int, hipStream_t);
template hipError_t launch_compact_tables<float2>(const float2*, float2*, int64_t, int, int, hipStream_t);

hipError_t launch_spline_setup(const double* y, double2* table, float2* table_f32, double2* work, double* scratch,
                               int n_ch, int ch, int n_r, double h, hipStream_t s)
{
    // a dispatch counts its work-items in 32 bits
    constexpr int64_t kChunk = int64_t(1) << 22;
    // A workgroup per channel costs 8.5 us per 1000 channels whatever their length up to
    // kSplineTile, a thread per channel about 0.75 us per knot until the lanes fill the GPU.
    // Measured, thread against workgroup per channel, with a one-tile build after it:
    // 260000 x 8 knots 50 / 1874 us, 10000 x 64 55 / 90, 16000 x 128 104 / 148, 1000 x 16
    // 18 / 17, 8000 x 256 202 / 84, 168 x 300 190 / 17, 168 x 2000 1390 / 18.
    const bool serial = n_ch > int64_t(96) * n_r;
    for (int64_t c0 = 0; c0 < n_ch; c0 += kChunk) {
        const int64_t nc = n_ch - c0 < kChunk ? n_ch - c0 : kChunk;
        if (serial)
            hipLaunchKernelGGL(spline_serial_kernel, dim3(unsigned((nc + 63) / 64)), dim3(64), 0, s, y, table,
                               table_f32, work, scratch, c0, int64_t(n_ch), ch, n_r, 6.0 / (h * h));
        else
            hipLaunchKernelGGL(spline_setup_kernel, dim3(unsigned(nc)), dim3(kSplineBlock), 0, s, y, table, table_f32,
                               work, scratch, c0, ch, n_r, 6.0 / (h * h));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace shk
