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
// Launch: workgroups remapped so each XCD works through one contiguous range of atoms
// (their tables then stay in that XCD's L2); the atom of a wave found by one wave-wide
// search or from a preload; plain stores; one point per lane, or several in large builds,
// some of which hold the atom's table in LDS (launch_proj_l).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

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
// (0.74 us per knot, 168 lanes of the GPU busy); this takes 9-11 us (13-14 before every load
// of a tile and of the c_k was issued ahead of the first wait).
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
    auto coefs = [&](int k0, double (&ck)[kSplinePer + 1]) {
#pragma unroll
        for (int i = 0; i <= kSplinePer; ++i) ck[i] = spline_c(k0 + i - 1 < 0 ? 0 : k0 + i - 1);
    };
    double d[kSplinePer];
    double carry = 0.0;
    for (int t = 0; t < nt; ++t) {
        const int base = t * kSplineTile;
        // slot j holds y[base - 1 + j] (beyond the ends, where no interior knot looks, the
        // end's value again); every load is issued before the first is waited for
        double yv[kSplinePer + 1];
#pragma unroll
        for (int q = 0; q <= kSplinePer; ++q) {
            const int k = base - 1 + tid + q * kSplineBlock;
            yv[q] = yc[k < 0 ? 0 : (k < n_r ? k : n_r - 1)];
        }
#pragma unroll
        for (int q = 0; q <= kSplinePer; ++q)
            if (q < kSplinePer || tid < 2) ys[spline_slot(tid + q * kSplineBlock)] = yv[q];
        const int k0 = base + tid * kSplinePer;
        double ck[kSplinePer + 1];  // c_{k0 - 1} .. c_{k0 + kSplinePer - 1}, asked for together
        coefs(k0, ck);
        __syncthreads();
        bool bad = false;
        Affine own{1.0, 0.0};
#pragma unroll
        for (int i = 0; i < kSplinePer; ++i) {
            const int j = tid * kSplinePer + i;
            const double rhs = six_over_h2 * (ys[spline_slot(j + 2)] - 2.0 * ys[spline_slot(j + 1)] + ys[spline_slot(j)]);
            d[i] = rhs;
            if (interior(k0 + i)) {
                own.b = (rhs - own.b) * ck[i + 1];
                own.a = -own.a * ck[i + 1];
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
                const double x = d[i] - v, den = 4.0 - ck[i], q = x * ck[i + 1];
                v = __builtin_fma(__builtin_fma(-q, den, x), ck[i + 1], q);
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
        double ck[kSplinePer + 1];
        coefs(k0, ck);
        Affine own{1.0, 0.0};
#pragma unroll
        for (int i = kSplinePer - 1; i >= 0; --i) {
            if (nt > 1) d[i] = k0 + i < n_r ? dc[k0 + i] : 0.0;
            if (interior(k0 + i)) {
                own.b = d[i] - ck[i + 1] * own.b;
                own.a = -ck[i + 1] * own.a;
            } else {
                own = Affine{0.0, 0.0};
            }
        }
        const Affine m = block_before<true>(own, tot);
        double v = m.a * carry + m.b;
#pragma unroll
        for (int i = kSplinePer - 1; i >= 0; --i) {
            v = interior(k0 + i) ? d[i] - ck[i + 1] * v : 0.0;
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
// point per lane): 29.6-29.8 us -> 27.6-28.0 us.  Which launches take it: kProjSmall.
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

// Points w0 .. w0 + 63 of a wave, those below `end`, one per lane and of any atoms, from
// tables of LMAX + 1 channels in memory.  The 64 offsets after the wave's first atom are held
// in the lanes, where each lane finds its atom; only points beyond them search on.
template <int LMAX, typename TIO>
__device__ __forceinline__ void proj_wave(const TIO* __restrict__ centers, const int64_t* __restrict__ offsets,
                                          int n_atoms, const TIO* __restrict__ points, int64_t n_points,
                                          const knot_t<TIO>* __restrict__ table, int n_tables,
                                          const int32_t* __restrict__ table_of_atom, const SplineGrid& g,
                                          TIO* __restrict__ out, int64_t w0, int64_t end)
{
    const int lane = threadIdx.x & 63;
    const int64_t j = w0 + lane;
    const TIO* p = points + 3 * (j < end ? j : w0);
    const double px = double(p[0]), py = double(p[1]), pz = double(p[2]);
    const int aw = max(wave_search(offsets, n_atoms, w0), 0);
    const int64_t after = offsets[min(aw + 1 + lane, n_atoms)];
    int k = 0;  // how many of them are <= j (63 at most)
#pragma unroll
    for (int s = 32; s > 0; s /= 2)
        if (__shfl(after, k + s - 1) <= j) k += s;
    if (j >= end) return;
    int a = min(aw + k, n_atoms - 1);
    int64_t o0 = offsets[a], o1 = offsets[a + 1];
    if (!(o0 <= j && j < o1)) {
        a = lane_search(offsets, n_atoms, j);
        o0 = offsets[a];
        o1 = offsets[a + 1];
    }
    if (!(o0 >= 0 && o0 <= j && j < o1 && o1 <= n_points)) return;
    const double c[3] = {double(centers[3 * a]), double(centers[3 * a + 1]), double(centers[3 * a + 2])};
    int t = table_of_atom ? table_of_atom[a] : a;
    t = t < 0 ? 0 : (t >= n_tables ? n_tables - 1 : t);
    proj_point<LMAX, TIO>(px, py, pz, c, table + int64_t(t) * g.n_r * (LMAX + 1), LMAX + 1, g,
                          out + nfun(LMAX) * o0 + (j - o0), o1 - o0);
}

// A workgroup's points, and the atom at their beginning with its own.
struct ProjShare {
    int64_t begin, end, o0, o1;
    int a;
};

// Persistent build for small lmax: a workgroup keeps the spline table of the atom it works
// on in LDS (of LMAX + 1 channels) and walks tiles of BT * PPL points.  A lookup
// scatters its lanes over as many cache lines, one tag check each: at lmax 3 in FP32 two
// thirds of the L1's cycles went there, and where the tables of many atoms outgrow the L2
// it waited for them as well.  Workgroups form groups of `group` (of the logical order, so
// in one XCD), each with consecutive points, whose tiles its workgroups take in turn: with
// group = 32 an XCD's CUs write side by side, which the HBM write path rewards, and each
// loads every table of the range; with group = 1 a workgroup loads one or two.
// A table costs as much as load_cost points, and so does an atom that has few of them: the
// points are dealt out by that cost (an atom's place in it is its offset plus its number of
// load costs, so a search finds a share's ends), and a run of fewer points than load_cost
// whose table is not the one held goes through memory, one point per lane, with what follows
// it, as do offsets that are inconsistent.  One atom of 3M points among 1000 of 10, in us
// with a table load for each atom and equal points, so, and without LDS: FP32 lmax 0 1329 / 15 /
// 22, lmax 2 2140 / 42 / 51, lmax 4 2821 / 113 / 89, FP64 lmax 1 1809 / 45 / 53, lmax 3 1492 /
// 126 / 103; four of 800000 among 300 of 300 FP32 lmax 0 64 / 26 / 17, lmax 2 189 / 47 / 45, lmax
// 4 176 / 120 / 85, FP64 lmax 1 167 / 46 / 55, lmax 3 176 / 136 / 110.  The same arithmetic, so
// the same bits.
// us against the best launch without LDS: 64 x 150k points FP64 lmax 1 116-122 / 141, FP32
// lmax 2 109-112 / 124, lmax 3 160 / 157, lmax 4 164 / 155, FP64 lmax 2 (64 x 100k) 143 /
// 147, lmax 3 345 / 304; 200 x 20k FP32 lmax 3 76 / 88, lmax 4 110 / 118; 1024 x 9400 FP32
// lmax 0 43 / 59, lmax 2 120 / 167, lmax 3 179 / 224, FP64 lmax 0 74 / 107, lmax 1 135 /
// 192, lmax 3 361 / 392; 512 x 4000 FP32 lmax 2 34 / 46, FP64 lmax 1 37 / 45.
template <int LMAX, typename TIO, int PPL, int BT>
__global__ __launch_bounds__(BT) void proj_lds_kernel(const TIO* __restrict__ centers,
                                                      const int64_t* __restrict__ offsets, int n_atoms,
                                                      const TIO* __restrict__ points, int64_t n_points,
                                                      const knot_t<TIO>* __restrict__ table,
                                                      int n_tables, const int32_t* __restrict__ table_of_atom,
                                                      SplineGrid g, TIO* __restrict__ out, int64_t group_cost,
                                                      int group_log, int load_cost)
{
    using KN = knot_t<TIO>;
    constexpr int F = nfun(LMAX), CH = LMAX + 1;
    extern __shared__ __align__(16) unsigned char lds[];
    KN* tab = reinterpret_cast<KN*>(lds);
    const uint32_t w = xcd_tile(blockIdx.x, gridDim.x);
    // The group's share: load_cost units before each atom's points, one for each of them.  One
    // wave finds it for all (every wave doing so took 1 us of a build's 12).
    ProjShare& share = *reinterpret_cast<ProjShare*>(lds);
    if (threadIdx.x < 64) {
        const int64_t gi = w >> group_log, cost = n_points + int64_t(n_atoms) * load_cost;
        const int64_t x[2] = {gi * group_cost, (gi + 1) * group_cost};
        int at[2];
        wave_searches<2>(n_atoms, [&](int k) { return offsets[k] + int64_t(k) * load_cost; }, x, at);
        int64_t from[2], till[2], end[2];  // the atom that each end of the share lies in, and where
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int b = max(at[i], 0);
            from[i] = offsets[b];
            till[i] = offsets[b + 1];
            // no share begins or ends within an atom's first or last points that are too few for a load
            const int64_t in = x[i] - (from[i] + (int64_t(b) + 1) * load_cost);
            const int64_t p = in < load_cost                       ? from[i]
                              : in < till[i] - from[i] - load_cost ? from[i] + in / 64 * 64
                                                                   : till[i];
            end[i] = x[i] >= cost ? n_points : (p < 0 || x[i] == 0 ? 0 : (p < n_points ? p : n_points));
        }
        if (threadIdx.x == 0) share = ProjShare{end[0], end[1], from[0], till[0], at[0]};
    }
    __syncthreads();
    const int64_t g0 = lane_value(share.begin, 0), g1 = lane_value(share.end, 0);
    int64_t o0 = lane_value(share.o0, 0), o1 = lane_value(share.o1, 0);  // the points of
    int a = lane_value(share.a, 0);                                      // the atom looked at last
    bool here = false;                      // whether it is the current one
    int t = -1;                             // the table held in LDS
    double c[3] = {};
    const uint32_t wi = w & ((1u << group_log) - 1);
    for (int64_t p0 = g0 + int64_t(wi) * (BT * PPL); p0 < g1; p0 += int64_t(BT * PPL) << group_log) {
        const int64_t p1 = p0 + BT * PPL < g1 ? p0 + BT * PPL : g1;
        int64_t pos = p0;
        while (pos < p1) {
            if (!(here && pos < o1)) {
                if (!(a >= 0 && o0 <= pos && pos < o1)) {
                    a = wave_search(offsets, n_atoms, pos);
                    o0 = offsets[max(a, 0)];
                    o1 = offsets[max(a, 0) + 1];
                }
                bool general = a < 0 || o0 < 0 || !(o0 <= pos && pos < o1) || o1 > n_points;  // inconsistent here
                int ta = 0;
                if (!general) {
                    ta = table_of_atom ? table_of_atom[a] : a;
                    ta = ta < 0 ? 0 : (ta >= n_tables ? n_tables - 1 : ta);
                    // the points of this atom that fall to this workgroup from here on
                    const int64_t left = (o1 < g1 ? o1 : g1) - pos, tile = p1 - pos;
                    general = ta != t && (left <= tile ? left : tile + ((left - tile) >> group_log)) < load_cost;
                }
                here = !general;
                if (general) {
                    const int64_t q = pos + BT < p1 ? pos + BT : p1, w0 = pos + (threadIdx.x & ~63u);
                    if (w0 < q)
                        proj_wave<LMAX, TIO>(centers, offsets, n_atoms, points, n_points, table, n_tables,
                                             table_of_atom, g, out, w0, q);
                    pos = q;
                    continue;
                }
                c[0] = double(centers[3 * a]);
                c[1] = double(centers[3 * a + 1]);
                c[2] = double(centers[3 * a + 2]);
                if (ta != t) {
                    t = ta;
                    __syncthreads();  // the previous table, or the share, is still read
                    const KN* src = table + int64_t(t) * g.n_r * CH;
                    typedef float v4 __attribute__((ext_vector_type(4), aligned(8)));  // a float pair's
                    const int n16 = int(g.n_r * CH * sizeof(KN) / 16);
                    for (int k = threadIdx.x; k < n16; k += BT)
                        reinterpret_cast<v4*>(tab)[k] = reinterpret_cast<const v4*>(src)[k];
                    if (sizeof(KN) == 8 && (g.n_r * CH & 1) && threadIdx.x == 0)
                        tab[g.n_r * CH - 1] = src[g.n_r * CH - 1];
                    __syncthreads();
                }
            }
            const int64_t e = o1 < p1 ? o1 : p1;
            int64_t j = pos + int64_t(threadIdx.x) * PPL;
            if (j < e) {
                int nvalid = PPL;
                if (j + PPL > e) {
                    // the atom's last lane takes its last PPL points (its neighbour, which
                    // takes some of them too, stores the same bits); atoms with fewer
                    // points before e store those there are
                    if (e - PPL >= o0) j = e - PPL;
                    else nvalid = int(e - j);
                }
                double px[PPL], py[PPL], pz[PPL];
#pragma unroll
                for (int q = 0; q < PPL; ++q) {
                    const TIO* p = points + 3 * (q < nvalid ? j + q : j);
                    px[q] = double(p[0]);
                    py[q] = double(p[1]);
                    pz[q] = double(p[2]);
                }
                proj_points<LMAX, TIO, PPL>(px, py, pz, c, tab, CH, g, out + F * o0 + (j - o0), o1 - o0, nvalid);
            }
            pos = e;
        }
    }
}

// Points per launch: keeps each grid well inside the 32-bit work-item count of a
// dispatch (a multiple of every lane width, so only the last launch has a tail).
constexpr int64_t kProjChunk = int64_t(1) << 28;

// The atoms of a launch over at most 64 are loaded into the lanes together with the points
// and found by a ballot, instead of by a search over the offsets first (a chain of dependent
// loads).  us with and without, 2 workgroups per CU, several points per lane: FP64 lmax 3, 64 x
// 14137 points 38.3 / 39.5, 64 x 150000 309 / 313; FP32 lmax 3 157 / 162, lmax 4, 64 x 50000
// 86.9 / 90.9; from lmax 5 on equal, so only the search there.
template <int P, int LMAX> constexpr bool kProjSmall = P == 1 || LMAX <= 4;

template <int LMAX, typename TIO, int P>
static hipError_t launch_proj_p(const ProjArgs<TIO>& A, const SplineGrid& g, size_t lds, hipStream_t s)
{
    for (int64_t j0 = 0; j0 < A.n_points; j0 += kProjChunk) {
        const int64_t nc = A.n_points - j0 < kProjChunk ? A.n_points - j0 : kProjChunk;
        const dim3 grid = dim3(unsigned((nc + 256 * P - 1) / (256 * P))), block = dim3(256);
        if (kProjSmall<P, LMAX> && A.n_atoms <= 64)
            hipLaunchKernelGGL((proj_kernel<LMAX, TIO, P, kProjSmall<P, LMAX>>), grid, block, lds, s, A.centers,
                               A.offsets, A.n_atoms, A.points, A.n_points, A.table, A.tab_ch, A.n_tables,
                               A.table_of_atom, g, A.out, j0);
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
static hipError_t launch_proj_lds(const ProjArgs<TIO>& A, const SplineGrid& g, hipStream_t s)
{
    if constexpr (LMAX <= kProjLdsMax<TIO>) {
        constexpr int BT = kProjLdsBlock<TIO, LMAX>, P = kProjPpl<TIO>;
        const int group_log = proj_lds_group<TIO, LMAX>(A.n_atoms, A.n_points) == 1 ? 0 : 5, wgs = kCus * (1024 / BT);
        const int64_t n_groups = wgs >> group_log, load_cost = kProjLoadCost + proj_lds_bytes<TIO, LMAX>(A.n_r) / 256;
        const int64_t group_cost = (A.n_points + A.n_atoms * load_cost + n_groups - 1) / n_groups;
        hipLaunchKernelGGL((proj_lds_kernel<LMAX, TIO, P, BT>), dim3(wgs), dim3(BT),
                           std::max(size_t(proj_lds_bytes<TIO, LMAX>(A.n_r)), sizeof(ProjShare)), s, A.centers,
                           A.offsets, A.n_atoms, A.points, A.n_points, A.table, A.n_tables, A.table_of_atom, g, A.out,
                           group_cost, group_log, int(load_cost));
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

template <int LMAX, typename TIO>
static hipError_t launch_proj_l(const ProjArgs<TIO>& A, hipStream_t s)
{
    const SplineGrid g{A.n_r, A.h, 1.0 / A.h, A.r_max, A.h * A.h / 6.0};
    if (A.n_points < kProjVecPoints && A.n_points * nfun(LMAX) * int64_t(sizeof(TIO)) < kProjVecBytes)
        return launch_proj_p<LMAX, TIO, 1>(A, g, 0, s);
    if (use_proj_lds<TIO, LMAX>(A.n_atoms, A.n_points, A.tab_ch, A.n_r)) return launch_proj_lds<LMAX, TIO>(A, g, s);
    return launch_proj_p<LMAX, TIO, kProjPpl<TIO>>(A, g, proj_cap_lds<TIO, LMAX>(A.n_atoms, A.n_points), s);
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
    // A workgroup per channel costs 7 us per 1000 channels whatever their length up to
    // kSplineTile, a thread per channel about 0.75 us per knot until the lanes fill the GPU.
    // Measured, thread against workgroup per channel, with a one-tile build after it:
    // 260000 x 8 knots 50 / 1568 us, 10000 x 64 56 / 72, 16000 x 128 106 / 115, 1000 x 16
    // 18 / 16, 8000 x 256 201 / 67, 168 x 300 191 / 12, 168 x 2000 1395 / 16.
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
