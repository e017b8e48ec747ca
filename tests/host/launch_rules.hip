// Test-only: host build of the rules that choose a launch from sizes and alignment, so that
// the lines between launches can be checked on the CPU.
#include "../../paper_2510_05282_amd/csrc/sh_proj.h"
#include "../../paper_2510_05282_amd/csrc/sh_rec.h"

// 0: no tables in LDS; else how many workgroups go side by side.
template <typename TIO, int LMAX>
static int proj_lds(int n_atoms, int64_t n_points, int tab_ch, int n_r)
{
    return shk::use_proj_lds<TIO, LMAX>(n_atoms, n_points, tab_ch, n_r)
               ? shk::proj_lds_group<TIO, LMAX>(n_atoms, n_points)
               : 0;
}

template <typename TIO>
static int proj_lds_of(int lmax, int n_atoms, int64_t n_points, int tab_ch, int n_r)
{
    switch (lmax) {
    case 0: return proj_lds<TIO, 0>(n_atoms, n_points, tab_ch, n_r);
    case 1: return proj_lds<TIO, 1>(n_atoms, n_points, tab_ch, n_r);
    case 2: return proj_lds<TIO, 2>(n_atoms, n_points, tab_ch, n_r);
    case 3: return proj_lds<TIO, 3>(n_atoms, n_points, tab_ch, n_r);
    case 4: return proj_lds<TIO, 4>(n_atoms, n_points, tab_ch, n_r);
    default: return proj_lds<TIO, 5>(n_atoms, n_points, tab_ch, n_r);
    }
}

extern "C" int rule_proj_lds(int f64, int lmax, int n_atoms, long n_points, int tab_ch, int n_r)
{
    return f64 ? proj_lds_of<double>(lmax, n_atoms, n_points, tab_ch, n_r)
               : proj_lds_of<float>(lmax, n_atoms, n_points, tab_ch, n_r);
}

// KiB of LDS reserved, plus 1000 where lanes take several points.
template <int ROWS>
static int store(int f64, int64_t n, int value, int in_bytes, int lines)
{
    const shk::StoreShape s = f64 ? shk::store_shape<ROWS, double>(n, value, in_bytes, lines)
                                  : shk::store_shape<ROWS, float>(n, value, in_bytes, lines);
    return (s.wide ? 1000 : 0) + int(s.lds / 1024);
}

extern "C" int rule_store(int rows, int f64, long n, int value, int in_bytes, int lines)
{
    switch (rows) {
    case 1: return store<1>(f64, n, value, in_bytes, lines);
    case 4: return store<4>(f64, n, value, in_bytes, lines);
    case 9: return store<9>(f64, n, value, in_bytes, lines);
    case 16: return store<16>(f64, n, value, in_bytes, lines);
    case 25: return store<25>(f64, n, value, in_bytes, lines);
    case 36: return store<36>(f64, n, value, in_bytes, lines);
    case 64: return store<64>(f64, n, value, in_bytes, lines);
    case 100: return store<100>(f64, n, value, in_bytes, lines);
    case 324: return store<324>(f64, n, value, in_bytes, lines);
    case 400: return store<400>(f64, n, value, in_bytes, lines);
    default: return -1;
    }
}

// KiB of LDS reserved, plus 1000 where lanes take several points, 2000 where the m are split,
// and 10000 times the degrees at a time.  kind: 0 real, 1 complex, 2 spinor.
static int rec(const shk::RecShape& f)
{
    return 10000 * f.unroll + (f.wide ? 1000 : 0) + (f.split ? 2000 : 0) + int(f.lds / 1024);
}

template <typename TIO>
static int rec_of(int kind, int lmax, int64_t n, int lines)
{
    const int64_t b = n * (lmax + 1) * (lmax + 1) * int64_t(sizeof(TIO));
    if (kind == 0) return rec(shk::rec_shape<TIO>(n, b, lines));
    return kind == 1 ? rec(shk::rec_cplx_shape<TIO, false>(n, 2 * b, lines))
                     : rec(shk::rec_cplx_shape<TIO, true>(n, 8 * b, lines));
}

// 0: loads that keep lines, 1: non-temporal, 2: kept off the lines.
template <typename TIO>
static int grad_read_of(int lmax, int64_t n, int lines)
{
    switch (lmax) {
    case 0: return int(shk::grad_read<0, TIO>(n, lines));
    case 1: return int(shk::grad_read<1, TIO>(n, lines));
    case 2: return int(shk::grad_read<2, TIO>(n, lines));
    case 3: return int(shk::grad_read<3, TIO>(n, lines));
    case 4: return int(shk::grad_read<4, TIO>(n, lines));
    default: return int(shk::grad_read<9, TIO>(n, lines));
    }
}

extern "C" int rule_grad_read(int f64, int lmax, long n, int lines)
{
    return f64 ? grad_read_of<double>(lmax, n, lines) : grad_read_of<float>(lmax, n, lines);
}

// Points per lane, plus 2000 where the m are split, and 10000 times the degrees at a time.
extern "C" int rule_grad_rec(int f64, int lmax, long n)
{
    const shk::GradRecShape f = f64 ? shk::grad_rec_shape<double>(lmax, n) : shk::grad_rec_shape<float>(lmax, n);
    return 10000 * f.unroll + (f.split ? 2000 : 0) + f.ppl;
}

extern "C" int rule_rec(int kind, int f64, int lmax, long n, int lines)
{
    return f64 ? rec_of<double>(kind, lmax, n, lines) : rec_of<float>(kind, lmax, n, lines);
}
