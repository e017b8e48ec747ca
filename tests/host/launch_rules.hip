// Test-only: host build of the rules that choose a launch from sizes and alignment, so that
// the lines between launches can be checked on the CPU.
#include "../../paper_2510_05282_amd/csrc/sh_proj.h"

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
