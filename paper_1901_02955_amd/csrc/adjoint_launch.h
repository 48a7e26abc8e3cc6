// Dispatch of the adjoint kernels for one element type (included once per type).
#pragma once

#include <cstdlib>

#include "snap_adjoint.h"
#include "snap_internal.h"

namespace snap {

// Blocks of up to 512 threads in rows of at most 2^22: a launch holds fewer than
// 2^32 threads along an axis, which a wave per line passes from 2^26 short lines
// on (8192 x 8192 x 2 in single precision: 27 GB for all arrays).
inline dim3 lane_grid(long long blocks) {
  const long long rows = (blocks + (1LL << 22) - 1) >> 22;
  return dim3((unsigned)((blocks + rows - 1) / rows), (unsigned)rows);
}

template <typename T, int NV, int D, bool HLLC, bool MIX>
void adj_lane_launch(const T* q, const T* r, const AdjArgs& a, T* P, const FoldOut<T>& fo,
                     hipStream_t st) {
  const int nd = D == 0 ? a.nx : (D == 1 ? a.ny : a.nz);
  const int nseg = lane_segments(nd), lw = lane_width(nd);
  const int nlw = lane_waves<T, D>() << (6 - lw);   // lines per workgroup
  const long long groups = D == 0 ? ((long long)a.ny * a.nz + nlw - 1) / nlw
                                  : (long long)((a.nx + nlw - 1) / nlw) * (D == 1 ? a.nz : a.ny);
  hipLaunchKernelGGL((k_adj_lane<T, NV, D, HLLC, MIX>), lane_grid(groups * nseg),
                     dim3(64 * lane_waves<T, D>()), 0, st, q, r, a, nseg, (int)groups, lw, P, fo);
}

// The y and z directions march along their lines (k_adj_march) in single
// precision with up to 7 variables, where the march's register window fits,
// where each variable's padded plane is smaller than 2 GiB, and on grids where
// it is the faster one (march_pays); otherwise they take the lane kernel. In
// double precision the march's window needs over 256 registers (five variables:
// 240 bytes of scratch per lane at two waves per SIMD). SNAP_ADJ_MARCH=0 selects
// the lane kernel everywhere, SNAP_ADJ_MARCH=1 (or a segment length in
// SNAP_ADJ_MARCH_SEG) the march on every grid where it fits.
template <typename T, int NV>
constexpr bool march_fits() {
  return sizeof(T) == 4 && NV <= 7;
}

// The march holds more cells per instruction (no halo lanes) but needs long
// lines in large numbers to fill the chip; the lane kernel fills it on any
// grid. Microseconds of one gradient step (single precision; march, lane):
// 5 variables 96x96x48 486, 376; 160x160x80 1247, 1172; 192x160x96 (six steps)
// 6881, 6652; 256x256x128 4002, 4580;
// 7 variables 96x96x48 637, 489; 160x160x80 1674, 1612; 256x256x128 5850, 6575.
// Of one right-hand-side adjoint, 5 and 7 variables: 200x200x110 (4.4e6 cells) 517,
// 538; 729, 797. The line lies between those sizes. Flat grids would cross
// over earlier (512x512x12, 3.1e6: 383, 461; 300x24x300, 2.2e6: 288, 318), narrow
// ones later (24x300x300, 2.2e6: 381, 338), which the rule leaves out.
// (read at every launch, so that a process can compare both kernels)
inline bool march_pays(const AdjArgs& a) {
  const char* e = getenv("SNAP_ADJ_MARCH");
  if (e && (e[0] == '0' || e[0] == '1')) return e[0] == '1';
  const char* seg = getenv("SNAP_ADJ_MARCH_SEG");
  if (seg && atoi(seg) > 0) return true;
  return (double)a.nx * a.ny * a.nz >= 4.2e6;
}

// The z direction folds the cells at least 3 from the y and z edges, after
// k_adj_xmerge has added the x copies' cotangents into the cells within 3 of
// an x edge (the separate fold pass then covers the rows of the 3 lowest and 3
// highest levels and those within 3 of a y edge), where that takes enough blocks
// (256 cells of a row) off the fold pass to pay for the merge's launch of 2 to 4 us.
// Microseconds of a right-hand-side adjoint in double precision without tracers
// (blocks saved: folded, not): 16x16x16 (100) 39.2, 36.5; 320x1x200 (388) 35.8,
// 32.8; 40x40x40 (1156) 49.4, 50.1; 16x1x2000 (1994) 31.1, 31.7; 96x80x64 (4292)
// 150, 159. Not under the mixture, whose fold costs the z kernel what it saves:
// 96 x 80 x 64 with six tracers in double precision 174 us and 71 for the separate
// fold, against 219 and 19. SNAP_ADJ_MARCH_FOLD=0 leaves every cell to the fold
// pass, SNAP_ADJ_MARCH_FOLD=1 folds on every grid that has such cells.
inline bool fold_pays(const AdjArgs& a) {
  if (a.nz <= 6) return false;
  const char* e = getenv("SNAP_ADJ_MARCH_FOLD");
  if (e && (e[0] == '0' || e[0] == '1')) return e[0] == '1';
  const long long rows = (long long)(!a.d3 ? 1 : (a.ny > 6 ? a.ny - 6 : 0)) * (a.nz - 6);
  return rows * ((a.nx + 255) / 256) >= 1024;
}

// Segment length of the march. A line is cut into as many segments as make the
// launch fastest by this estimate: a segment takes its cells plus 6 for the halo
// it recomputes; m = blocks per compute unit share each SIMD, which issues 0.5,
// 0.8 or 0.95 of the time with one, two or three waves (up to `waves` at once).
// For 256 x 256 x 128 that gives 43-cell z and y segments, the measured best
// (24, 32, 43 and 64 cells: 1.100, 1.107, 1.085 and 1.133 ms per right-hand-side
// adjoint); for 192 x 160 x 96, where 32-cell segments left one to two waves per
// SIMD, 16 cells (189 -> 140 us in z, 176 -> 123 in y). SNAP_ADJ_MARCH_SEG
// overrides the length.
inline int march_seglen(int nd, long long lines, int waves) {
  const char* e = getenv("SNAP_ADJ_MARCH_SEG");
  const int v = e ? atoi(e) : 0;
  int best = (nd + (v > 0 ? v : nd) - 1) / (v > 0 ? v : nd);
  if (v <= 0) {
    constexpr double issue[3] = {0.5, 0.8, 0.95};
    constexpr long long CUS = 256;
    const long long row = (lines + 255) / 256;
    double cost = 1e300;
    for (int n = 1; n <= nd / 4 + 1; ++n) {
      const int len = (nd + n - 1) / n;
      const long long m = (row * ((nd + len - 1) / len) + CUS - 1) / CUS;
      const double c = (double)m * (len + 6) / issue[(m < waves ? m : waves) - 1];
      if (c < cost) {
        cost = c;
        best = n;
      }
    }
  }
  return (nd + best - 1) / best;
}

template <typename T, int NV, int D, bool HLLC>
void adj_march_launch(const T* q, const T* r, const AdjArgs& a, T* P, const MarchFold<T>& fo,
                      hipStream_t st) {
  const int nd = D == 2 ? a.nz : a.ny;
  const long long lines = (long long)a.nx * (D == 2 ? a.ny : a.nz);
  const int seg = march_seglen(nd, lines, NV <= 5 ? 3 : 2);
  const dim3 grid((unsigned)((lines + 255) / 256), (unsigned)((nd + seg - 1) / seg));
  hipLaunchKernelGGL((k_adj_march<T, NV, D, HLLC>), grid, dim3(256), 0, st, q, r, a, seg, P, fo);
}

template <typename T, int NV, bool HLLC, bool MIX>
int adj_rhs_nv(const AdjWork& w, const AdjArgs& a, const void* q, const void* rb, void* out,
               int mode, double alpha, double beta, const void* y, double gam, hipStream_t st) {
  const T* qs = static_cast<const T*>(q);
  const T* r = static_cast<const T*>(rb);
  T* P = static_cast<T*>(w.P);
  FoldOut<T> fo{static_cast<T*>(out), static_cast<const T*>(y), mode, 0, alpha, beta, gam};
  adj_lane_launch<T, NV, 0, HLLC, MIX>(qs, r, a, P, fo, st);
  // the march addresses each variable's plane with 32-bit byte offsets
  const bool planes_small = a.sv * (long long)sizeof(T) < (1LL << 31) &&
                            a.rv * (long long)sizeof(T) < (1LL << 31);
  const bool zfold = !MIX && fold_pays(a);
  if (zfold) {
    const long long n = (long long)(a.nx > 6 ? 6 : a.nx) * a.ny * a.nz;
    hipLaunchKernelGGL((k_adj_xmerge<T, NV>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       P, a);
  }
  bool marched = false;
  if constexpr (march_fits<T, NV>() && !MIX) {
    if (planes_small && march_pays(a)) {
      const MarchFold<T> none{nullptr, nullptr, 0, T(0), T(0), T(0)};
      const MarchFold<T> mf{static_cast<T*>(out), static_cast<const T*>(y), mode,
                            static_cast<T>(alpha), static_cast<T>(beta), static_cast<T>(gam)};
      if (a.d3) adj_march_launch<T, NV, 1, HLLC>(qs, r, a, P, none, st);
      adj_march_launch<T, NV, 2, HLLC>(qs, r, a, P, zfold ? mf : none, st);
      marched = true;
    }
  }
  if (!marched) {
    if (a.d3) adj_lane_launch<T, NV, 1, HLLC, MIX>(qs, r, a, P, fo, st);
    FoldOut<T> zf = fo;
    zf.fold = zfold ? 1 : 0;
    adj_lane_launch<T, NV, 2, HLLC, MIX>(qs, r, a, P, zf, st);
  }
  // falling condensates (mixture): the reverse of the sedimentation terms
  if constexpr (MIX) {
    if (a.sed.on) {
      const dim3 sgrid(a.ny * (a.nz + 2), (a.nx + 255) / 256);
      hipLaunchKernelGGL((k_adj_sediment<T, NV>), sgrid, dim3(256), 0, st, qs, r, a, P);
    }
  }
  // every row, or after a folding z march the rows it left
  const int ye = !a.d3 ? 0 : (a.ny > 6 ? 6 : a.ny);
  const int rows = zfold ? 6 * a.ny + (a.nz - 6) * ye : a.ny * a.nz;
  const dim3 fgrid(rows, (a.nx + 255) / 256);
  hipLaunchKernelGGL((k_adj_consfold<T, NV, MIX>), fgrid, dim3(256), 0, st, qs, P, r, a, fo,
                     zfold ? 1 : 0);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T, bool HLLC, bool MIX>
int adj_rhs_t(const AdjWork& w, const AdjArgs& a, const void* q, const void* rb, void* out,
              int mode, double alpha, double beta, const void* y, double gam, hipStream_t st) {
  int r = -1;
  switch (a.nvar) {
#define SNAP_ADJ_CASE(NVV)                                                      \
  case NVV:                                                                     \
    r = adj_rhs_nv<T, NVV, HLLC, MIX>(w, a, q, rb, out, mode, alpha, beta, y, gam, st); \
    break;
    case 5:   // the mixture needs tracers
      if constexpr (!MIX) r = adj_rhs_nv<T, 5, HLLC, false>(w, a, q, rb, out, mode, alpha, beta, y, gam, st);
      break;
    SNAP_ADJ_CASE(6)
    SNAP_ADJ_CASE(7)
    SNAP_ADJ_CASE(8)
    SNAP_ADJ_CASE(9)
    SNAP_ADJ_CASE(10)
    SNAP_ADJ_CASE(11)
    SNAP_ADJ_CASE(12)
    SNAP_ADJ_CASE(13)
#undef SNAP_ADJ_CASE
    default: r = -1;
  }
  return r;
}

}  // namespace snap
