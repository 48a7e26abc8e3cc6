// Fused right-hand-side / Runge-Kutta stage kernels.
//
// One launch evaluates the full right-hand side of Sec. 4 (eq. forward) for a
// block of cells and either stores it (rhs mode) or applies one stage of the
// TVD Runge-Kutta step of Sec. 4.3 (stage mode):
//     out = ca * Qn + cb * (Qs + dt * R(Qs)).
// Face states and fluxes never leave the chip: primitive variables of a plane
// of cells and the face values / fluxes of its two in-plane directions are
// staged through LDS, and (3-D) the vertical direction is marched with a
// per-thread register window of five levels.
//
// 3-D kernel: a workgroup owns a TX x TY column tile and a chunk of levels;
//   it walks up the chunk, and per level
//     (P) writes the primitives of the tile and its 3-cell x/y halo to LDS,
//     (R) reconstructs every cell of the tile plus one halo cell on each side
//         in x and in y (WENO5, both faces of the cell),
//     (L) evaluates LMARS at every x and y face of the tile,
//     (D) forms the divergence with the vertical flux difference that the
//         thread's own register window produced, adds gravity, and writes.
// 2-D (x-z) kernel: a workgroup owns a TX x TZ tile of the x-z plane and runs
//   the same P/R/L/D phases once, with z as the second in-plane axis.
#pragma once

#include "snap_device.h"

// Optional scheduling fence between per-variable reconstructions: keeps the
// compiler from interleaving all variables' WENO work (which raises register
// pressure and costs occupancy in double precision).
#ifdef SNAP_SCHED_FENCE
#define SNAP_VAR_FENCE() __builtin_amdgcn_sched_barrier(0)
#else
#define SNAP_VAR_FENCE() ((void)0)
#endif

namespace snap {

#ifndef SNAP_MAX_PASSES
#define SNAP_MAX_PASSES 8
#endif

struct StageArgs {
  const void* qs;   // padded state whose right-hand side is taken (ghosts filled)
  const void* qn;   // padded Q^n for the stage combination (may alias out); unused if ca == 0
  void* out;        // padded next state (stage mode) or interior rhs (rhs mode)
  int rhs_mode;     // 1: out = R (interior layout); 0: stage combination (padded layout)
  double ca, cb, dt;
  int nx, ny, nz;
  int gy;                  // 3 in 3-D, 0 in 2-D
  long long sy, sz, sv;    // padded strides (elements)
  long long ry, rz, rv;    // interior (rhs) strides
  int tiles_x, tiles_y, nchunk, tz;
  // 3-D only. pass_map = 0: block -> (tile, chunk) through the XCD-aware
  // order, chunk kc covering levels kc*tz .. min(kc*tz + tz, nz) - 1.
  // pass_map = 1 (a launch of exactly one workgroup per compute unit per
  // chunk, all co-resident): chunk kc = blockIdx / tiles, i.e. the dispatch
  // pass, covering levels kb[kc] .. kb[kc+1] - 1; consecutive blocks of a
  // pass go to different XCDs, and the tiles one XCD receives are adjacent.
  int pass_map;
  int kb[SNAP_MAX_PASSES + 1];
  double dxi, dyi, dzi;    // 1 / spacing
  double gamma, gm1, inv_gm1, grav, eps;
  int linear;
  const double* rbar_c;  // nz + 6
  const double* pbar_c;
  const double* rbar_f;  // nz + 1
  const double* pbar_f;
  Mixture mix;           // mixture equation of state (kernels instantiated with MIX)
  Sediment sed;          // sedimentation (3-D: SED kernel instances; 2-D: a kernel of its own)
  // Time step from the device: when smax is set, dt = cfl / (the maximum
  // signal speed whose IEEE bits smax holds, written by the reduction kernel
  // earlier on the stream) and a.dt is unused. When dt_out is set, block 0
  // stores the dt it used there.
  const unsigned long long* smax;
  double cfl;
  double* dt_out;
  // GF_ON: the kernel reads each ghost cell it needs (the halo of its tile,
  // 3-D: also the window levels below 0 and above nz - 1) from the interior
  // cell the ghost fill copies (ghost_src, momentum normal to a reflecting wall
  // negated), so no fill has to precede it; GF_RX / GF_RY / GF_RZ: that axis
  // reflects (else it is periodic).
  int ghost;
  // Next step's time step (kernels that read ghosts in place):
  // with smax_out set, the kernel also reduces the maximum signal speed of its
  // output (the quantity and the arithmetic of the CFL reduction kernel, so the
  // dt formed from it is the same) into *smax_out with atomicMax; with
  // smax_zero set, block 0 clears *smax_zero (a slot that a later launch of
  // the step fills).
  unsigned long long* smax_out;
  unsigned long long* smax_zero;
  // With the time step from the device (smax set): block 0 stores 1 here if
  // that time step is not finite and positive, i.e. the reduced state had a
  // non-finite or non-positive density or pressure somewhere.
  unsigned long long* state_flag;
  // 3-D only: no more workgroups than Stage3DShape's LOW instances run at once
  int low;
  int half;   // 3-D only: the half tile where the kernel has one (Tile3For)
  // 1: q holds rho - rhobar_k and E - pbar_k / (gamma - 1) (perturbation
  // storage, passive tracers only); 0: the full conserved state.
  int pert;
};

// References of level k for the conversion of the stored state: ra is added
// to the stored density to give rho, rs and ps are subtracted from rho and p
// to give rho' and p'; pe is added to (gamma - 1)(E_stored - K) to give p.
struct LevelRef {
  double ra, rs, ps, pe;
};
__device__ __forceinline__ LevelRef level_ref(int pert, double rbar, double pbar) {
  LevelRef r;
  r.ra = pert ? rbar : 0.0;
  r.rs = pert ? 0.0 : rbar;
  r.ps = pert ? 0.0 : pbar;
  r.pe = pert ? pbar : 0.0;
  return r;
}
enum : int { GF_ON = 1, GF_RX = 2, GF_RY = 4, GF_RZ = 8 };

// The 3-D stage kernels that can read ghosts in place (GF_ON): those without
// tracers. The others keep the fill. Some have the registers for it by now (as
// compiled, with the fill and without: mixture in single precision with four
// tracers 237, 239, with six 243, 245, with rain 227, 229; passive with two 160,
// 167, with four 165, 167), while others would spill more (passive with three and
// five in single precision, with four in double); none has been timed without it.
// (The 2-D kernels all can.)
constexpr bool ghosts_in_place(int ntracer) { return ntracer == 0; }

// 3-D kernels that can reduce the signal speed of their output (smax_out).
// (The 2-D kernels of the passive gas all can.)
template <typename T, int NT>
constexpr bool fused_speed() { return ghosts_in_place(NT); }


// The stage's time step (uniform over the launch).
__device__ __forceinline__ double stage_dt(const StageArgs& a) {
  if (a.smax == nullptr) return a.dt;
  return a.cfl / __longlong_as_double(static_cast<long long>(*a.smax));
}

// Block 0 records the time step of the launch where the caller asked for it,
// and raises the state flag if that time step is not finite and positive.
__device__ __forceinline__ void store_stage_dt(const StageArgs& a, double dt) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    if (a.dt_out != nullptr) *a.dt_out = dt;
    if (a.state_flag != nullptr && !(dt > 0.0 && dt <= 1.79769313486231570815e308))
      *a.state_flag = 1ULL;
  }
}

template <typename T>
__device__ __forceinline__ double to_d(T v) {
  return static_cast<double>(v);
}

// Load the NV conserved values of padded element offset `off` and convert them
// to primitives with the level references (rb, pb).
// Conserved -> primitive with the kernel's equation of state: passive tracers,
// or the mixture (MIX) with coefficients mx.
template <int NV, bool MIX>
__device__ __forceinline__ void cons_to_prim_eos(const double (&c)[NV], double ra, double rb,
                                                 double pb, double gm1, const Mixture& mx,
                                                 double (&x)[NV]) {
  if constexpr (MIX)
    cons_to_prim_mix<NV>(c, rb, pb, gm1, mx, x);   // full storage only (ra = 0)
  else
    cons_to_prim<NV>(c, ra, rb, pb, gm1, x);
}

// Single-precision storage with passive tracers: the velocities, kinetic
// energy and tracer fractions in single precision, where nothing cancels, and
// only the two differences that do, rho - rhobar and (gamma - 1)(E - K) -
// pbar, in double precision (one rounding each, then to single precision).
// The reciprocal of rho is the hardware estimate (1 ulp).
template <int NV>
__device__ __forceinline__ void cons_to_prim_sp(const float (&c)[NV], double ra, double rb,
                                                double pb, double gm1, float (&x)[NV]) {
  const float inv = __builtin_amdgcn_rcpf(c[0] + static_cast<float>(ra));
  const float u = c[1] * inv, v = c[2] * inv, w = c[3] * inv;
  const float K = 0.5f * fmaf(c[3], w, fmaf(c[2], v, c[1] * u));
  x[0] = static_cast<float>(static_cast<double>(c[0]) - rb);
  x[1] = u;
  x[2] = v;
  x[3] = w;
  x[4] = static_cast<float>(fma(gm1, static_cast<double>(c[4]) - static_cast<double>(K), -pb));
#pragma unroll
  for (int t = 5; t < NV; ++t) x[t] = c[t] * inv;
}

template <typename T, int NV, bool MIX = false>
__device__ __forceinline__ void load_prim(const T* __restrict__ q, long long off, long long sv,
                                          const LevelRef& lr, double gm1, const Mixture& mx,
                                          T (&x)[NV]) {
  if constexpr (sizeof(T) == 4 && !MIX) {
    float c[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) c[v] = q[off + v * sv];
    cons_to_prim_sp<NV>(c, lr.ra, lr.rs, lr.ps, gm1, x);
  } else {
    double c[NV], xd[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) c[v] = to_d(q[off + v * sv]);
    cons_to_prim_eos<NV, MIX>(c, lr.ra, lr.rs, lr.ps, gm1, mx, xd);
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v] = static_cast<T>(xd[v]);
  }
}

// passive tracers
template <typename T, int NV>
__device__ __forceinline__ void load_prim(const T* __restrict__ q, long long off, long long sv,
                                          const LevelRef& lr, double gm1, T (&x)[NV]) {
  if constexpr (sizeof(T) == 4) {
    float c[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) c[v] = q[off + v * sv];
    cons_to_prim_sp<NV>(c, lr.ra, lr.rs, lr.ps, gm1, x);
  } else {
    double c[NV], xd[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) c[v] = to_d(q[off + v * sv]);
    cons_to_prim<NV>(c, lr.ra, lr.rs, lr.ps, gm1, xd);
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v] = static_cast<T>(xd[v]);
  }
}

// The factor by which riemann_flux scales the face flux: the passive LMARS
// returns twice the flux (lmars_flux), the others the flux itself. The flux
// differences are multiplied by the inverse spacing over this factor (a power
// of two, so the scaled spacing is exact).
template <bool MIX, bool HLLC>
constexpr double flux_scale() {
  return (!MIX && !HLLC) ? 2.0 : 1.0;
}

// Face flux of the kernel's Riemann solver (LMARS, or HLLC with passive
// tracers) and equation of state, times flux_scale<MIX, HLLC>(). left: the
// upwind side (not set under the mixture).
template <typename T, int NV, bool MIX, bool HLLC>
__device__ __forceinline__ void riemann_flux(const T (&xl)[NV], const T (&xr)[NV], int nrm,
                                             T rref, T pref, T gamma, T inv_gm1, T gm1,
                                             const Mixture& mx, T (&f)[NV], bool& left) {
  static_assert(!(MIX && HLLC), "HLLC takes passive tracers");
  if constexpr (HLLC)
    hllc_flux<T, NV>(xl, xr, nrm, rref, pref, gamma, inv_gm1, f, left);
  else if constexpr (MIX)
    lmars_flux_mix<T, NV>(xl, xr, nrm, rref, pref, gm1, mx, f);
  else
    lmars_flux<T, NV>(xl, xr, nrm, rref, pref, gamma, inv_gm1, f, left);
}

// Variables whose in-plane face states are reconstructed on both sides: all of
// them under the mixture, whose flux needs both sides' fractions; the five
// dynamic ones with passive tracers, whose flux is the mass flux times the
// upwind side's fraction (phase L reconstructs that one value per face). In
// 3-D and single precision one tracer keeps both sides: it gains no wave, and
// saves the barrier before the last fluxes (686 -> 678 us per step of
// 256 x 192 x 96).
template <typename T, int NV, bool MIX, bool D3>
constexpr int two_sided() {
  return MIX || (D3 && sizeof(T) == 4 && NV == 6) ? NV : 5;
}

// The 3-D kernels that reconstruct the tangential velocities, too, on the upwind
// side of a face only: LMARS with passive tracers in double precision, unpacked
// item addresses. The interface velocity takes rho', the normal velocity and p'
// of both sides, so those three are reconstructed per cell, and the two others
// per face once its side is known: two of five two-sided reconstructions become
// one-sided, for five more reads of the plane (registers selected in z) per
// face. 256 x 256 x 128, four steps: 6365 -> 6156 us; 75 x 60 x 40 129 -> 126; with
// tracers, where not packed, within 0 to 1.5 % on 256 x 192 x 96. Not in single
// precision: the dry instance takes 171 registers under the scheduling of
// its file, which is two waves per SIMD instead of three (2301 -> 2817 us, 250 x 187
// x 101, four steps). Held to three waves it compiles to 161 without spills, a form
// that has not been timed. Not in the 2-D kernels: one domain of 256 x 256, where
// every wave is waited for, took 718 -> 735 us in twenty steps, the batch of 64 in
// single precision 1.1 % longer (80 -> 82 registers, six waves to five, in the
// kernel of that time). HLLC and the mixture keep both sides, too; neither was tried.
template <typename T, int ND, bool MIX, bool HLLC, bool PACK>
constexpr bool upwind_tangential() {
  return sizeof(T) == 8 && ND == 5 && !MIX && !HLLC && !PACK;
}

// Output of one interior cell: either R itself or the stage combination (the
// new state is left in R).
template <typename T, int NV>
__device__ __forceinline__ void write_cell(const StageArgs& a, const T* __restrict__ qs,
                                           long long poff, long long roff, T (&R)[NV]) {
  if (a.rhs_mode) {
    T* __restrict__ o = static_cast<T*>(a.out);
#pragma unroll
    for (int v = 0; v < NV; ++v) o[roff + v * a.rv] = R[v];
    return;
  }
  const T dt = static_cast<T>(stage_dt(a)), ca = static_cast<T>(a.ca), cb = static_cast<T>(a.cb);
  T* o = static_cast<T*>(a.out);
  const T* qn = static_cast<const T*>(a.qn);
  if (a.ca != 0.0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const T t = qs[poff + v * a.sv] + dt * R[v];
      R[v] = ca * qn[poff + v * a.sv] + cb * t;
      o[poff + v * a.sv] = R[v];
    }
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const T t = qs[poff + v * a.sv] + dt * R[v];
      R[v] = cb * t;
      o[poff + v * a.sv] = R[v];
    }
  }
}

// Signal speed sum_d (|u_d| + c) / dx_d (IEEE bits) of one 2-D cell's new state
// q under the passive gas, in the CFL kernel's order and operations (no
// contraction); level references rbo, pbo are added back (perturbation storage).
template <typename T, int NV>
__device__ __forceinline__ unsigned long long speed_bits_2d(const StageArgs& a, const T (&q)[NV],
                                                            double rbo, double pbo) {
#pragma clang fp contract(off)
  const double rho = static_cast<double>(q[0]) + rbo, mx = q[1], my = q[2], mz = q[3];
  const double E = q[4];
  const double inv = 1.0 / rho;
  const double u = mx * inv, v = my * inv, w = mz * inv;
  const double K = 0.5 * ((mx * u + my * v) + mz * w);
  const double p = a.gm1 * (E - K) + pbo;
  const double cs = sqrt(a.gamma * p / rho);
  double sp = (fabs(u) + cs) * a.dxi;
  sp = sp + (fabs(w) + cs) * a.dzi;
  if (!(rho > 0.0) || !(p > 0.0)) sp = __builtin_nan("");
  return (unsigned long long)__double_as_longlong(sp);
}

// ---------------------------------------------------------------------------
// LDS plane shared by both kernels: primitives with a 3-cell halo and, per
// in-plane axis, one value per face (first the left face state, then, after
// the LMARS phase, the flux). The right face state of each face stays in the
// registers of the thread that reconstructed it; the items beyond the RREG
// rounds, reconstructed one (cell, variable) pair at a time, park it in QS.
//
// Work items of the reconstruction and LMARS phases (one list; within the
// RREG rounds the same thread takes an item in both):
//   x items: cells ii = -1 .. TX along each row jj = 0 .. TY-1;
//   second-axis items: cells jj = -1 .. TY along each column ii = 0 .. TX-1.
// Item (cell c) writes the left state of face c+1 and keeps the right state
// of face c; in the LMARS phase it evaluates face c (for c >= 0).
// ---------------------------------------------------------------------------
template <int TX, int TY>
struct PlaneItems {
  static constexpr int NTHR = TX * TY;
  static constexpr int NRX = (TX + 2) * TY;
  static constexpr int NRS = TX * (TY + 2);
  static constexpr int NR = NRX + NRS;
  static constexpr int ROUNDS = (NR + NTHR - 1) / NTHR;
#ifndef SNAP_RREG
#define SNAP_RREG 2
#endif
  static constexpr int RREG = ROUNDS < SNAP_RREG ? ROUNDS : SNAP_RREG;
  static constexpr int NSPILL = NR - RREG * NTHR > 0 ? NR - RREG * NTHR : 1;
};

template <typename T, int NV, int TX, int TY>
struct Plane {
  T P[NV][TY + 6][TX + 6];
  T FX[NV][TY][TX + 1];
  T FY[NV][TY + 1][TX];
  T QS[PlaneItems<TX, TY>::NSPILL][NV];
};

// Thread index used for item lists: the waves of a workgroup take turns at
// the rounds that not every wave gets (e.g. 576 items over 4 waves), rotated
// by block so that co-resident workgroups put the extra round on different
// SIMDs.
template <int NTHR>
__device__ __forceinline__ int item_thread() {
  if constexpr (NTHR % 64 == 0 && NTHR >= 128)
    return (threadIdx.x + 64 * (blockIdx.x % (NTHR / 64))) % NTHR;
  else
    return threadIdx.x;
}

// Decode item `it` into (axis, ii, jj); returns false if the cell lies outside
// the active w x h part of a ragged tile.
template <int TX, int TY>
__device__ __forceinline__ bool plane_item(int it, int w, int h, bool& xaxis, int& ii, int& jj) {
  using I = PlaneItems<TX, TY>;
  if (it < I::NRX) {
    xaxis = true;
    ii = it % (TX + 2) - 1;
    jj = it / (TX + 2);
    return ii <= w && jj < h;
  }
  const int r = it - I::NRX;
  xaxis = false;
  ii = r % TX;
  jj = r / TX - 1;
  return ii < w && jj <= h;
}

// Phase R: WENO5 of every item cell; left states to LDS, right states kept
// (in registers for the RREG rounds, in QS for the items beyond them).
// An x item reads a row of the plane (stride 1), a second-axis item a column
// (stride TX + 6), so one code path serves both. With RPF the five stencil
// values of variable v + 1 are read from LDS before variable v is
// reconstructed: the LDS latency then overlaps that reconstruction instead of
// stalling the wave at the start of every variable. RPF is off where those
// five live values would push the kernel past an occupancy step.
template <typename T, int NV>
constexpr bool reconstruct_prefetch() {
  // single precision with 1 or 8 tracers: 167 -> 178 and 256 -> 257 registers
  return !(sizeof(T) == 4 && (NV == 6 || NV == 13));
}

// SPLIT: the items beyond the RREG rounds (64 of the 576 of a 16 x 16 tile)
// are split by variable, one (cell, variable) pair per thread and pass, so
// that every wave takes a share instead of one wave reconstructing all their
// variables while the others wait at the barrier. Without SPLIT they are a
// last round of whole items, which needs fewer registers: the callers keep
// that form where the split would cost a wave per SIMD or add spills.
// ND: the variables reconstructed (the first ND of NV, two_sided).
template <typename T, int NV, int ND, int TX, int TY, bool SPLIT = true>
__device__ __forceinline__ void phase_reconstruct(Plane<T, NV, TX, TY>& S, int w, int h, T eps,
                                                  bool linear,
                                                  T (&QP)[PlaneItems<TX, TY>::RREG][ND]) {
  using I = PlaneItems<TX, TY>;
  constexpr bool RPF = reconstruct_prefetch<T, NV>();
  constexpr int PV = (TY + 6) * (TX + 6);   // plane stride between variables
  constexpr int FXV = TY * (TX + 1), FYV = (TY + 1) * TX;
  constexpr int NSP = I::NR - I::RREG * I::NTHR;   // cells left after the RREG rounds
  if constexpr (SPLIT && NSP > 0) {
    constexpr int NSUB = NSP * ND;
    const int t0 = item_thread<I::NTHR>();
#pragma unroll
    for (int m = 0; m < (NSUB + I::NTHR - 1) / I::NTHR; ++m) {
      const int sub = t0 + m * I::NTHR;
      const int v = sub / NSP, c = sub - v * NSP;
      const int it = I::RREG * I::NTHR + c;
      bool xa;
      int ii, jj;
      if (sub < NSUB && plane_item<TX, TY>(it, w, h, xa, ii, jj)) {
        const int st = xa ? 1 : TX + 6;
        const T* src = (xa ? &S.P[0][jj + 3][ii + 1] : &S.P[0][jj + 1][ii + 3]) + v * PV;
        T cur[5];
#pragma unroll
        for (int mm = 0; mm < 5; ++mm) cur[mm] = src[mm * st];
        T qm, qp;
        weno5_cell<T>(cur[0], cur[1], cur[2], cur[3], cur[4], eps, linear, qm, qp);
        if (xa ? ii < w : jj < h) {
          if (xa)
            S.FX[v][jj][ii + 1] = qm;
          else
            S.FY[v][jj + 1][ii] = qm;
        }
        S.QS[c][v] = qp;
      }
    }
  }
  constexpr int NROUND = SPLIT ? I::RREG : I::ROUNDS;
#pragma unroll
  for (int r = 0; r < NROUND; ++r) {
    const int it = item_thread<I::NTHR>() + r * I::NTHR;
    bool xa;
    int ii, jj;
    if (it < I::NR && plane_item<TX, TY>(it, w, h, xa, ii, jj)) {
      const int st = xa ? 1 : TX + 6;
      const T* src = xa ? &S.P[0][jj + 3][ii + 1] : &S.P[0][jj + 1][ii + 3];
      T* dst = xa ? &S.FX[0][jj][ii + 1] : &S.FY[0][jj + 1][ii];
      const int dv = xa ? FXV : FYV;
      const bool put = xa ? ii < w : jj < h;
      T qp[ND];
      T cur[5];
      if constexpr (RPF) {
#pragma unroll
        for (int m = 0; m < 5; ++m) cur[m] = src[m * st];
      }
#pragma unroll
      for (int v = 0; v < ND; ++v) {
        T nxt[5];
        if constexpr (RPF) {
          if (v + 1 < ND) {
#pragma unroll
            for (int m = 0; m < 5; ++m) nxt[m] = src[(v + 1) * PV + m * st];
          }
        } else {
#pragma unroll
          for (int m = 0; m < 5; ++m) cur[m] = src[v * PV + m * st];
        }
        T qm;
        weno5_cell<T>(cur[0], cur[1], cur[2], cur[3], cur[4], eps, linear, qm, qp[v]);
        if (put) dst[v * dv] = qm;
        SNAP_VAR_FENCE();
        if constexpr (RPF) {
          if (v + 1 < ND) {
#pragma unroll
            for (int m = 0; m < 5; ++m) cur[m] = nxt[m];
          }
        }
      }
#pragma unroll
      for (int v = 0; v < ND; ++v) {
        if (r < I::RREG)
          QP[r < I::RREG ? r : 0][v] = qp[v];
        else
          S.QS[it - I::RREG * I::NTHR][v] = qp[v];
      }
    }
  }
}

// The upwind value of one variable at a face between cells c-1 and c of a line
// of the plane: cells c-3 .. c+1 in order from the left side, c+2 .. c-2 from
// the right, so the side only picks the five addresses (lo: cell c-3, stride st).
template <typename T>
struct UpwindStencil {
  const T* p[5];
  __device__ __forceinline__ UpwindStencil(const T* lo, int st, bool left) {
    const int step = left ? st : -st;
    p[0] = lo + (left ? 0 : 5 * st);
#pragma unroll
    for (int m = 1; m < 5; ++m) p[m] = p[m - 1] + step;
  }
  __device__ __forceinline__ T face(int off, T eps, bool linear) const {
    return weno5_face<T>(p[0][off], p[1][off], p[2][off], p[3][off], p[4][off], eps, linear);
  }
};

// Phase L: the flux at every face of the tile, by the item that holds its right
// state. x faces use the reference of their row (xref); second-axis faces use
// sref(face index). SNRM is the index of the second axis's velocity; the flux
// is called in two branches, each with a constant normal, so that picking the
// normal velocity and adding p* need no selects over the velocity components.
// Passive tracers: once a face's flux is known, so is its upwind side, and the
// item reconstructs each tracer there from the plane (UpwindStencil) and
// multiplies by the mass flux. Against the two-sided reconstruction of every cell
// it saves a fifth of the WENO instructions, the face states' way through LDS and
// the right states' registers.
template <typename T, int NV, int ND, int TX, int TY, int SNRM, bool MIX, bool HLLC,
          typename XRef, typename SRef>
__device__ __forceinline__ void phase_lmars(Plane<T, NV, TX, TY>& S, int w, int h, T eps,
                                            bool linear, T gamma, T inv_gm1, T gm1,
                                            const Mixture& mx, XRef xref, SRef sref,
                                            const T (&QP)[PlaneItems<TX, TY>::RREG][ND]) {
  using I = PlaneItems<TX, TY>;
#pragma unroll
  for (int r = 0; r < I::ROUNDS; ++r) {
    const int it = item_thread<I::NTHR>() + r * I::NTHR;
    bool xa;
    int ii, jj;
    if (it < I::NR && plane_item<TX, TY>(it, w, h, xa, ii, jj) && ii >= 0 && jj >= 0) {
      T xl[ND], xr[ND], f[ND];
#pragma unroll
      for (int v = 0; v < ND; ++v) {
        xr[v] = r < I::RREG ? QP[r < I::RREG ? r : 0][v] : S.QS[it - I::RREG * I::NTHR][v];
        xl[v] = xa ? S.FX[v][jj][ii] : S.FY[v][jj][ii];
      }
      T rr, pr;
      bool left = false;
      // 2-D: the face's references are loaded ahead of the branch, both axes in one
      // go (64 x 64, double precision, 20 steps: 547 -> 540 us; 256 x 256 724 ->
      // 708). Not HLLC, whose instances of other tile shapes then contract
      // differently: 1.8e-6 apart in single precision. Not the mixture, for which it
      // was not measured
      constexpr bool REF = SNRM == 3 && !HLLC && !MIX;
      if constexpr (REF) {
        if (xa)
          xref(jj, rr, pr);
        else
          sref(jj, rr, pr);
      }
      if (xa) {
        if constexpr (!REF) xref(jj, rr, pr);
        riemann_flux<T, ND, MIX, HLLC>(xl, xr, 1, rr, pr, gamma, inv_gm1, gm1, mx, f, left);
      } else {
        if constexpr (!REF) sref(jj, rr, pr);
        riemann_flux<T, ND, MIX, HLLC>(xl, xr, SNRM, rr, pr, gamma, inv_gm1, gm1, mx, f, left);
      }
#pragma unroll
      for (int v = 0; v < ND; ++v) {
        if (xa)
          S.FX[v][jj][ii] = f[v];
        else
          S.FY[v][jj][ii] = f[v];
      }
      if (ND < NV && r < I::RREG) {
        T* dst = xa ? &S.FX[ND][jj][ii] : &S.FY[ND][jj][ii];
        const int dv = xa ? TY * (TX + 1) : (TY + 1) * TX;
        const UpwindStencil<T> u(xa ? &S.P[0][jj + 3][ii] : &S.P[0][jj][ii + 3], xa ? 1 : TX + 6,
                                 left);
#pragma unroll
        for (int v = ND; v < NV; ++v) {
          dst[(v - ND) * dv] = f[0] * u.face(v * (TY + 6) * (TX + 6), eps, linear);
          SNAP_VAR_FENCE();
        }
      }
      if (HLLC && ND < NV && r >= I::RREG)
        S.QS[it - I::RREG * I::NTHR][0] = left ? T(1) : T(0);   // for phase_tracer_rest
    }
  }
}

// Phases R and L of the kernels that reconstruct the tangential velocities on
// the upwind side (upwind_tangential): three variables per cell item, then at a
// face the two tangential velocities and the tracers from the plane.
template <typename T, int NV, int TX, int TY, int SNRM>
__device__ __forceinline__ void phase_reconstruct_sides(Plane<T, NV, TX, TY>& S, int w, int h,
                                                        T eps, bool linear,
                                                        T (&QP)[PlaneItems<TX, TY>::RREG][3]) {
  using I = PlaneItems<TX, TY>;
  constexpr int PV = (TY + 6) * (TX + 6);   // plane stride between variables
  constexpr int FXV = TY * (TX + 1), FYV = (TY + 1) * TX;
  constexpr int NSP = I::NR - I::RREG * I::NTHR;   // cells left after the RREG rounds
  // plane of the m-th reconstructed variable: rho', the normal velocity, p'
  auto plane = [](int m, bool xa) { return m == 0 ? 0 : (m == 1 ? (xa ? 1 : SNRM) : 4); };
  if constexpr (NSP > 0) {
    constexpr int NSUB = NSP * 3;
    const int t0 = item_thread<I::NTHR>();
#pragma unroll
    for (int m = 0; m < (NSUB + I::NTHR - 1) / I::NTHR; ++m) {
      const int sub = t0 + m * I::NTHR;
      const int v = sub / NSP, c = sub - v * NSP;
      const int it = I::RREG * I::NTHR + c;
      bool xa;
      int ii, jj;
      if (sub < NSUB && plane_item<TX, TY>(it, w, h, xa, ii, jj)) {
        const int st = xa ? 1 : TX + 6;
        const T* src = (xa ? &S.P[0][jj + 3][ii + 1] : &S.P[0][jj + 1][ii + 3]) + plane(v, xa) * PV;
        T cur[5];
#pragma unroll
        for (int mm = 0; mm < 5; ++mm) cur[mm] = src[mm * st];
        T qm, qp;
        weno5_cell<T>(cur[0], cur[1], cur[2], cur[3], cur[4], eps, linear, qm, qp);
        if (xa ? ii < w : jj < h) {
          if (xa)
            S.FX[v][jj][ii + 1] = qm;
          else
            S.FY[v][jj + 1][ii] = qm;
        }
        S.QS[c][v] = qp;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < I::RREG; ++r) {
    const int it = item_thread<I::NTHR>() + r * I::NTHR;
    bool xa;
    int ii, jj;
    if (it < I::NR && plane_item<TX, TY>(it, w, h, xa, ii, jj)) {
      const int st = xa ? 1 : TX + 6;
      const T* src = xa ? &S.P[0][jj + 3][ii + 1] : &S.P[0][jj + 1][ii + 3];
      T* dst = xa ? &S.FX[0][jj][ii + 1] : &S.FY[0][jj + 1][ii];
      const int dv = xa ? FXV : FYV;
      const bool put = xa ? ii < w : jj < h;
      T qp[3];
      T cur[5];
#pragma unroll
      for (int m = 0; m < 5; ++m) cur[m] = src[m * st];
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        T nxt[5];
        if (v + 1 < 3) {
#pragma unroll
          for (int m = 0; m < 5; ++m) nxt[m] = src[plane(v + 1, xa) * PV + m * st];
        }
        T qm;
        weno5_cell<T>(cur[0], cur[1], cur[2], cur[3], cur[4], eps, linear, qm, qp[v]);
        if (put) dst[v * dv] = qm;
        SNAP_VAR_FENCE();
        if (v + 1 < 3) {
#pragma unroll
          for (int m = 0; m < 5; ++m) cur[m] = nxt[m];
        }
      }
#pragma unroll
      for (int v = 0; v < 3; ++v) QP[r][v] = qp[v];
    }
  }
}

template <typename T, int NV, int TX, int TY, int SNRM, typename XRef, typename SRef>
__device__ __forceinline__ void phase_lmars_sides(Plane<T, NV, TX, TY>& S, int w, int h, T eps,
                                                  bool linear, T gamma, T inv_gm1, XRef xref,
                                                  SRef sref,
                                                  const T (&QP)[PlaneItems<TX, TY>::RREG][3]) {
  using I = PlaneItems<TX, TY>;
#pragma unroll
  for (int r = 0; r < I::ROUNDS; ++r) {
    const int it = item_thread<I::NTHR>() + r * I::NTHR;
    bool xa;
    int ii, jj;
    if (it < I::NR && plane_item<TX, TY>(it, w, h, xa, ii, jj) && ii >= 0 && jj >= 0) {
      T xl[3], xr[3];
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        xr[v] = r < I::RREG ? QP[r < I::RREG ? r : 0][v] : S.QS[it - I::RREG * I::NTHR][v];
        xl[v] = xa ? S.FX[v][jj][ii] : S.FY[v][jj][ii];
      }
      T rr, pr;
      if (xa)
        xref(jj, rr, pr);
      else
        sref(jj, rr, pr);
      constexpr int PV = (TY + 6) * (TX + 6);
      T* dst = xa ? &S.FX[0][jj][ii] : &S.FY[0][jj][ii];
      const int dv = xa ? TY * (TX + 1) : (TY + 1) * TX;
      const LmarsFace<T> o = lmars_side<T>(xl, xr, rr, pr, gamma);
      const UpwindStencil<T> u(xa ? &S.P[0][jj + 3][ii] : &S.P[0][jj][ii + 3], xa ? 1 : TX + 6,
                               o.left);
      const int n = xa ? 1 : SNRM, t1 = xa ? 2 : 1, t2 = xa ? 3 : 5 - SNRM;
      const T q1 = u.face(t1 * PV, eps, linear);
      SNAP_VAR_FENCE();
      const T q2 = u.face(t2 * PV, eps, linear);
      T f[5];
      lmars_rest<T>(o, q1, q2, gamma, inv_gm1, f);
      dst[0] = f[0];
      dst[n * dv] = f[1];
      dst[t1 * dv] = f[2];
      dst[t2 * dv] = f[3];
      dst[4 * dv] = f[4];
      if (NV > 5 && r < I::RREG) {
#pragma unroll
        for (int v = 5; v < NV; ++v) {
          dst[v * dv] = f[0] * u.face(v * PV, eps, linear);
          SNAP_VAR_FENCE();
        }
      }
    }
  }
}

// The tracer fluxes of the faces beyond the RREG rounds (64 of the 544 of a
// 16 x 16 tile), one (face, tracer) pair per thread and pass so that every wave
// takes a share (a barrier after phase_lmars). The upwind side is the one the
// flux took, or two tiles that share a face could carry different values through
// it: the sign of the mass flux under LMARS, which forms it as a product with
// the interface velocity; under HLLC, where it is a sum that rounding can leave
// with either sign in still air, the side phase_lmars left in QS.
template <typename T, int NV, int ND, int TX, int TY, bool HLLC>
__device__ __forceinline__ void phase_tracer_rest(Plane<T, NV, TX, TY>& S, int w, int h, T eps,
                                                  bool linear) {
  using I = PlaneItems<TX, TY>;
  constexpr int NSP = I::NR - I::RREG * I::NTHR;
  if constexpr (ND < NV && NSP > 0) {
    constexpr int NSUB = NSP * (NV - ND);
    const int t0 = item_thread<I::NTHR>();
#pragma unroll
    for (int m = 0; m < (NSUB + I::NTHR - 1) / I::NTHR; ++m) {
      const int sub = t0 + m * I::NTHR;
      const int v = ND + sub / NSP;
      bool xa;
      int ii, jj;
      if (sub < NSUB &&
          plane_item<TX, TY>(I::RREG * I::NTHR + sub % NSP, w, h, xa, ii, jj) && ii >= 0 &&
          jj >= 0) {
        const T f0 = xa ? S.FX[0][jj][ii] : S.FY[0][jj][ii];
        const bool left = HLLC ? S.QS[sub % NSP][0] != T(0) : f0 > T(0);
        const UpwindStencil<T> u(xa ? &S.P[0][jj + 3][ii] : &S.P[0][jj][ii + 3], xa ? 1 : TX + 6,
                                 left);
        const T q = u.face(v * (TY + 6) * (TX + 6), eps, linear);
        (xa ? S.FX[v][jj][ii] : S.FY[v][jj][ii]) = f0 * q;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same phases for square tiles with the items' addresses packed, for the
// 3-D kernels whose registers decide how many waves a SIMD holds. The addresses
// of an item follow from its thread alone, so the compiler forms them before
// the level loop and keeps every one (plane and face offsets per round and
// phase) in a register of its own: 16 to 20 of them. Here an item is one word
// per round, unpacked on every level (ItemCodes::get hides it from the
// compiler's hoisting), and x and second-axis faces share one variable stride
// (TX == TY), so that one offset serves both.
// On 256 x 192 x 96 a double-precision step with two tracers then fits two waves
// per SIMD: 1980 -> 1376 us; without tracers, where no wave is won, unpacking
// costs 3.5 % (567 -> 585 us, single precision), so those kernels keep the
// unpacked phases.
// ---------------------------------------------------------------------------
template <int NV, int TX, int TY>
struct ItemCodes {
  using I = PlaneItems<TX, TY>;
  static constexpr int NSP = I::NR - I::RREG * I::NTHR;   // items beyond the rounds
  static constexpr int PV = (TY + 6) * (TX + 6), DV = TY * (TX + 1), ROW = TX + 6;
  static_assert(TX == TY && NSP > 0 && I::NTHR % NSP == 0 && PV <= 1024 && (NV + 1) * DV <= 4096,
                "square tiles");
  enum : unsigned { XA = 1u << 22, PUT = 1u << 23, VALID = 1u << 24, FACE = 1u << 25 };
  unsigned c[I::RREG + 1];   // the rounds' items, then the item beyond them (by thread % NSP)

  __device__ __forceinline__ ItemCodes(int w, int h) {
    const int t0 = item_thread<I::NTHR>();
#pragma unroll
    for (int r = 0; r <= I::RREG; ++r) {
      bool xa;
      int ii, jj;
      const bool ok = plane_item<TX, TY>(r * I::NTHR + (r < I::RREG ? t0 : t0 % NSP), w, h, xa, ii, jj);
      const int src = xa ? (jj + 3) * ROW + ii + 1 : (jj + 1) * ROW + ii + 3;
      const int dst = xa ? jj * (TX + 1) + ii + 1 : NV * DV + (jj + 1) * TX + ii;
      c[r] = !ok ? 0u
                 : (unsigned)src | (unsigned)dst << 10 | (xa ? XA : 0u) | VALID |
                       ((xa ? ii < w : jj < h) ? PUT : 0u) | (ii >= 0 && jj >= 0 ? FACE : 0u);
    }
  }
  __device__ __forceinline__ unsigned get(int r) const {
    unsigned x = c[r];
    asm volatile("" : "+v"(x));
    return x;
  }
  // offsets of an item: its stencil (cell c-2) in the plane, the face c+1, the
  // distance of two cells and of two faces of its line
  static __device__ __forceinline__ int src(unsigned x) { return (int)(x & 1023u); }
  static __device__ __forceinline__ int dst(unsigned x) { return (int)((x >> 10) & 4095u); }
  static __device__ __forceinline__ int cell(unsigned x) { return (x & XA) ? 1 : ROW; }
  static __device__ __forceinline__ int face(unsigned x) { return (x & XA) ? 1 : TX; }
};

// Phase R (as phase_reconstruct with SPLIT).
template <typename T, int NV, int ND, int TX, int TY>
__device__ __forceinline__ void packed_reconstruct(Plane<T, NV, TX, TY>& S,
                                                   const ItemCodes<NV, TX, TY>& IC, T eps,
                                                   bool linear,
                                                   T (&QP)[PlaneItems<TX, TY>::RREG][ND]) {
  using C = ItemCodes<NV, TX, TY>;
  using I = PlaneItems<TX, TY>;
  constexpr bool RPF = reconstruct_prefetch<T, NV>();
  T* base = &S.P[0][0][0];
  T* fb = reinterpret_cast<T*>(reinterpret_cast<char*>(&S) + sizeof(S.P));
  constexpr int NSUB = C::NSP * ND;
  {
    const unsigned x = IC.get(I::RREG);
    const int t0 = item_thread<I::NTHR>(), c = t0 % C::NSP, st = C::cell(x);
#pragma unroll
    for (int m = 0; m < (NSUB + I::NTHR - 1) / I::NTHR; ++m) {
      const int sub = t0 + m * I::NTHR, v = sub / C::NSP;
      if (sub < NSUB && (x & C::VALID)) {
        const T* src = base + C::src(x) + v * C::PV;
        T qm, qp;
        weno5_cell<T>(src[0], src[st], src[2 * st], src[3 * st], src[4 * st], eps, linear, qm, qp);
        if (x & C::PUT) fb[C::dst(x) + v * C::DV] = qm;
        S.QS[c][v] = qp;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < I::RREG; ++r) {
    const unsigned x = IC.get(r);
    if (x & C::VALID) {
      const int st = C::cell(x);
      const T* src = base + C::src(x);
      T* dst = fb + C::dst(x);
      const bool put = (x & C::PUT) != 0;
      T cur[5];
      if constexpr (RPF) {
#pragma unroll
        for (int m = 0; m < 5; ++m) cur[m] = src[m * st];
      }
#pragma unroll
      for (int v = 0; v < ND; ++v) {
        T nxt[5];
        if constexpr (RPF) {
          if (v + 1 < ND) {
#pragma unroll
            for (int m = 0; m < 5; ++m) nxt[m] = src[(v + 1) * C::PV + m * st];
          }
        } else {
#pragma unroll
          for (int m = 0; m < 5; ++m) cur[m] = src[v * C::PV + m * st];
        }
        T qm;
        weno5_cell<T>(cur[0], cur[1], cur[2], cur[3], cur[4], eps, linear, qm, QP[r][v]);
        if (put) dst[v * C::DV] = qm;
        SNAP_VAR_FENCE();
        if constexpr (RPF) {
          if (v + 1 < ND) {
#pragma unroll
            for (int m = 0; m < 5; ++m) cur[m] = nxt[m];
          }
        }
      }
    }
  }
}

// Phase L (as phase_lmars; one reference rref, pref for every face of the level).
template <typename T, int NV, int ND, int TX, int TY, int SNRM, bool MIX, bool HLLC>
__device__ __forceinline__ void packed_lmars(Plane<T, NV, TX, TY>& S,
                                             const ItemCodes<NV, TX, TY>& IC, T eps, bool linear,
                                             T gamma, T inv_gm1, T gm1, const Mixture& mx, T rref,
                                             T pref, const T (&QP)[PlaneItems<TX, TY>::RREG][ND]) {
  using C = ItemCodes<NV, TX, TY>;
  using I = PlaneItems<TX, TY>;
  T* base = &S.P[0][0][0];
  T* fb = reinterpret_cast<T*>(reinterpret_cast<char*>(&S) + sizeof(S.P));
#pragma unroll
  for (int r = 0; r <= I::RREG; ++r) {
    const unsigned x = IC.get(r);
    if ((x & C::FACE) && (r < I::RREG || item_thread<I::NTHR>() < C::NSP)) {
      T* fp = fb + C::dst(x) - C::face(x);
      T xl[ND], xr[ND], f[ND];
#pragma unroll
      for (int v = 0; v < ND; ++v) {
        xr[v] = r < I::RREG ? QP[r < I::RREG ? r : 0][v] : S.QS[item_thread<I::NTHR>()][v];
        xl[v] = fp[v * C::DV];
      }
      bool left = false;
      if (x & C::XA)
        riemann_flux<T, ND, MIX, HLLC>(xl, xr, 1, rref, pref, gamma, inv_gm1, gm1, mx, f, left);
      else
        riemann_flux<T, ND, MIX, HLLC>(xl, xr, SNRM, rref, pref, gamma, inv_gm1, gm1, mx, f, left);
#pragma unroll
      for (int v = 0; v < ND; ++v) fp[v * C::DV] = f[v];
      if (ND < NV && r < I::RREG) {
        const int st = C::cell(x);
        const UpwindStencil<T> u(base + C::src(x) - st, st, left);
#pragma unroll
        for (int v = ND; v < NV; ++v) {
          fp[v * C::DV] = f[0] * u.face(v * C::PV, eps, linear);
          SNAP_VAR_FENCE();
        }
      }
      if (HLLC && ND < NV && r == I::RREG)
        S.QS[item_thread<I::NTHR>()][0] = left ? T(1) : T(0);   // for packed_tracer_rest
    }
  }
}

// As phase_tracer_rest.
template <typename T, int NV, int ND, int TX, int TY, bool HLLC>
__device__ __forceinline__ void packed_tracer_rest(Plane<T, NV, TX, TY>& S,
                                                   const ItemCodes<NV, TX, TY>& IC, T eps,
                                                   bool linear) {
  using C = ItemCodes<NV, TX, TY>;
  using I = PlaneItems<TX, TY>;
  if constexpr (ND < NV) {
    constexpr int NSUB = C::NSP * (NV - ND);
    T* base = &S.P[0][0][0];
    T* fb = reinterpret_cast<T*>(reinterpret_cast<char*>(&S) + sizeof(S.P));
    const unsigned x = IC.get(I::RREG);
    if (x & C::FACE) {
      T* fp = fb + C::dst(x) - C::face(x);
      const T f0 = fp[0];
      const int st = C::cell(x);
      const bool left = HLLC ? S.QS[item_thread<I::NTHR>() % C::NSP][0] != T(0) : f0 > T(0);
      const UpwindStencil<T> u(base + C::src(x) - st, st, left);
#pragma unroll
      for (int m = 0; m < (NSUB + I::NTHR - 1) / I::NTHR; ++m) {
        const int sub = item_thread<I::NTHR>() + m * I::NTHR, v = ND + sub / C::NSP;
        if (sub < NSUB) fp[v * C::DV] = f0 * u.face(v * C::PV, eps, linear);
      }
    }
  }
}

// Halo item it of the plane: 6 cells beyond each x edge of every row, then 6
// beyond each second-axis edge of every column. Returns false outside the
// active part of a ragged tile.
template <int TX, int TY>
__device__ __forceinline__ bool halo_item(int it, int w, int h, int& ii, int& jj) {
  // selects rather than two branches that each write one of ii / jj: the
  // compiler would merge those writes into one store through a selected
  // address and keep ii, jj in scratch memory
  const bool xs = it < 6 * TY;   // x halo (columns left / right of the tile)
  const int r = xs ? it : it - 6 * TY;
  const int m = r % 6, q = r / 6;
  const int e = m < 3 ? m - 3 : (xs ? w : h) + m - 3;
  ii = xs ? e : q;
  jj = xs ? q : e;
  return q < (xs ? h : w);
}

// The 3-D kernels that split the reconstruction's last items by variable
// (phase_reconstruct; the packed form always does): not the unpacked ones with
// the sedimentation terms, which are held to two waves per SIMD in single
// precision.
template <typename T, int NT, bool MIX, bool SED>
constexpr bool split_reconstruct() {
  return !SED;
}

// ---------------------------------------------------------------------------
// 3-D kernel
// ---------------------------------------------------------------------------
template <typename T, int NV>
__device__ __forceinline__ void load_cons(const T* __restrict__ q, long long off, long long sv,
                                          T (&c)[NV]) {
#pragma unroll
  for (int v = 0; v < NV; ++v) c[v] = q[off + v * sv];
}

template <typename T, int NV, bool MIX>
__device__ __forceinline__ void cons_to_prim_t(const T (&c)[NV], const LevelRef& lr, double gm1,
                                               const Mixture& mx, T (&x)[NV]) {
  if constexpr (sizeof(T) == 4 && !MIX) {
    cons_to_prim_sp<NV>(c, lr.ra, lr.rs, lr.ps, gm1, x);
    return;
  }
  double cd[NV], xd[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) cd[v] = static_cast<double>(c[v]);
  cons_to_prim_eos<NV, MIX>(cd, lr.ra, lr.rs, lr.ps, gm1, mx, xd);
#pragma unroll
  for (int v = 0; v < NV; ++v) x[v] = static_cast<T>(xd[v]);
}

// SED (mixture with falling condensates): the sedimentation terms of Sec. 2
// (the fall fluxes of mass, momentum and energy through the z faces and the
// frictional heating, sediment_cell) are added to the right-hand side in phase
// D from the window's levels s-1, s, s+1; these instances load nothing a
// level ahead, which makes room for that work in the registers.
//
// Registers decide how many waves a SIMD holds (168 each for three, 256 for
// two), and the kernels with tracers sit around those steps. Per instance:
//   pack   item addresses packed (ItemCodes): 16 to 20 registers fewer for 3.5 %
//          more instructions, where that saves a wave or the spills;
//   ahead  the next level's halo, window and stage-combination values loaded a
//          level ahead: 4 NV registers, where they leave the waves in place;
//   waves  the waves per SIMD the registers are held to (1: left alone).
// Microseconds per SSP-RK3 step on 256 x 192 x 96 with passive tracers, before
// (every variable two-sided, unpacked, loaded ahead in single precision) and now:
//   single precision   2 tracers 918, 756; 3: 1027, 861; 4: 1145, 953; 5: 1241, 1095
//   double precision   2 tracers 1983, 1370; 3: 2237, 1722; 4 (HLLC): 2614, 2251
// Packed further, single precision with six tracers took 1345 -> 1390 us (72 bytes
// of scratch per lane), so from six on the registers are left alone. The
// sedimentation instances load nothing ahead, which makes room for their fall
// fluxes, and are held to two waves; packed from six tracers on, where they
// spilled (moist step with six tracers on 160 x 144 x 96: 1020 -> 961 us).
// LOW: a launch that more waves per SIMD do not help, of at most one workgroup per
// compute unit, or two in single precision, where the registers left alone hold two
// waves: the instances whose held registers spill, that gave up the loads ahead for
// a wave, or that are packed leave all that there (75 x 60 x 40, double precision, 3
// tracers: 187 us held, 175; single precision with 2 to 5 tracers, held and not:
// 40 x 40 x 40 with 4 tracers 130, 123; 200 x 4 x 100, 1.3 workgroups per compute unit,
// 105, 103; 112, 110; 124, 118; 136, 127).
template <typename T, int NT, bool MIX, bool SED, bool LOW = false>
struct Stage3DShape {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr bool pack = SED   ? F32 && NT >= 6
                               : MIX ? F32 && (NT == 6 || NT == 8)
                               : F32 ? (NT == 4 || NT == 5) && !LOW
                                     : NT >= 2 && NT <= 4;
  static constexpr bool ahead =
      !SED && (F32 ? NT <= 6 && (MIX || NT == 0 || NT == 6 || LOW) : NT == 0);
  static constexpr int waves = LOW                    ? 1
                               : SED                  ? (F32 || NT == 1 ? 2 : 1)
                               : MIX                  ? (F32 && NT >= 6 ? 2 : 1)
                               : F32 && NT >= 1 && NT <= 5 ? 3
                               : !F32 && NT >= 2 && NT <= 4 ? 2
                                                      : 1;
  // the instances for which a LOW one exists
  static constexpr bool has_low = !MIX && !SED && (F32 ? NT >= 2 && NT <= 5 : NT == 3 || NT == 4);
};
template <typename T, int NT, int TX, int TY, bool MIX = false, bool HLLC = false,
          bool SED = false, bool LOW = false>
__global__ void __launch_bounds__(TX* TY, (Stage3DShape<T, NT, MIX, SED, LOW>::waves))
    k_stage3d(StageArgs a) {
  constexpr int NV = 5 + NT;
  constexpr bool GF = ghosts_in_place(NT);
  static_assert(!SED || (MIX && NT > 0 && !HLLC), "sedimentation needs the mixture");
  using I = PlaneItems<TX, TY>;
  constexpr int NHALO = 6 * (TX + TY);
  constexpr int HR = (NHALO + I::NTHR - 1) / I::NTHR;   // halo items per thread
  constexpr bool PF = Stage3DShape<T, NT, MIX, SED, LOW>::ahead;
  __shared__ Plane<T, NV, TX, TY> S;
  const T* __restrict__ qs = static_cast<const T*>(a.qs);

  const int tid = threadIdx.x;
  const int ti = tid % TX, tj = tid / TX;
  int tx, ty, k0, k1;
  if (a.pass_map) {
    const int tiles = a.tiles_x * a.tiles_y;
    const int kc = blockIdx.x / tiles;
    const int r = blockIdx.x - kc * tiles;
    const int t = (r % 8) * (tiles / 8) + r / 8;
    tx = t % a.tiles_x;
    ty = t / a.tiles_x;
    k0 = a.kb[kc];
    k1 = a.kb[kc + 1];
  } else {
    const int L = xcd_logical_block(blockIdx.x, gridDim.x);
    tx = L % a.tiles_x;
    const int rr_ = L / a.tiles_x;
    ty = rr_ % a.tiles_y;
    const int kc = rr_ / a.tiles_y;
    k0 = kc * a.tz;
    k1 = min(k0 + a.tz, a.nz);
  }
  const int i0 = tx * TX, j0 = ty * TY;
  const int w = min(TX, a.nx - i0), h = min(TY, a.ny - j0);
  const bool act = ti < w && tj < h;
  const T eps = static_cast<T>(a.eps), gamma = static_cast<T>(a.gamma);
  const T inv_gm1 = static_cast<T>(a.inv_gm1), gm1t = static_cast<T>(a.gm1);
  const T dzi = static_cast<T>(a.dzi);   // the sedimentation terms' own differences
  // inverse spacings for the flux differences (the fluxes carry flux_scale)
  constexpr double FSI = 1.0 / flux_scale<MIX, HLLC>();
  const T fdx = static_cast<T>(a.dxi * FSI), fdy = static_cast<T>(a.dyi * FSI);
  const T fdz = static_cast<T>(a.dzi * FSI);
  const bool linear = a.linear != 0;
  // read before any store: the stores of the level loop could alias *a.smax,
  // and a load inside the loop would be repeated at every level
  const double dtd = stage_dt(a);
  store_stage_dt(a, dtd);
  constexpr bool FS = fused_speed<T, NT>();
  if constexpr (FS) {
    if (a.smax_zero != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *a.smax_zero = 0ULL;
  }
  // running maximum (IEEE bits) of the output's signal speed: one LDS slot per
  // thread, which keeps it out of the registers the level loop needs
  __shared__ unsigned long long smx_lds[FS ? TX * TY : 1];
  if constexpr (FS) smx_lds[tid] = 0ULL;
  const bool combine = a.rhs_mode == 0;
  const bool use_qn = combine && a.ca != 0.0;
  const T* qn = static_cast<const T*>(a.qn);

  // padded offset of (i, j, k) with interior coordinates (k may be a ghost level)
  auto poff = [&](int i, int j, int k) -> long long {
    return (long long)(k + NG) * a.sz + (long long)(j + NG) * a.sy + (i + NG);
  };
  const int ic = i0 + (act ? ti : 0), jc = j0 + (act ? tj : 0);
  const long long col = poff(ic, jc, 0) - (long long)NG * a.sz;   // offset of level -3

  // halo items of this thread (fixed across levels) and their column offsets;
  // with ghost_free a halo cell beyond the domain is read at the interior cell
  // the fill would copy (its momentum normal to a reflecting wall is negated
  // where it is planed)
  int hii[HR], hjj[HR];
  bool hok[HR];
  long long hoff[HR];
#pragma unroll
  for (int r = 0; r < HR; ++r) {
    const int it = item_thread<I::NTHR>() + r * I::NTHR;
    hok[r] = it < NHALO && halo_item<TX, TY>(it, w, h, hii[r], hjj[r]);
    int gi = i0 + hii[r], gj = j0 + hjj[r];
    if (GF && (a.ghost & GF_ON) && hok[r]) {
      bool fx, fy;
      gi = ghost_src(gi, a.nx, (a.ghost & GF_RX) ? 1 : 0, fx);
      gj = ghost_src(gj, a.ny, (a.ghost & GF_RY) ? 1 : 0, fy);
    }
    hoff[r] = hok[r] ? poff(gi, gj, 0) - (long long)NG * a.sz : 0;
  }
  auto lev = [&](int k) -> long long { return (long long)(k + NG) * a.sz; };
  // level read for window level k (uniform): k itself, or with GF_ON the
  // level a z ghost copies; zf: rho w changes sign (mirror at a z wall)
  auto zsrc = [&](int k, bool& zf) -> int {
    zf = false;
    if (GF && (a.ghost & GF_ON) && (k < 0 || k >= a.nz))
      return ghost_src(k, a.nz, (a.ghost & GF_RZ) ? 1 : 0, zf);
    return k;
  };

  constexpr int ND = two_sided<T, NV, MIX, true>();
  constexpr bool PACK = Stage3DShape<T, NT, MIX, SED, LOW>::pack && TX == TY;
  constexpr bool TAN = upwind_tangential<T, ND, MIX, HLLC, PACK>();
  constexpr int N2 = TAN ? 3 : ND;
  T W[5][NV];     // primitives of levels s-1 .. s+3 (own column)
  // left states at the vertical face above the current level; for the variables
  // that are reconstructed on the upwind side only, their values on level s-2
  T qmc[NV];
  T fzc[NV];      // vertical flux at the lower face of the current level
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    qmc[v] = T(0);
    fzc[v] = T(0);
  }
  if (act) {
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      const int k = k0 - 3 + l;
      bool zf;
      T c[NV];
      load_cons<T, NV>(qs, col + lev(zsrc(k, zf)), a.sv, c);
      if (zf) c[3] = -c[3];
      cons_to_prim_t<T, NV, MIX>(c, level_ref(a.pert, a.rbar_c[k + NG], a.pbar_c[k + NG]), a.gm1,
                                 a.mix, W[l]);
    }
  }
  // prefetched raw conserved values: halo cells of the next level to be
  // planed, the window's next level, and this level's own Qs / Qn
  T hc[HR][NV];
  if constexpr (PF) {
#pragma unroll
    for (int r = 0; r < HR; ++r)
      if (hok[r]) load_cons<T, NV>(qs, hoff[r] + lev(k0), a.sv, hc[r]);
  }
  // this level's own Qs (and Qn): the stage combination and the gravity work
  auto load_own = [&](int s, T (&qsc)[NV], T (&qnc)[NV]) {
    if (combine) {
      load_cons<T, NV>(qs, col + lev(s), a.sv, qsc);
      if (use_qn) load_cons<T, NV>(qn, col + lev(s), a.sv, qnc);
    } else {
      qsc[3] = qs[col + lev(s) + 3 * a.sv];
    }
  };

  T QP[I::RREG][N2];
  const ItemCodes<PACK ? NV : 1, PACK ? TX : 16, PACK ? TY : 16> IC(w, h);
  for (int s = k0 - 2; s < k1; ++s) {
    T wc[NV], qsc[NV], qnc[NV];
    bool wzf;
    const int wsrc = zsrc(s + 3, wzf);
    if constexpr (PF) {
      if (act) {
        load_cons<T, NV>(qs, col + lev(wsrc), a.sv, wc);
        if (s >= k0) load_own(s, qsc, qnc);
      }
    }
    if (s >= k0) {
      // ---- (P) primitives of level s: own cell from the window, halo prefetched
      const double rbs = a.rbar_c[s + NG], pbs = a.pbar_c[s + NG];
      const LevelRef lrs = level_ref(a.pert, rbs, pbs);
      if (act) {
#pragma unroll
        for (int v = 0; v < NV; ++v) S.P[v][tj + 3][ti + 3] = W[1][v];
      }
#pragma unroll
      for (int r = 0; r < HR; ++r) {
        if (hok[r]) {
          T x[NV];
          if constexpr (!PF) load_cons<T, NV>(qs, hoff[r] + lev(s), a.sv, hc[r]);
          if (GF && (a.ghost & GF_ON) && (a.ghost & (GF_RX | GF_RY))) {
            const int gi = i0 + hii[r], gj = j0 + hjj[r];
            if ((a.ghost & GF_RX) && (gi < 0 || gi >= a.nx)) hc[r][1] = -hc[r][1];
            if ((a.ghost & GF_RY) && (gj < 0 || gj >= a.ny)) hc[r][2] = -hc[r][2];
          }
          cons_to_prim_t<T, NV, MIX>(hc[r], lrs, a.gm1, a.mix, x);
#pragma unroll
          for (int v = 0; v < NV; ++v) S.P[v][hjj[r] + 3][hii[r] + 3] = x[v];
          if constexpr (PF) {
            if (s + 1 < k1) load_cons<T, NV>(qs, hoff[r] + lev(s + 1), a.sv, hc[r]);
          }
        }
      }
      __syncthreads();
      // ---- (R) WENO5 in x and y ---------------------------------------------
      if constexpr (PACK)
        packed_reconstruct<T, NV, ND, TX, TY>(S, IC, eps, linear, QP);
      else if constexpr (TAN)
        phase_reconstruct_sides<T, NV, TX, TY, 2>(S, w, h, eps, linear, QP);
      else
        phase_reconstruct<T, NV, ND, TX, TY, split_reconstruct<T, NT, MIX, SED>()>(S, w, h, eps,
                                                                                  linear, QP);
      __syncthreads();
      // ---- (L) LMARS at x and y faces (level references) ---------------------
      const T rbT = static_cast<T>(rbs), pbT = static_cast<T>(pbs);
      auto levref = [&](int, T& r, T& p) {
        r = rbT;
        p = pbT;
      };
      if constexpr (PACK) {
        packed_lmars<T, NV, ND, TX, TY, 2, MIX, HLLC>(S, IC, eps, linear, gamma, inv_gm1, gm1t,
                                                      a.mix, rbT, pbT, QP);
        __syncthreads();
        packed_tracer_rest<T, NV, ND, TX, TY, HLLC>(S, IC, eps, linear);
      } else {
        if constexpr (TAN)
          phase_lmars_sides<T, NV, TX, TY, 2>(S, w, h, eps, linear, gamma, inv_gm1, levref, levref,
                                              QP);
        else
          phase_lmars<T, NV, ND, TX, TY, 2, MIX, HLLC>(S, w, h, eps, linear, gamma, inv_gm1, gm1t,
                                                       a.mix, levref, levref, QP);
        __syncthreads();
        phase_tracer_rest<T, NV, ND, TX, TY, HLLC>(S, w, h, eps, linear);
      }
    }
    // ---- vertical direction, own column: face s+1/2 (z-face index s+1) -------
    T dfz[NV];
    if (act) {
      if constexpr (!PF) load_cons<T, NV>(qs, col + lev(wsrc), a.sv, wc);
      if (wzf) wc[3] = -wc[3];
      cons_to_prim_t<T, NV, MIX>(wc, level_ref(a.pert, a.rbar_c[s + 3 + NG], a.pbar_c[s + 3 + NG]),
                                 a.gm1, a.mix, W[4]);
      if constexpr (TAN) {
        T qmn[ND], qpn[ND];
#pragma unroll
        for (int v = 0; v < ND; ++v) {
          if (v == 1 || v == 2) continue;
          weno5_cell<T>(W[0][v], W[1][v], W[2][v], W[3][v], W[4][v], eps, linear, qmn[v], qpn[v]);
          SNAP_VAR_FENCE();
        }
        if (s >= k0 - 1) {
          T fz[ND];
          bool left;
          auto upwind = [&](int v) {   // levels s-2 .. s+2 up, or s+3 .. s-1 down
            return weno5_face<T>(left ? qmc[v] : W[4][v], left ? W[0][v] : W[3][v],
                                 left ? W[1][v] : W[2][v], left ? W[2][v] : W[1][v],
                                 left ? W[3][v] : W[0][v], eps, linear);
          };
          const T xl[3] = {qmc[0], qmc[3], qmc[4]}, xr[3] = {qpn[0], qpn[3], qpn[4]};
          const LmarsFace<T> o = lmars_side<T>(xl, xr, static_cast<T>(a.rbar_f[s + 1]),
                                               static_cast<T>(a.pbar_f[s + 1]), gamma);
          left = o.left;
          const T q1 = upwind(1);
          SNAP_VAR_FENCE();
          const T q2 = upwind(2);
          T f[5];
          lmars_rest<T>(o, q1, q2, gamma, inv_gm1, f);
          fz[0] = f[0];
          fz[1] = f[2];
          fz[2] = f[3];
          fz[3] = f[1];
          fz[4] = f[4];
#pragma unroll
          for (int v = 0; v < ND; ++v) {
            dfz[v] = fz[v] - fzc[v];
            fzc[v] = fz[v];
          }
          // tracers: the upwind side's value (levels s-2 .. s+2 up, or s+3 .. s-1 down)
#pragma unroll
          for (int v = ND; v < NV; ++v) {
            const T fq = fz[0] * upwind(v);
            dfz[v] = fq - fzc[v];
            fzc[v] = fq;
            SNAP_VAR_FENCE();
          }
        }
#pragma unroll
        for (int v = 0; v < ND; ++v) qmc[v] = v == 1 || v == 2 ? W[0][v] : qmn[v];
#pragma unroll
        for (int v = ND; v < NV; ++v) qmc[v] = W[0][v];
      } else {
        T qmn[ND], qpn[ND];
#pragma unroll
        for (int v = 0; v < ND; ++v) {
          weno5_cell<T>(W[0][v], W[1][v], W[2][v], W[3][v], W[4][v], eps, linear, qmn[v], qpn[v]);
          SNAP_VAR_FENCE();
        }
        if (s >= k0 - 1) {
          T fz[ND];
          bool left = false;
          T xl[ND];
#pragma unroll
          for (int v = 0; v < ND; ++v) xl[v] = qmc[v];
          riemann_flux<T, ND, MIX, HLLC>(xl, qpn, 3, static_cast<T>(a.rbar_f[s + 1]),
                                         static_cast<T>(a.pbar_f[s + 1]), gamma, inv_gm1, gm1t,
                                         a.mix, fz, left);
#pragma unroll
          for (int v = 0; v < ND; ++v) {
            dfz[v] = fz[v] - fzc[v];
            fzc[v] = fz[v];
          }
          // tracers: the upwind side's value (levels s-2 .. s+2 up, or s+3 .. s-1 down)
#pragma unroll
          for (int v = ND; v < NV; ++v) {
            const T q = weno5_face<T>(left ? qmc[v] : W[4][v], left ? W[0][v] : W[3][v],
                                      left ? W[1][v] : W[2][v], left ? W[2][v] : W[1][v],
                                      left ? W[3][v] : W[0][v], eps, linear);
            const T fq = fz[0] * q;
            dfz[v] = fq - fzc[v];
            fzc[v] = fq;
            SNAP_VAR_FENCE();
          }
        }
#pragma unroll
        for (int v = 0; v < ND; ++v) qmc[v] = qmn[v];
#pragma unroll
        for (int v = ND; v < NV; ++v) qmc[v] = W[0][v];
      }
    }
    // ---- (D) divergence, gravity, output -------------------------------------
    if (ND < NV && s >= k0) __syncthreads();   // the last tracer fluxes
    if (s >= k0 && act) {
      if constexpr (!PF) load_own(s, qsc, qnc);
      T R[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        T r = -((S.FX[v][tj][ti + 1] - S.FX[v][tj][ti]) * fdx);
        r = r - (S.FY[v][tj + 1][ti] - S.FY[v][tj][ti]) * fdy;
        R[v] = r - dfz[v] * fdz;
      }
      const T grav = static_cast<T>(a.grav);
      R[3] = R[3] - grav * W[1][0];
      R[4] = R[4] - grav * qsc[3];
      if constexpr (SED) {
        const bool wall_lo = a.sed.closed_z && s == 0, wall_up = a.sed.closed_z && s == a.nz - 1;
        sediment_cell<T, NV>(W[0], W[1], W[2], static_cast<T>(a.rbar_c[s - 1 + NG]),
                             static_cast<T>(a.pbar_c[s - 1 + NG]), static_cast<T>(a.rbar_c[s + NG]),
                             static_cast<T>(a.pbar_c[s + NG]), static_cast<T>(a.rbar_c[s + 1 + NG]),
                             static_cast<T>(a.pbar_c[s + 1 + NG]), wall_lo, wall_up, a.mix, a.sed,
                             dzi, grav, R);
      }
      const long long po = col + lev(s);
      if (!combine) {
        T* __restrict__ o = static_cast<T*>(a.out);
        const long long ro = (long long)s * a.rz + (long long)jc * a.ry + ic;
#pragma unroll
        for (int v = 0; v < NV; ++v) o[ro + v * a.rv] = R[v];
      } else {
        const T dt = static_cast<T>(dtd), ca = static_cast<T>(a.ca), cb = static_cast<T>(a.cb);
        T* o = static_cast<T*>(a.out);
        T ov[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const T t = qsc[v] + dt * R[v];
          ov[v] = use_qn ? ca * qnc[v] + cb * t : cb * t;
          o[po + v * a.sv] = ov[v];
        }
        if constexpr (FS) {
          if (a.smax_out != nullptr) {
            // sum_d (|u_d| + c) / dx_d of the new state (times 1 / dx_d), in the CFL kernel's
            // order and operations (no contraction)
#pragma clang fp contract(off)
            // (perturbation storage: rho and p with the level references added back)
            const double rbo = a.pert ? a.rbar_c[s + NG] : 0.0;
            const double pbo = a.pert ? a.pbar_c[s + NG] : 0.0;
            const double rho = static_cast<double>(ov[0]) + rbo, mx = ov[1], my = ov[2], mz = ov[3];
            const double E = ov[4];
            const double inv = 1.0 / rho;
            const double u = mx * inv, v = my * inv, w = mz * inv;
            const double K = 0.5 * ((mx * u + my * v) + mz * w);
            const double p = a.gm1 * (E - K) + pbo;
            const double cs = sqrt(a.gamma * p / rho);
            double sp = (fabs(u) + cs) * a.dxi;
            sp = sp + (fabs(v) + cs) * a.dyi;
            sp = sp + (fabs(w) + cs) * a.dzi;
            if (!(rho > 0.0) || !(p > 0.0)) sp = __builtin_nan("");
            const unsigned long long sb = (unsigned long long)__double_as_longlong(sp);
            const unsigned long long cur = smx_lds[tid];
            smx_lds[tid] = sb > cur ? sb : cur;
          }
        }
      }
    }
    // shift the window
#pragma unroll
    for (int l = 0; l < 4; ++l)
#pragma unroll
      for (int v = 0; v < NV; ++v) W[l][v] = W[l + 1][v];
  }
  if constexpr (FS) {
    if (a.smax_out != nullptr) {
      unsigned long long smx = smx_lds[tid];
      for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o2 = __shfl_xor(smx, off, 64);
        smx = o2 > smx ? o2 : smx;
      }
      if ((threadIdx.x & 63) == 0) atomicMax(a.smax_out, smx);
    }
  }
}

// ---------------------------------------------------------------------------
// 2-D (x-z) tile: TX x TZ tile number L of the plane, z is the second in-plane
// axis. Shared by the single-domain kernel and the batched (ensemble) kernel.
// Small domains are bound by launches and latency, so a step is three launches:
// ghost values are read at their sources (GF_ON) and the last stage reduces the
// next step's signal speed (SPEED: not in a batch, whose time steps come from the
// host). With three fills and the reduction's two launches
// beside them a device-dt step of 64 x 64 cells in double precision took 43 us,
// without them 27 us; a batched step of 64 domains (50 368 cells on average)
// in single precision 386 -> 371 us.
// ---------------------------------------------------------------------------
template <typename T, int NT, int TX, int TZ, bool MIX, bool HLLC, bool SPEED>
__device__ __forceinline__ void stage2d_tile(const StageArgs& a, int L,
                                             Plane<T, 5 + NT, TX, TZ>& S) {
  constexpr int NV = 5 + NT;
  using I = PlaneItems<TX, TZ>;
  const T* __restrict__ qs = static_cast<const T*>(a.qs);

  const int tid = threadIdx.x;
  const int ti = tid % TX, tk = tid / TX;
  const int tx = L % a.tiles_x;
  const int tzi = L / a.tiles_x;
  const int i0 = tx * TX, k0 = tzi * TZ;
  const int w = min(TX, a.nx - i0), h = min(TZ, a.nz - k0);
  const bool act = ti < w && tk < h;
  const T eps = static_cast<T>(a.eps), gamma = static_cast<T>(a.gamma);
  const T inv_gm1 = static_cast<T>(a.inv_gm1), gm1t = static_cast<T>(a.gm1);
  // inverse spacings for the flux differences (the fluxes carry flux_scale)
  constexpr double FSI = 1.0 / flux_scale<MIX, HLLC>();
  const T fdx = static_cast<T>(a.dxi * FSI), fdz = static_cast<T>(a.dzi * FSI);
  const bool linear = a.linear != 0;

  auto poff = [&](int i, int k) -> long long { return (long long)(k + NG) * a.sz + (i + NG); };

  // ---- (P) primitives of the tile and its halo --------------------------------
  if (act) {
    const int k = k0 + tk;
    T x[NV];
    load_prim<T, NV, MIX>(qs, poff(i0 + ti, k), a.sv,
                          level_ref(a.pert, a.rbar_c[k + NG], a.pbar_c[k + NG]), a.gm1, a.mix, x);
#pragma unroll
    for (int v = 0; v < NV; ++v) S.P[v][tk + 3][ti + 3] = x[v];
  }
  for (int it = item_thread<I::NTHR>(); it < 6 * (TX + TZ); it += I::NTHR) {
    int ii, kk;
    if (halo_item<TX, TZ>(it, w, h, ii, kk)) {
      const int k = k0 + kk;
      int gi = i0 + ii, gk = k;
      bool fx = false, fz = false;
      if (a.ghost & GF_ON) {   // a ghost cell: read at the cell the fill copies
        gi = ghost_src(gi, a.nx, (a.ghost & GF_RX) ? 1 : 0, fx);
        gk = ghost_src(gk, a.nz, (a.ghost & GF_RZ) ? 1 : 0, fz);
      }
      T c[NV], x[NV];
      load_cons<T, NV>(qs, poff(gi, gk), a.sv, c);
      if (fx) c[1] = -c[1];
      if (fz) c[3] = -c[3];
      cons_to_prim_t<T, NV, MIX>(c, level_ref(a.pert, a.rbar_c[k + NG], a.pbar_c[k + NG]), a.gm1,
                                 a.mix, x);
#pragma unroll
      for (int v = 0; v < NV; ++v) S.P[v][kk + 3][ii + 3] = x[v];
    }
  }
  __syncthreads();
  constexpr int ND = two_sided<T, NV, MIX, false>();
  T QP[I::RREG][ND];
  phase_reconstruct<T, NV, ND, TX, TZ>(S, w, h, eps, linear, QP);
  __syncthreads();
  auto xref = [&](int kk, T& r, T& p) {
    r = static_cast<T>(a.rbar_c[k0 + kk + NG]);
    p = static_cast<T>(a.pbar_c[k0 + kk + NG]);
  };
  auto zref = [&](int fk, T& r, T& p) {
    r = static_cast<T>(a.rbar_f[k0 + fk]);
    p = static_cast<T>(a.pbar_f[k0 + fk]);
  };
  phase_lmars<T, NV, ND, TX, TZ, 3, MIX, HLLC>(S, w, h, eps, linear, gamma, inv_gm1, gm1t, a.mix,
                                               xref, zref, QP);
  __syncthreads();
  if constexpr (ND < NV) {
    phase_tracer_rest<T, NV, ND, TX, TZ, HLLC>(S, w, h, eps, linear);
    __syncthreads();
  }
  unsigned long long smx = 0ULL;
  if (act) {
    T R[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const T r = -((S.FX[v][tk][ti + 1] - S.FX[v][tk][ti]) * fdx);
      R[v] = r - (S.FY[v][tk + 1][ti] - S.FY[v][tk][ti]) * fdz;
    }
    const int i = i0 + ti, k = k0 + tk;
    const long long po = poff(i, k);
    const T grav = static_cast<T>(a.grav);
    R[3] = R[3] - grav * S.P[0][tk + 3][ti + 3];
    R[4] = R[4] - grav * qs[po + 3 * a.sv];
    const long long ro = (long long)k * a.rz + i;
    write_cell<T, NV>(a, qs, po, ro, R);
    if constexpr (SPEED) {
      if (a.smax_out != nullptr)
        smx = speed_bits_2d<T, NV>(a, R, a.pert ? a.rbar_c[k + NG] : 0.0,
                                   a.pert ? a.pbar_c[k + NG] : 0.0);
    }
  }
  // the next step's signal speed: one atomic per wave, and none where the
  // running maximum (read once, perhaps stale, never too large) already covers it
  if constexpr (SPEED) {
    if (a.smax_out != nullptr) {
      for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o2 = __shfl_xor(smx, off, 64);
        smx = o2 > smx ? o2 : smx;
      }
      if ((threadIdx.x & 63) == 0 &&
          smx > __hip_atomic_load(a.smax_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(a.smax_out, smx);
    }
  }
}

template <typename T, int NT, int TX, int TZ, bool MIX = false, bool HLLC = false>
__global__ void __launch_bounds__(TX* TZ) k_stage2d(StageArgs a) {
  __shared__ Plane<T, 5 + NT, TX, TZ> S;
  store_stage_dt(a, stage_dt(a));
  if (a.smax_zero != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *a.smax_zero = 0ULL;
  stage2d_tile<T, NT, TX, TZ, MIX, HLLC, !MIX>(a, xcd_logical_block(blockIdx.x, gridDim.x), S);
}

// Ensemble of 2-D domains in one persistent launch: work item w is tile
// w - first[m] of member m (first[m] <= w < first[m+1]); every block walks the
// items w = blockIdx.x, blockIdx.x + gridDim.x, ... A barrier closes every tile:
// its last phase still reads the primitive plane (density perturbation for the
// gravity source) that the next tile's first phase overwrites.
// The single-precision instances of 32 x 8 and 8 x 32 cells are held to six waves per
// SIMD, which they held before they read ghosts in place (82 and 95 registers).
template <typename T, int NT, int TX, int TZ>
constexpr int batch_waves() {
  return sizeof(T) == 4 && NT == 0 && TX * TZ == 256 && (TX == 8 || TZ == 8) ? 6 : 1;
}
template <typename T, int NT, int TX, int TZ, bool MIX = false, bool HLLC = false>
__global__ void __launch_bounds__(TX* TZ, (batch_waves<T, NT, TX, TZ>())) k_stage2d_batched(const StageArgs* __restrict__ descs,
                                                            const int* __restrict__ first, int n) {
  __shared__ Plane<T, 5 + NT, TX, TZ> S;
  const int total = first[n];
  for (int w = blockIdx.x; w < total; w += gridDim.x) {
    int lo = 0, hi = n;   // first[lo] <= w < first[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (first[mid] <= w)
        lo = mid;
      else
        hi = mid;
    }
    const StageArgs a = descs[lo];
    stage2d_tile<T, NT, TX, TZ, MIX, HLLC, false>(a, w - first[lo], S);
    __syncthreads();
  }
}

}  // namespace snap
