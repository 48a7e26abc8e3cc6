// Instantiation and dispatch of the stage kernels for one element type.
// Included by the stage_*.hip files, one per element type and kernel family,
// so that the instantiation sets compile in parallel.
#pragma once

#include "snap_internal.h"

namespace snap {

// Tile shape per element type and variable count: the largest of 16 x 16,
// 16 x 8 and 8 x 8 whose LDS plane stays within 56 KiB, so that at least two
// (usually three) workgroups share a compute unit's 160 KiB of LDS.
template <typename T, int NT>
struct TileFor {
  static constexpr int NV = 5 + NT;
  static constexpr bool BIG = sizeof(Plane<T, NV, 16, 16>) <= 56 * 1024;
  static constexpr bool MID = sizeof(Plane<T, NV, 16, 8>) <= 56 * 1024;
#if defined(SNAP_TILE_X) && defined(SNAP_TILE_Y)
  static constexpr int TX = NT == 0 ? SNAP_TILE_X : (BIG || MID ? 16 : 8);
  static constexpr int TY = NT == 0 ? SNAP_TILE_Y : (BIG ? 16 : 8);
#else
  static constexpr int TX = BIG || MID ? 16 : 8;
  static constexpr int TY = BIG ? 16 : 8;
#endif
};

// Tile of the 3-D kernels. Passive tracers: 16 x 16 while two workgroups share
// a compute unit (80 KiB each): double precision runs two waves per SIMD at
// best, which two workgroups of 256 threads are, and the square tile has less
// halo (2.25 reconstructions and 1.75 conversions per cell, against 2.38 and
// 2.13 with 16 x 8).
template <typename T, int NT, bool MIX>
struct Tile3For {
  static constexpr bool SQ = !MIX && sizeof(Plane<T, 5 + NT, 16, 16>) <= 80 * 1024;
  static constexpr int TX = SQ ? 16 : TileFor<T, NT>::TX;
  static constexpr int TY = SQ ? 16 : TileFor<T, NT>::TY;
  // half: the smaller tile of TileFor is there too (StageArgs::half), for the
  // domains that the square one pads more (half_pays)
  static constexpr bool half = TX != TileFor<T, NT>::TX || TY != TileFor<T, NT>::TY;
};

// MIX: the mixture equation of state (instantiated for NT >= 1 only; with no
// tracers the mixture is the dry gas). HLLC: the HLLC Riemann solver (passive
// tracers).
template <typename T, int NT, bool MIX, bool HLLC = false>
int launch_nt(bool d3, const StageArgs& a, int nblocks, hipStream_t st) {
  constexpr int TX = TileFor<T, NT>::TX, TY = TileFor<T, NT>::TY;
  constexpr bool M = MIX && NT > 0;
  constexpr int TX3 = Tile3For<T, NT, M>::TX, TY3 = Tile3For<T, NT, M>::TY;
  constexpr bool LOW = Stage3DShape<T, NT, M, false>::has_low;
  constexpr bool HALF = Tile3For<T, NT, M>::half;
  if (d3 && HALF && a.half)
    hipLaunchKernelGGL((k_stage3d<T, NT, TX, TY, M, HLLC, false, HALF>), dim3(nblocks),
                       dim3(TX * TY), 0, st, a);
  else if (d3 && LOW && a.low)
    hipLaunchKernelGGL((k_stage3d<T, NT, TX3, TY3, M, HLLC, false, LOW>), dim3(nblocks),
                       dim3(TX3 * TY3), 0, st, a);
  else if (d3)
    hipLaunchKernelGGL((k_stage3d<T, NT, TX3, TY3, M, HLLC>), dim3(nblocks), dim3(TX3 * TY3), 0,
                       st, a);
  else
    hipLaunchKernelGGL((k_stage2d<T, NT, TX, TY, M, HLLC>), dim3(nblocks), dim3(TX * TY), 0, st,
                       a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T, int NT, bool MIX, bool HLLC = false>
int occupancy_nt(bool d3, bool half = false) {
  constexpr int TX = TileFor<T, NT>::TX, TY = TileFor<T, NT>::TY;
  constexpr bool M = MIX && NT > 0;
  constexpr int TX3 = Tile3For<T, NT, M>::TX, TY3 = Tile3For<T, NT, M>::TY;
  constexpr bool HALF = Tile3For<T, NT, M>::half;
  int n = 0;
  const bool f = HALF && d3 && half;
  const void* k =
      f    ? reinterpret_cast<const void*>(&k_stage3d<T, NT, TX, TY, M, HLLC, false, HALF>)
      : d3 ? reinterpret_cast<const void*>(&k_stage3d<T, NT, TX3, TY3, M, HLLC>)
           : reinterpret_cast<const void*>(&k_stage2d<T, NT, TX, TY, M, HLLC>);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, d3 && !f ? TX3 * TY3 : TX * TY, 0) !=
      hipSuccess)
    return 0;
  return n;
}

// 3-D stage kernels with the sedimentation terms (mixture, NT >= 1).
template <typename T, int NT>
int launch_sed_nt(const StageArgs& a, int nblocks, hipStream_t st) {
  constexpr int TX = TileFor<T, NT>::TX, TY = TileFor<T, NT>::TY;
  hipLaunchKernelGGL((k_stage3d<T, NT, TX, TY, true, false, true>), dim3(nblocks), dim3(TX * TY),
                     0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T, int NT>
int occupancy_sed_nt() {
  constexpr int TX = TileFor<T, NT>::TX, TY = TileFor<T, NT>::TY;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &n, reinterpret_cast<const void*>(&k_stage3d<T, NT, TX, TY, true, false, true>),
          TX * TY, 0) != hipSuccess)
    return 0;
  return n;
}

template <typename T>
int launch_sed_t(int ntracer, const StageArgs& a, int nblocks, hipStream_t st) {
  switch (ntracer) {
    case 1: return launch_sed_nt<T, 1>(a, nblocks, st);
    case 2: return launch_sed_nt<T, 2>(a, nblocks, st);
    case 3: return launch_sed_nt<T, 3>(a, nblocks, st);
    case 4: return launch_sed_nt<T, 4>(a, nblocks, st);
    case 5: return launch_sed_nt<T, 5>(a, nblocks, st);
    case 6: return launch_sed_nt<T, 6>(a, nblocks, st);
    case 7: return launch_sed_nt<T, 7>(a, nblocks, st);
    case 8: return launch_sed_nt<T, 8>(a, nblocks, st);
    default: return -1;
  }
}

template <typename T>
int occupancy_sed_t(int ntracer) {
  switch (ntracer) {
    case 1: return occupancy_sed_nt<T, 1>();
    case 2: return occupancy_sed_nt<T, 2>();
    case 3: return occupancy_sed_nt<T, 3>();
    case 4: return occupancy_sed_nt<T, 4>();
    case 5: return occupancy_sed_nt<T, 5>();
    case 6: return occupancy_sed_nt<T, 6>();
    case 7: return occupancy_sed_nt<T, 7>();
    case 8: return occupancy_sed_nt<T, 8>();
    default: return 0;
  }
}

// Without tracers the mixture is the dry gas, and the kernels are the ones of
// stage_dry_f64.hip / stage_dry_f32.hip, so that no other translation unit
// instantiates them.
template <typename T>
int launch_dry(bool hllc, bool d3, const StageArgs& a, int nblocks, hipStream_t st) {
  if constexpr (sizeof(T) == 8)
    return launch_stage_dry_f64(hllc, d3, a, nblocks, st);
  else
    return launch_stage_dry_f32(hllc, d3, a, nblocks, st);
}

template <typename T>
int occupancy_dry(bool hllc, bool d3) {
  if constexpr (sizeof(T) == 8)
    return occupancy_dry_f64(hllc, d3);
  else
    return occupancy_dry_f32(hllc, d3);
}

// Workgroups of the stage kernel that fit on one compute unit (0 if unknown).
template <typename T, bool MIX, bool HLLC = false>
int occupancy_t(int ntracer, bool d3, bool half) {
  switch (ntracer) {
    case 0: return occupancy_dry<T>(HLLC, d3);
    case 1: return occupancy_nt<T, 1, MIX, HLLC>(d3, half);
    case 2: return occupancy_nt<T, 2, MIX, HLLC>(d3, half);
    case 3: return occupancy_nt<T, 3, MIX, HLLC>(d3, half);
    case 4: return occupancy_nt<T, 4, MIX, HLLC>(d3, half);
    case 5: return occupancy_nt<T, 5, MIX, HLLC>(d3, half);
    case 6: return occupancy_nt<T, 6, MIX, HLLC>(d3, half);
    case 7: return occupancy_nt<T, 7, MIX, HLLC>(d3, half);
    case 8: return occupancy_nt<T, 8, MIX, HLLC>(d3, half);
    default: return 0;
  }
}

template <typename T, bool MIX, bool HLLC = false>
int launch_stage_t(int ntracer, bool d3, const StageArgs& a, int nblocks, hipStream_t st) {
  switch (ntracer) {
    case 0: return launch_dry<T>(HLLC, d3, a, nblocks, st);
    case 1: return launch_nt<T, 1, MIX, HLLC>(d3, a, nblocks, st);
    case 2: return launch_nt<T, 2, MIX, HLLC>(d3, a, nblocks, st);
    case 3: return launch_nt<T, 3, MIX, HLLC>(d3, a, nblocks, st);
    case 4: return launch_nt<T, 4, MIX, HLLC>(d3, a, nblocks, st);
    case 5: return launch_nt<T, 5, MIX, HLLC>(d3, a, nblocks, st);
    case 6: return launch_nt<T, 6, MIX, HLLC>(d3, a, nblocks, st);
    case 7: return launch_nt<T, 7, MIX, HLLC>(d3, a, nblocks, st);
    case 8: return launch_nt<T, 8, MIX, HLLC>(d3, a, nblocks, st);
    default: return -1;
  }
}

template <typename T, int NT>
TileShape tile_nt(bool d3, bool mix, bool half) {
  using P = Tile3For<T, NT, false>;
  using F = TileFor<T, NT>;
  return d3 && !mix && !half ? TileShape{P::TX, P::TY} : TileShape{F::TX, F::TY};
}

template <typename T>
TileShape tile_t(int nv, bool d3, bool mix, bool half) {
  switch (nv - 5) {
    case 0: return tile_nt<T, 0>(d3, mix, half);
    case 1: return tile_nt<T, 1>(d3, mix, half);
    case 2: return tile_nt<T, 2>(d3, mix, half);
    case 3: return tile_nt<T, 3>(d3, mix, half);
    case 4: return tile_nt<T, 4>(d3, mix, half);
    case 5: return tile_nt<T, 5>(d3, mix, half);
    case 6: return tile_nt<T, 6>(d3, mix, half);
    case 7: return tile_nt<T, 7>(d3, mix, half);
    default: return tile_nt<T, 8>(d3, mix, half);
  }
}

}  // namespace snap
