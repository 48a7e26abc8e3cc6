// Stage kernels with the HLLC Riemann solver, passive tracers, element type float.
#include "stage_launch.h"

namespace snap {

int launch_stage_hllc_f32(int ntracer, bool d3, StageArgs a, int nblocks, hipStream_t st) {
  return launch_stage_t<float, false, true>(ntracer, d3, a, nblocks, st);
}

int occupancy_hllc_f32(int ntracer, bool d3, bool half) {
  return occupancy_t<float, false, true>(ntracer, d3, half);
}

}  // namespace snap
