// Device evaluation of travelling-wave boundary values (kernels_wave.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "lbmhpde.h"

namespace lbm {

// One instance's rows, and where they go.
struct WaveRows {
  double* rows;
  double dx, dt;
  lbm_wave w;
  int n, ip, ir;   // nodes; the exponents p and r where they are whole numbers, else -1
};
WaveRows wave_rows(double* rows, int n, double dx, double dt, const lbm_wave& w);
// rows[s * 2 layers + k] = phi*(x_node(k), w.t0 + (s + 1) dt) of wave w for
// s < steps, k < 2 layers (node k for k < layers, else n - 2 layers + k); a
// device array of steps * 2 layers doubles, for each of `count` instances.  The
// waves must be valid.
hipError_t launch_wave_rows(const WaveRows* w, int count, int64_t steps, int layers, hipStream_t s);

}  // namespace lbm
