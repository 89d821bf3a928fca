// Launcher of the four-lanes-per-orbit DOP853 kernels (lane_quad.h).
#include "lane_quad.h"

namespace chx {

namespace {
template <class S>
hipError_t go(bool adaptive, const StepArgs &a, hipStream_t s) {
  const unsigned grid = (unsigned)((a.n + 15) / 16);
  if (adaptive)
    hipLaunchKernelGGL((lane_quad_rka_kernel<S>), dim3(grid), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((lane_quad_rk_kernel<S>), dim3(grid), dim3(64), 0, s, a);
  return hipGetLastError();
}
}  // namespace

// The SALI pair alone, the square-root LD, and an ensemble whose quads give
// each of the 1,024 SIMDs at most two wavefronts (n = 32,768), for the double
// pendulum one (n = 16,384: its stages issue enough to fill a SIMD, and
// repeating the trigonometry in four lanes costs more).  Measured, one lane
// against four: Henon-Heiles adaptive, T = 40: n = 4,096 1.77 / 0.81 ms,
// 16,384 1.80 / 0.87, 32,768 2.18 / 1.56, 65,536 2.51 / 2.68; fixed step,
// 1,000 steps: 4.69 / 1.46, 4.74 / 1.63, 4.82 / 2.68, 4.83 / 4.78; quartic
// N = 3 adaptive: 2.48 / 1.01, 2.54 / 1.13, 2.57 / 1.74, 2.63 / 2.94; double
// pendulum fixed: 2.15 / 1.57, 2.24 / 1.81, 2.36 / 3.10, adaptive 1.82 / 1.16,
// 1.93 / 1.33, 2.01 / 2.07.
bool lane_quad_wanted(int sys, const StepArgs &a) {
  if (a.m_s != 2 || a.n_l != 0 || ((a.ind & CHX_IND_LD) && a.ld_p != 0.5)) return false;
  return a.n <= (sys == SYS_DP ? 16384 : 32768);
}

hipError_t launch_lane_quad(int sys, int ndof, bool adaptive, const StepArgs &a, hipStream_t s) {
  switch (sys) {
  case SYS_HH: return go<SysHH>(adaptive, a, s);
  case SYS_QUARTIC:
    return ndof == 1 ? go<SysQuartic<1>>(adaptive, a, s)
         : ndof == 2 ? go<SysQuartic<2>>(adaptive, a, s) : go<SysQuartic<3>>(adaptive, a, s);
  case SYS_HARMONIC:
    return ndof == 1 ? go<SysHarmonic<1>>(adaptive, a, s)
         : ndof == 2 ? go<SysHarmonic<2>>(adaptive, a, s) : go<SysHarmonic<3>>(adaptive, a, s);
  case SYS_DP: return go<SysDP>(adaptive, a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace chx
