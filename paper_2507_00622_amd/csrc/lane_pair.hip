// Launcher of the two-lanes-per-orbit Yoshida-4 kernels (lane_pair.h).
#include "lane_pair.h"

namespace chx {

namespace {
template <class S>
hipError_t go(const StepArgs &a, hipStream_t s) {
  hipLaunchKernelGGL((lane_pair_kernel<S>), dim3((unsigned)((a.n + 31) / 32)), dim3(64), 0, s, a);
  return hipGetLastError();
}
}  // namespace

// The SALI pair alone, the square-root LD, and at most 32,768 orbits: one
// wavefront of pairs per SIMD.  Measured, Henon-Heiles, 4,000 steps, one lane
// against two: with energy n = 8,192 0.92 / 0.84 ms, 32,768 1.35 / 1.26,
// 65,536 1.77 / 2.04; with the LD 1.21 / 1.07, 1.33 / 1.26, 1.43 / 1.95;
// 796 orbits, LD, 20,000 steps 6.1 / 4.0 ms.  With one degree of freedom and no
// LD a step is too short to share: quartic N = 1, 1,500 steps, n = 500 0.307 /
// 0.326 ms, 32,000 0.364 / 0.385.
bool lane_pair_wanted(int ndof, const StepArgs &a) {
  if (ndof == 1 && !(a.ind & CHX_IND_LD)) return false;
  return a.m_s == 2 && a.n_l == 0 && !((a.ind & CHX_IND_LD) && a.ld_p != 0.5) && a.n <= 32768;
}

hipError_t launch_lane_pair(int sys, int ndof, const StepArgs &a, hipStream_t s) {
  switch (sys) {
  case SYS_HH: return go<SysHH>(a, s);
  case SYS_QUARTIC:
    return ndof == 1 ? go<SysQuartic<1>>(a, s)
         : ndof == 2 ? go<SysQuartic<2>>(a, s) : go<SysQuartic<3>>(a, s);
  case SYS_HARMONIC:
    return ndof == 1 ? go<SysHarmonic<1>>(a, s)
         : ndof == 2 ? go<SysHarmonic<2>>(a, s) : go<SysHarmonic<3>>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace chx
