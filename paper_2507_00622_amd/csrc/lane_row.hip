// Launcher of the row-per-orbit kernels of the lane systems (lane_row.h).
#include "lane_row.h"

namespace chx {

namespace {
template <class S, bool RK>
hipError_t go(const StepArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)((a.n + 3) / 4));
  if constexpr (RK)
    hipLaunchKernelGGL((lane_row_rk_kernel<S>), grid, dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((lane_row_kernel<S>), grid, dim3(64), 0, s, a);
  return hipGetLastError();
}
template <bool RK>
hipError_t dispatch(int sys, int ndof, const StepArgs &a, hipStream_t s) {
  switch (sys) {
  case SYS_HH: return go<SysHH, RK>(a, s);
  case SYS_QUARTIC:
    return ndof == 1 ? go<SysQuartic<1>, RK>(a, s)
         : ndof == 2 ? go<SysQuartic<2>, RK>(a, s) : go<SysQuartic<3>, RK>(a, s);
  case SYS_HARMONIC:
    return ndof == 1 ? go<SysHarmonic<1>, RK>(a, s)
         : ndof == 2 ? go<SysHarmonic<2>, RK>(a, s) : go<SysHarmonic<3>, RK>(a, s);
  case SYS_DP:
    if constexpr (RK) return go<SysDP, RK>(a, s);
  }
  return hipErrorInvalidValue;
}
}  // namespace

// Three to twelve vectors (lanes 12..14 stay idle, lane 15 is DOP853's state)
// and the LD's roots split in halves only for p = 1/2.  The line: a row takes
// 16 lanes where the one-lane kernel takes one, so it is ahead while its wavefronts,
// four orbits each, find a SIMD of their own (4,096 orbits), and DOP853, whose
// rows shorten the step by more, also with two (8,192).  Milliseconds, one lane
// per orbit against a row:
//                                          n = 4000     8192         16384
//   Yoshida-4, Henon-Heiles, M = 6         0.95  0.75   1.01  1.08   1.06  2.13
//              quartic N = 3, M = 3        1.01  0.82   1.06  1.34   1.11  2.56
//              quartic N = 3, M = 12       2.56  1.53   2.59  2.11   2.61  2.89
//   DOP853,    Henon-Heiles, M = 6         3.63  1.18   3.70  1.99   3.71  3.58
//              quartic N = 3, M = 3        3.93  1.30   3.50  2.20   3.55  4.16
//              quartic N = 3, M = 12       12.1  2.22   11.9  2.28   11.8  4.28
//              double pendulum, M = 6      13.8  4.01   14.0  7.16   13.9  13.8
// A checkpoint's pivots go through the row one after another, which a Yoshida-4
// row makes up for between checkpoints if they are K (N - 1) >= 5 steps and
// degrees of freedom apart.  One lane against a row, 4,000 orbits, 1,000 steps
// (microseconds): M = 3, Henon-Heiles K = 1 723 / 914, 2 527 / 598, 4 420 / 433,
// harmonic N = 3 K = 1 743 / 841, 2 528 / 558; M = 4 (400 steps), quartic N = 1
// K = 1 373 / 506, 5 251 / 265, 10 234 / 233; Henon-Heiles M = 6 K = 5 353 / 318.
bool lane_row_wanted(int ndof, bool rk, const StepArgs &a) {
  const int M = a.m_s + a.n_l;
  if (!rk && (int64_t)a.K * (ndof - 1) < 5) return false;
  if (M < 3 || M > 12 || ((a.ind & CHX_IND_LD) && a.ld_p != 0.5)) return false;
  return a.n <= (rk ? 8192 : 4096);
}

hipError_t launch_lane_row(int sys, int ndof, bool rk, const StepArgs &a, hipStream_t s) {
  return rk ? dispatch<true>(sys, ndof, a, s) : dispatch<false>(sys, ndof, a, s);
}

}  // namespace chx
