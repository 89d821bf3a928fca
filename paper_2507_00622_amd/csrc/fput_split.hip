// Launcher of the row-per-vector FPU kernels, Yoshida-4.
#include "fput_split.h"

namespace chx {

namespace {
template <int N>
hipError_t go(const StepArgs &a, hipStream_t s) {
  if (a.m_s == 2)
    hipLaunchKernelGGL((fput_split_kernel<N, 2>), dim3((unsigned)((a.n + 1) / 2)), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((fput_split_kernel<N, 4>), dim3((unsigned)a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}
}  // namespace

// Two to four SALI/GALI vectors, no Lyapunov set, and at most 2,048 orbits: up
// to two wavefronts of the split rows per SIMD (half that with two vectors).
// Measured, one row against a row per vector: N = 11, four vectors, adaptive,
// T = 20: n = 1,000 2.79 / 1.59 ms, 2,048 2.94 / 2.30, 4,096 3.09 / 3.40;
// Yoshida-4, 4,000 steps: 2.08 / 1.32, 2.23 / 2.12, 2.29 / 3.53; N = 16, two
// vectors, adaptive: 1.63 / 1.23, 1.61 / 1.25, 1.78 / 1.88; Yoshida-4: 1.37 /
// 1.21, 1.40 / 1.23, 1.59 / 2.00.  With three vectors the fourth row repeats one,
// and Yoshida-4 stops at one wavefront per SIMD (1,200 steps, microseconds: N = 3,
// n = 1,500 587 / 660, 2,040 590 / 674; N = 6, 640 / 692, 644 / 686).
bool fput_split_wanted(bool rk, const StepArgs &a) {
  if (a.n_l != 0 || a.m_s < 2 || a.m_s > 4) return false;
  return a.n <= (a.m_s == 3 && !rk ? 1024 : 2048);
}

hipError_t launch_fput_split(int ndof, const StepArgs &a, hipStream_t s) {
  switch (ndof) {
  case 2: return go<2>(a, s);
  case 3: return go<3>(a, s);
  case 4: return go<4>(a, s);
  case 5: return go<5>(a, s);
  case 6: return go<6>(a, s);
  case 7: return go<7>(a, s);
  case 8: return go<8>(a, s);
  case 9: return go<9>(a, s);
  case 10: return go<10>(a, s);
  case 11: return go<11>(a, s);
  case 12: return go<12>(a, s);
  case 13: return go<13>(a, s);
  case 14: return go<14>(a, s);
  case 15: return go<15>(a, s);
  case 16: return go<16>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace chx
