// Launcher of the row-per-vector FPU kernels, adaptive DOP8(5).
#include "fput_split.h"

namespace chx {

namespace {
template <int N>
hipError_t go(const StepArgs &a, hipStream_t s) {
  if (a.m_s == 2)
    hipLaunchKernelGGL((fput_split_rka_kernel<N, 2>), dim3((unsigned)((a.n + 1) / 2)), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((fput_split_rka_kernel<N, 4>), dim3((unsigned)a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_fput_split_rka(int ndof, const StepArgs &a, hipStream_t s) {
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
