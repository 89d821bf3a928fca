// lane_pair.h -- Yoshida-4 for small ensembles with the SALI pair: two lanes
// per orbit.
//
// One lane per orbit leaves a small ensemble on a few wavefronts, each alone
// on its SIMD and paced by one lane's instruction stream (the state, two
// vectors, the LD's 2N roots).  Here both lanes of a pair integrate the
// state, lane v carries vector v, and each takes half of the LD's roots (lane
// 0 those of the momenta, lane 1 those of the force), their sums exchanged by
// DPP once per checkpoint.  Every
// value takes the operations of the one-lane kernel in their order: the
// results have the same bits, so a subset of an ensemble may cross from one
// kernel to the other.
#pragma once
#include "lane_kernel.h"

namespace chx {

// M = 1: the lane's own vector is w[0]; the base's checkpoint is not used.
template <class S>
struct PairOrbit : LaneOrbit<S, 1, false, -1> {
  using Base = LaneOrbit<S, 1, false, -1>;
  using Base::D;
  using Base::F;
  using Base::N;
  using Base::x;
  using Base::w;
  int v;  // lane of the pair = its vector

  __device__ static __forceinline__ double other(double u) {
    return __builtin_amdgcn_update_dpp(0.0, u, 0xB1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
  }
  __device__ void load(const StepArgs &a, int64_t i) {
    v = threadIdx.x & 1;
    StepArgs b = a;
    b.w = a.w + (int64_t)v * D * a.pitch;
    b.gm = a.gm + (int64_t)v * a.pitch;
    b.ge = a.ge + (int64_t)v * a.pitch;
    Base::load(b, i);
  }
  __device__ void store(const StepArgs &a, int64_t i) const {
    const int64_t P = a.pitch;
#pragma unroll
    for (int c = 0; c < D; ++c) a.w[((int64_t)v * D + c) * P + i] = w[0][c];
    a.gm[v * P + i] = this->gm[0];
    a.ge[v * P + i] = this->ge[0];
    if (v == 0) {
#pragma unroll
      for (int c = 0; c < D; ++c) a.x[c * P + i] = x[c];
      a.sc[SC_LD * P + i] = this->ld;
      a.sc[SC_GPREV * P + i] = this->gprev;
      a.sc[SC_SALI_MIN2 * P + i] = this->smin2;
      a.sc[SC_SALI_LAST2 * P + i] = this->slast2;
      a.sc[SC_T_CHAOS * P + i] = this->tch;
      a.sc[SC_EERR * P + i] = this->eerr;
      a.sc[SC_T_END * P + i] = this->tend;
      a.st[i] = this->st;
    }
  }
  __device__ void block(const StepArgs &a, const StepCoef &k, int blk) {
    const bool do_ld = (a.ind & CHX_IND_LD) != 0;
    double sum = 0.0;  // this lane's roots: the momenta's or the force's
    this->kick_state(k.hk0);
    this->kick_vectors(a, k.hk0);
    for (int s = 0; s + 1 < blk; ++s) {
      Base::step_body(a, k);
      if (do_ld) {
#pragma unroll
        for (int r = 0; r < N; ++r) add_sqrt_ld(v == 0 ? x[N + r] : F[r], sum);
      }
      this->kick_state(k.hk0);  // first kick of the next step
      this->kick_vectors(a, k.hkm);
    }
    Base::step_body(a, k);
    if (do_ld) {
      double g = 0.0;
#pragma unroll
      for (int r = 0; r < N; ++r) add_sqrt_ld(v == 0 ? x[N + r] : F[r], g);
      this->ld_block(k, sum + other(sum), g + other(g));
    }
    this->kick_vectors(a, k.hk0);
  }
  // Checkpoint at t (LaneOrbit::checkpoint); the decisions are taken on
  // values equal in both lanes.
  __device__ bool checkpoint(const StepArgs &a, double t) {
    this->tend = t;
    bool finite = true;
#pragma unroll
    for (int c = 0; c < D; ++c) finite = finite && __builtin_isfinite(x[c]);
    if (!finite) {
      this->st = CHX_ORBIT_NONFINITE;
      return false;
    }
    bool escaped = false;
    if (a.escape_r2 > 0.0) {
      double r2 = 0.0;
#pragma unroll
      for (int r = 0; r < N; ++r) r2 = __builtin_fma(x[r], x[r], r2);
      escaped = r2 > a.escape_r2;
    }
    this->unit_set(1);
    double s2 = 0.0;
    const bool do_sali = (a.ind & CHX_IND_SALI) != 0;
    if (do_sali) {
      double sp = 0.0, sm = 0.0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const double o = other(w[0][c]);
        const double u = v == 0 ? w[0][c] : o, z = v == 0 ? o : w[0][c];
        const double ap = u + z, am = u - z;
        sp = __builtin_fma(ap, ap, sp);
        sm = __builtin_fma(am, am, sm);
      }
      s2 = __builtin_fmin(sp, sm);
      this->slast2 = s2;
      this->smin2 = __builtin_fmin(this->smin2, s2);
      if (s2 < a.thr2 && __builtin_isnan(this->tch)) this->tch = t;
    }
    if (a.ind & CHX_IND_ENERGY) {
      double kin = 0.0;
#pragma unroll
      for (int r = 0; r < N; ++r) kin = __builtin_fma(x[N + r], x[N + r], kin);
      const double e =
          __builtin_fabs(__builtin_fma(0.5, kin, S::potential(x, a.prm)) - this->H0);
      this->eerr = __builtin_fmax(this->eerr, e);
    }
    if (escaped) {
      this->st = CHX_ORBIT_ESCAPED;
      return false;
    }
    if (a.early_exit && do_sali && s2 < a.thr2) {
      this->st = CHX_ORBIT_EXITED;
      return false;
    }
    return true;
  }
};

// 32 orbits per wavefront; both lanes of a pair take the same branches.
template <class S>
__global__ void __launch_bounds__(64) lane_pair_kernel(const StepArgs a) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 1;
  if (i >= a.n) return;
  if (a.st[i] != CHX_ORBIT_OK) return;
  PairOrbit<S> o;
  o.load(a, i);
  const StepCoef k(a.dt);
  int64_t s = a.s_begin;
  const int64_t K = a.K;
  while (s < a.s_end) {
    int64_t next = (s / K + 1) * K;
    if (next > a.n_total) next = a.n_total;
    o.block(a, k, (int)(next - s));
    s = next;
    if (!o.checkpoint(a, (double)s * a.dt)) break;
  }
  int64_t j = i;
  asm volatile("" : "+v"(j));
  o.store(a, j);
}

}  // namespace chx
