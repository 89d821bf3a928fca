// lane_row.h -- small ensembles of the lane systems with three or more
// deviation vectors: a 16-lane row per orbit, lane v holding vector v
// (Yoshida-4 and fixed-step DOP853).
//
// One lane per orbit integrates its M vectors in turn, and a small ensemble is
// paced by that one lane's instruction stream.  Here a lane has one vector.
// Yoshida-4: every lane also integrates the state and takes half of the LD's
// roots, even lanes those of the momenta, odd lanes those of the force.
// DOP853: lane 15 holds the state, whose stages reach the row by
// row_newbcast.  Gram-Schmidt: once pivot l is normalised it goes from lane l to the
// row by row_newbcast, and every later lane projects it out.
// Every value takes the operations of the one-lane kernel in their order: the
// results have the same bits, so a subset of an ensemble may cross from one
// kernel to the other.
//
// Bound: the chain of one lane's step (state, one vector), an FP64 instruction
// about every 6.5 cycles from a wavefront alone on its SIMD.  Henon-Heiles, 4,000
// orbits, SALI, GALI_2, four exponents, LD and energy: 2,000 Yoshida-4 steps
// 0.95 -> 0.75 ms, 500 DOP853 steps 3.63 -> 1.18 ms; more beside lane_row_wanted.
#pragma once
#include "fput_row.h"
#include "lane_quad.h"

namespace chx {

namespace lanerow {

// Vectors of a row at a checkpoint: the SALI/GALI set back to unit length,
// SALI, Gram-Schmidt of the Lyapunov set (LaneOrbit::checkpoint).
// y: this lane's vector (v < M) or anything; returns SALI^2.
template <int D>
__device__ __forceinline__ double vectors(const StepArgs &a, int v, int M, double (&y)[D],
                                          double &gm, int &ge, bool do_sali) {
  using fputrow::bcast;
  const int m_s = a.m_s;
  auto norm2 = [&]() {
    double r2 = 0.0;
#pragma unroll
    for (int c = 0; c < D; ++c) r2 = __builtin_fma(y[c], y[c], r2);
    return r2;
  };
  if (v < m_s) {
    const double r2 = norm2();
    const double inv = rsqrt_nr(r2);
#pragma unroll
    for (int c = 0; c < D; ++c) y[c] *= inv;
    grow(gm, ge, r2);
  }
  double s2 = 0.0;
  if (do_sali) {
    double sp = 0.0, sm = 0.0;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      const double u = bcast<0>(y[c]), z = bcast<1>(y[c]);
      const double ap = u + z, am = u - z;
      sp = __builtin_fma(ap, ap, sp);
      sm = __builtin_fma(am, am, sm);
    }
    s2 = __builtin_fmin(sp, sm);
  }
  fputrow::static_for<0, 12>([&](auto lc) {
    constexpr int l = decltype(lc)::value;
    if (l >= m_s && l < M) {
      if (v == l) {
        const double r2 = norm2();
        const double inv = rsqrt_nr(r2);
#pragma unroll
        for (int c = 0; c < D; ++c) y[c] *= inv;
        grow(gm, ge, r2);
      }
      double p[D];
#pragma unroll
      for (int c = 0; c < D; ++c) p[c] = bcast<l>(y[c]);
      if (v > l && v < M) {
        double d = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) d = __builtin_fma(p[c], y[c], d);
#pragma unroll
        for (int c = 0; c < D; ++c) y[c] = __builtin_fma(-d, p[c], y[c]);
      }
    }
  });
  return s2;
}

// What the rest of a checkpoint at t decides and keeps, from the state x
// (equal in every lane); false when the orbit stops.  O: the accumulators.
template <class S, class O>
__device__ __forceinline__ bool decide(const StepArgs &a, double t, const double *x, O &o,
                                       bool escaped, bool do_sali, double s2) {
  constexpr int N = S::N;
  if (do_sali) {
    o.slast2 = s2;
    o.smin2 = __builtin_fmin(o.smin2, s2);
    if (s2 < a.thr2 && __builtin_isnan(o.tch)) o.tch = t;
  }
  if (a.ind & CHX_IND_ENERGY) {
    double e;
    if constexpr (has_hamiltonian<S>::value) {
      e = __builtin_fabs(S::hamiltonian(x, a.prm) - o.H0);
    } else {
      double kin = 0.0;
#pragma unroll
      for (int r = 0; r < N; ++r) kin = __builtin_fma(x[N + r], x[N + r], kin);
      e = __builtin_fabs(__builtin_fma(0.5, kin, S::potential(x, a.prm)) - o.H0);
    }
    o.eerr = __builtin_fmax(o.eerr, e);
  }
  if (escaped) {
    o.st = CHX_ORBIT_ESCAPED;
    return false;
  }
  if (a.early_exit && do_sali && s2 < a.thr2) {
    o.st = CHX_ORBIT_EXITED;
    return false;
  }
  return true;
}
template <class S>
__device__ __forceinline__ bool finite_state(const double *x) {
  bool finite = true;
#pragma unroll
  for (int c = 0; c < 2 * S::N; ++c) finite = finite && __builtin_isfinite(x[c]);
  return finite;
}
template <class S>
__device__ __forceinline__ bool has_escaped(const StepArgs &a, const double *x) {
  if (!(a.escape_r2 > 0.0)) return false;
  double r2 = 0.0;
#pragma unroll
  for (int r = 0; r < S::N; ++r) r2 = __builtin_fma(x[r], x[r], r2);
  return r2 > a.escape_r2;
}

}  // namespace lanerow

template <class S>
struct RowOrbit : LaneOrbit<S, 1, false, -1> {
  using Base = LaneOrbit<S, 1, false, -1>;
  using Base::D;
  using Base::F;
  using Base::N;
  using Base::w;
  using Base::x;
  int v, M;

  __device__ static __forceinline__ double other(double u) {
    return __builtin_amdgcn_update_dpp(0.0, u, 0xB1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
  }
  __device__ void load(const StepArgs &a, int64_t i) {
    v = threadIdx.x & 15;
    M = a.m_s + a.n_l;
    const int64_t k = v < M ? v : M - 1;  // the rest repeat the last vector
    StepArgs b = a;
    b.w = a.w + k * D * a.pitch;
    b.gm = a.gm + k * a.pitch;
    b.ge = a.ge + k * a.pitch;
    Base::load(b, i);
  }
  __device__ void store(const StepArgs &a, int64_t i) const {
    const int64_t P = a.pitch;
    if (v < M) {
#pragma unroll
      for (int c = 0; c < D; ++c) a.w[((int64_t)v * D + c) * P + i] = w[0][c];
      a.gm[v * P + i] = this->gm[0];
      a.ge[v * P + i] = this->ge[0];
    }
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
    const bool momenta = (v & 1) == 0;
    double sum = 0.0;  // this lane's roots: the momenta's or the force's
    this->kick_state(k.hk0);
    this->kick_vectors(a, k.hk0);
    for (int s = 0; s + 1 < blk; ++s) {
      Base::step_body(a, k);
      if (do_ld) {
#pragma unroll
        for (int r = 0; r < N; ++r) add_sqrt_ld(momenta ? x[N + r] : F[r], sum);
      }
      this->kick_state(k.hk0);  // first kick of the next step
      this->kick_vectors(a, k.hkm);
    }
    Base::step_body(a, k);
    if (do_ld) {
      double g = 0.0;
#pragma unroll
      for (int r = 0; r < N; ++r) add_sqrt_ld(momenta ? x[N + r] : F[r], g);
      this->ld_block(k, sum + other(sum), g + other(g));
    }
    this->kick_vectors(a, k.hk0);
  }
  __device__ bool checkpoint(const StepArgs &a, double t) {
    this->tend = t;
    if (!lanerow::finite_state<S>(x)) {
      this->st = CHX_ORBIT_NONFINITE;
      return false;
    }
    const bool escaped = lanerow::has_escaped<S>(a, x);
    const bool do_sali = (a.ind & CHX_IND_SALI) != 0;
    const double s2 = lanerow::vectors(a, v, M, w[0], this->gm[0], this->ge[0], do_sali);
    return lanerow::decide<S>(a, t, x, *this, escaped, do_sali, s2);
  }
};

template <class S>
struct RowRK {
  static constexpr int N = S::N, D = 2 * N, SL = 15;  // SL: the state's lane
  static constexpr bool GEN = has_hamiltonian<S>::value;
  double y[D];  // lanes v < M: vector v; lane 15: the state
  double gm;
  int ge;
  double ld, smin2, slast2, tch, eerr, H0, tend;
  int st, v, M;
  bool state;

  __device__ void load(const StepArgs &a, int64_t i) {
    v = threadIdx.x & 15;
    M = a.m_s + a.n_l;
    state = v == SL;
    const int64_t k = v < M ? v : M - 1, P = a.pitch;
    const double *src = state ? a.x : a.w + k * D * P;
#pragma unroll
    for (int c = 0; c < D; ++c) y[c] = src[c * P + i];
    gm = a.gm[k * P + i];
    ge = a.ge[k * P + i];
    ld = a.sc[SC_LD * P + i];
    smin2 = a.sc[SC_SALI_MIN2 * P + i];
    slast2 = a.sc[SC_SALI_LAST2 * P + i];
    tch = a.sc[SC_T_CHAOS * P + i];
    eerr = a.sc[SC_EERR * P + i];
    H0 = a.sc[SC_H0 * P + i];
    tend = a.sc[SC_T_END * P + i];
    st = CHX_ORBIT_OK;
  }
  __device__ void store(const StepArgs &a, int64_t i) const {
    const int64_t P = a.pitch;
    if (state || v < M) {
      double *dst = state ? a.x : a.w + (int64_t)v * D * P;
#pragma unroll
      for (int c = 0; c < D; ++c) dst[c * P + i] = y[c];
    }
    if (v < M) {
      a.gm[v * P + i] = gm;
      a.ge[v * P + i] = ge;
    }
    if (state) {
      a.sc[SC_LD * P + i] = ld;
      a.sc[SC_SALI_MIN2 * P + i] = smin2;
      a.sc[SC_SALI_LAST2 * P + i] = slast2;
      a.sc[SC_T_CHAOS * P + i] = tch;
      a.sc[SC_EERR * P + i] = eerr;
      a.sc[SC_T_END * P + i] = tend;
      a.st[i] = st;
    }
  }
  // one fixed step of size h
  __device__ __forceinline__ void rk_step(const StepArgs &a, double h, bool do_ld) {
    using fputrow::bcast;
    const dop853::Coef cf = dop853::coef();
    double k[12][D], g = 0.0;
    dop853::static_for<0, 12>([&](auto ic) {
      quad::stage<S, decltype(ic)::value>(a, cf, h, do_ld, y, state, k, g,
                                          [](double u) { return bcast<SL>(u); });
    });
#pragma unroll
    for (int c = 0; c < D; ++c) y[c] += dop853::final_sum(cf, k, c);
    if (do_ld) ld = __builtin_fma(h, bcast<SL>(g), ld);
  }
  __device__ bool checkpoint(const StepArgs &a, double t) {
    using fputrow::bcast;
    tend = t;
    double x[D];
#pragma unroll
    for (int c = 0; c < D; ++c) x[c] = bcast<SL>(y[c]);
    if (!lanerow::finite_state<S>(x)) {
      st = CHX_ORBIT_NONFINITE;
      return false;
    }
    const bool escaped = lanerow::has_escaped<S>(a, x);
    const bool do_sali = (a.ind & CHX_IND_SALI) != 0;
    const double s2 = lanerow::vectors(a, v, M, y, gm, ge, do_sali);
    return lanerow::decide<S>(a, t, x, *this, escaped, do_sali, s2);
  }
};

// Four orbits per wavefront; rows beyond the ensemble or already stopped do
// nothing (all lanes of a row take the same branch).
template <class S>
__global__ void __launch_bounds__(64) lane_row_kernel(const StepArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 4);
  if (i >= a.n) return;
  if (a.st[i] != CHX_ORBIT_OK) return;
  RowOrbit<S> o;
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
  o.store(a, i);
}

template <class S>
__global__ void __launch_bounds__(64) lane_row_rk_kernel(const StepArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 4);
  if (i >= a.n) return;
  if (a.st[i] != CHX_ORBIT_OK) return;
  RowRK<S> o;
  o.load(a, i);
  const bool do_ld = (a.ind & CHX_IND_LD) != 0;
  int64_t s = a.s_begin;
  const int64_t K = a.K;
  while (s < a.s_end) {
    int64_t next = (s / K + 1) * K;
    if (next > a.n_total) next = a.n_total;
    for (int64_t j = s; j < next; ++j) o.rk_step(a, a.dt, do_ld);
    s = next;
    if (!o.checkpoint(a, (double)s * a.dt)) break;
  }
  o.store(a, i);
}

}  // namespace chx
