// lane_quad.h -- DOP853 (fixed step and adaptive) for small ensembles with
// the SALI pair: four lanes per orbit.
//
// One lane per orbit leaves a small ensemble on a few wavefronts, each alone
// on its SIMD and paced by the latency of one lane's instruction stream:
// the state's twelve stages, then each vector's.  Here lane 0 of a quad holds
// the state, lane 1 the first and lane 2 the second vector (lane 3 repeats
// lane 2 and stores nothing), and the three pass through the stages together:
// every lane sums its own object's stage derivatives, the state's stage goes
// to the quad by DPP (quad_perm), and each lane keeps the derivative that is
// its own, h f(Y) or h Df(Y) dY.  Nothing passes through LDS.  Every
// component is computed by the operations of the one-lane kernel in their
// order, and so are the error sums over the components (lane 0's, then 1's,
// then 2's, handed on by DPP): the results have the same bits.
//
// Bound: instruction issue and latency at one wavefront per SIMD.  About 900
// instructions per attempt against 2,000 for a lane that does all three
// objects.
#pragma once
#include "lane_rk.h"

namespace chx {

namespace quad {

// one component's contributions to dop853::err_terms, before they are squared
// and summed
template <int D2>
__device__ __forceinline__ void err_ratios(dop853::Coef cf, const double (&k)[12][D2], int c, double y, double yn,
                                           double sb, double rtol, double atol, double &r5,
                                           double &r3) {
  const double sk = __builtin_fma(rtol, __builtin_fmax(__builtin_fabs(y), __builtin_fabs(yn)),
                                  atol);
  r5 = dop853::err5_sum(cf, k, c) / sk;
  r3 = (sb - dop853::BHH1 * k[0][c] - dop853::BHH2 * k[8][c] - dop853::BHH3 * k[11][c]) / sk;
}

template <int CTRL>
__device__ __forceinline__ double qp(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, CTRL, 0xf, 0xf, true);
}
// lane L of each quad to the whole quad
template <int L>
__device__ __forceinline__ double from(double v) {
  return qp<L * 0x55>(v);
}

// Stage I of an orbit's objects, one per lane: k_I = h times the object's
// derivative at Y = y + sum_j a_Ij k_j, where the state's lane gives the state's
// stage to the others (from_state); the LD integrand of the state into
// g (the state's lane has the orbit's).
template <class S, int I, int D, class F>
__device__ __forceinline__ void stage(const StepArgs &a, dop853::Coef cf, double h, bool do_ld,
                                      const double (&y)[D], bool state, double (&k)[12][D],
                                      double &g, F &&from_state) {
  constexpr int N = S::N;
  double Y[D];
#pragma unroll
  for (int c = 0; c < D; ++c) Y[c] = y[c] + dop853::stage_sum<I>(cf, k, c);
  double f[D];  // the state's lane: f(Y)
  if constexpr (has_hamiltonian<S>::value) {
    double X[D], dY[1][D], df[1][D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      X[c] = from_state(Y[c]);
      dY[0][c] = Y[c];
    }
    S::template rhs_multi<1>(X, dY, f, df, a.prm);
#pragma unroll
    for (int c = 0; c < D; ++c) k[I][c] = h * (state ? f[c] : df[0][c]);
  } else {
    double q[N], F_[N], Hs[S::NH];
#pragma unroll
    for (int r = 0; r < N; ++r) q[r] = from_state(Y[r]);
    S::force(q, F_, a.prm);
    S::hess_scaled(q, h, Hs, a.prm);
#pragma unroll
    for (int r = 0; r < N; ++r) {
      double s = 0.0;
#pragma unroll
      for (int j = 0; j < N; ++j) s = __builtin_fma(Hs[hidx(N, r, j)], Y[j], s);
      f[r] = Y[N + r];
      f[N + r] = -F_[r];
      k[I][r] = h * Y[N + r];
      k[I][N + r] = state ? h * f[N + r] : -s;
    }
  }
  if constexpr (dop853::B[I] != 0.0) {
    if (do_ld) {
      double gi = 0.0;
      if constexpr (has_hamiltonian<S>::value) {
#pragma unroll
        for (int c = 0; c < D; ++c) gi += sqrt_ld(f[c]);
      } else {
#pragma unroll
        for (int r = 0; r < N; ++r) gi += sqrt_ld(f[r]) + sqrt_ld(f[N + r]);
      }
      g = __builtin_fma(dop853::B[I], gi, g);
    }
  }
  // each stage finishes before the next: run ahead, the value chain of
  // all twelve would keep every stage's intermediates live
#pragma unroll
  for (int c = 0; c < D; ++c) asm volatile("" : "+v"(k[I][c]));
}

}  // namespace quad

template <class S>
struct QuadRK {
  static constexpr int N = S::N, D = 2 * N;
  static constexpr bool GEN = has_hamiltonian<S>::value;
  double y[D];  // lane 0: the state; lanes 1, 2 (and 3): a deviation vector
  double gm;    // growth of this lane's vector
  int ge;
  double ld, smin2, slast2, tch, eerr, H0, tend;  // the orbit's, in every lane
  int st;
  int role;     // lane within the quad
  bool state;   // role 0

  __device__ void load(const StepArgs &a, int64_t i) {
    role = threadIdx.x & 3;
    state = role == 0;
    const int v = role == 1 ? 0 : 1;
    const int64_t P = a.pitch;
    const double *src = state ? a.x : a.w + (int64_t)v * D * P;
#pragma unroll
    for (int c = 0; c < D; ++c) y[c] = src[c * P + i];
    gm = a.gm[v * P + i];
    ge = a.ge[v * P + i];
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
    if (role < 3) {
      const int v = role == 1 ? 0 : 1;
      double *dst = state ? a.x : a.w + (int64_t)v * D * P;
#pragma unroll
      for (int c = 0; c < D; ++c) dst[c * P + i] = y[c];
      if (!state) {
        a.gm[v * P + i] = gm;
        a.ge[v * P + i] = ge;
      }
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
    const dop853::Coef cf = dop853::coef();
    double k[12][D], g = 0.0;
    dop853::static_for<0, 12>(
        [&](auto ic) { quad::stage<S, decltype(ic)::value>(a, cf, h, do_ld, y, state, k, g, quad::from<0>); });
#pragma unroll
    for (int c = 0; c < D; ++c) y[c] += dop853::final_sum(cf, k, c);
    if (do_ld) ld = __builtin_fma(h, quad::from<0>(g), ld);
  }

  // one attempted step of size h (RKOrbit::rk_attempt): this lane's new
  // object in yn, the new LD in ldn; returns the orbit's error estimate
  __device__ __forceinline__ double rk_attempt(const StepArgs &a, double h, bool do_ld,
                                               double (&yn)[D], double &ldn) {
    using namespace quad;
    const dop853::Coef cf = dop853::coef();
    double k[12][D], g = 0.0;
    dop853::static_for<0, 12>(
        [&](auto ic) { quad::stage<S, decltype(ic)::value>(a, cf, h, do_ld, y, state, k, g, quad::from<0>); });
    ldn = do_ld ? __builtin_fma(h, from<0>(g), ld) : ld;
    double r5[D], r3[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      const double sb = dop853::final_sum(cf, k, c);
      yn[c] = y[c] + sb;
      err_ratios(cf, k, c, y[c], yn[c], sb, a.rtol, a.atol, r5[c], r3[c]);
    }
    // the sums run over the state's components, then each vector's: every
    // lane adds its own to what the lane before handed on
    double e5 = 0.0, e3 = 0.0;
    dop853::static_for<0, 3>([&](auto lc) {
      constexpr int L = decltype(lc)::value;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        e5 = __builtin_fma(r5[c], r5[c], e5);
        e3 = __builtin_fma(r3[c], r3[c], e3);
      }
      e5 = from<L>(e5);
      e3 = from<L>(e3);
    });
    const double deno = __builtin_fma(0.01, e3, e5);
    if (!(deno > 0.0)) return deno == 0.0 ? 0.0 : deno;  // NaN stays NaN
    return e5 / sqrt((double)(D * 3) * deno);
  }

  // Checkpoint at t (LaneOrbit::checkpoint); returns false when the orbit
  // stops.  Every decision is taken on values equal in all four lanes.
  __device__ bool checkpoint(const StepArgs &a, double t) {
    using namespace quad;
    tend = t;
    double x[D];
    bool finite = true;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      x[c] = from<0>(y[c]);
      finite = finite && __builtin_isfinite(x[c]);
    }
    if (!finite) {
      st = CHX_ORBIT_NONFINITE;
      return false;
    }
    bool escaped = false;
    if (a.escape_r2 > 0.0) {
      double r2 = 0.0;
#pragma unroll
      for (int r = 0; r < N; ++r) r2 = __builtin_fma(x[r], x[r], r2);
      escaped = r2 > a.escape_r2;
    }
    double r2 = 0.0;
#pragma unroll
    for (int c = 0; c < D; ++c) r2 = __builtin_fma(y[c], y[c], r2);
    const double inv = rsqrt_nr(r2);
    if (!state) {
#pragma unroll
      for (int c = 0; c < D; ++c) y[c] *= inv;
      grow(gm, ge, r2);
    }
    double s2 = 0.0;
    const bool do_sali = (a.ind & CHX_IND_SALI) != 0;
    if (do_sali) {
      double sp = 0.0, sm = 0.0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const double u = from<1>(y[c]), v = from<2>(y[c]);
        const double ap = u + v, am = u - v;
        sp = __builtin_fma(ap, ap, sp);
        sm = __builtin_fma(am, am, sm);
      }
      s2 = __builtin_fmin(sp, sm);
      slast2 = s2;
      smin2 = __builtin_fmin(smin2, s2);
      if (s2 < a.thr2 && __builtin_isnan(tch)) tch = t;
    }
    if (a.ind & CHX_IND_ENERGY) {
      double e;
      if constexpr (GEN) {
        e = __builtin_fabs(S::hamiltonian(x, a.prm) - H0);
      } else {
        double kin = 0.0;
#pragma unroll
        for (int r = 0; r < N; ++r) kin = __builtin_fma(x[N + r], x[N + r], kin);
        e = __builtin_fabs(__builtin_fma(0.5, kin, S::potential(x, a.prm)) - H0);
      }
      eerr = __builtin_fmax(eerr, e);
    }
    if (escaped) {
      st = CHX_ORBIT_ESCAPED;
      return false;
    }
    if (a.early_exit && do_sali && s2 < a.thr2) {
      st = CHX_ORBIT_EXITED;
      return false;
    }
    return true;
  }
};

// 16 orbits per wavefront; quads beyond the ensemble or already stopped do
// nothing (all four lanes take the same branch).
template <class S>
__global__ void __launch_bounds__(64) lane_quad_rk_kernel(const StepArgs a) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
  if (i >= a.n) return;
  if (a.st[i] != CHX_ORBIT_OK) return;
  QuadRK<S> o;
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
  int64_t ob = i;
  asm volatile("" : "+v"(ob));
  o.store(a, ob);
}

// The adaptive solver: the loop of lane_rka_kernel, one per quad.
template <class S>
__global__ void __launch_bounds__(64) lane_quad_rka_kernel(const StepArgs a) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
  if (i >= a.n) return;
  if (a.st[i] != CHX_ORBIT_OK) return;
  constexpr int D = 2 * S::N;
  QuadRK<S> o;
  o.load(a, i);
  const int64_t P = a.pitch;
  double h = a.sc[SC_H * P + i];
  if (!(h > 0.0)) h = a.dt;  // the first step
  bool rej = a.sc[SC_REJ * P + i] != 0.0;
  double nacc = a.sc[SC_NACC * P + i], nrej = a.sc[SC_NREJ * P + i];
  double emax = a.sc[SC_ERR_MAX * P + i], elast = a.sc[SC_ERR_LAST * P + i];
  const bool do_ld = (a.ind & CHX_IND_LD) != 0;
  const int64_t K = a.K;
  int64_t s = a.s_begin;
  int64_t next = (s / K + 1) * K;
  if (next > a.n_total) next = a.n_total;
  double t = (double)s * a.dt;
  double tb = (double)next * a.dt;
  int attempts = 0;
  while (s < a.s_end) {
    if (t >= tb) {
      s = next;
      if (!o.checkpoint(a, tb)) break;
      if (s >= a.s_end) break;
      next = (s / K + 1) * K;
      if (next > a.n_total) next = a.n_total;
      t = tb;
      tb = (double)next * a.dt;
      attempts = 0;
    }
    double hh = h;
    bool last = false;
    if (t + 1.01 * hh >= tb) {
      hh = tb - t;
      last = true;
    }
    double yn[D], ldn;
    const double err = o.rk_attempt(a, hh, do_ld, yn, ldn);
    bool mine = true;
#pragma unroll
    for (int c = 0; c < D; ++c) mine = mine && __builtin_isfinite(yn[c]);
    // the state's lane decides (a vector's overflow shows in err)
    const bool finite = __builtin_isfinite(err) && __builtin_isfinite(ldn) &&
                        ((__ballot(mine) >> (threadIdx.x & 60)) & 1ull);
    if (!finite) {
      o.st = CHX_ORBIT_NONFINITE;
      break;
    }
    if (++attempts > dop853::MAX_ATTEMPTS) {
      o.st = CHX_ORBIT_STEP_FAILED;
      break;
    }
    const double q = sqrt(sqrt(sqrt(err)));
    double fac = q / dop853::SAFE;
    if (fac > dop853::FACC1) fac = dop853::FACC1;
    if (err <= 1.0) {
      if (fac < dop853::FACC2) fac = dop853::FACC2;
      double hnew = hh / fac;
      if (rej && hnew > hh) hnew = hh;
      rej = false;
      h = hnew;
      nacc += 1.0;
      emax = fmax(emax, err);
      elast = err;
#pragma unroll
      for (int c = 0; c < D; ++c) o.y[c] = yn[c];
      o.ld = ldn;
      t = last ? tb : t + hh;
    } else {
      h = hh / fac;
      rej = true;
      nrej += 1.0;
    }
  }
  int64_t ob = i;
  asm volatile("" : "+v"(ob));
  o.store(a, ob);
  if (o.state) {
    a.sc[SC_H * P + ob] = h;
    a.sc[SC_REJ * P + ob] = rej ? 1.0 : 0.0;
    a.sc[SC_NACC * P + ob] = nacc;
    a.sc[SC_NREJ * P + ob] = nrej;
    a.sc[SC_ERR_MAX * P + ob] = emax;
    a.sc[SC_ERR_LAST * P + ob] = elast;
  }
}

}  // namespace chx
