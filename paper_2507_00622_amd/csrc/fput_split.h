// fput_split.h -- FPU chains with two to four SALI/GALI vectors in small
// ensembles: R 16-lane rows per orbit (R = 2 for two vectors, 4 for three or
// four), each row carrying the whole state and one of the vectors.
//
// The component rows (fput_crow.h, fput_crow_rk.h) give an orbit one row, which
// integrates the state and then one vector after the other: a thousand orbits
// are 250 wavefronts, each alone on a SIMD and paced by its own instruction
// stream.  With a row per vector the stream is the state's and one vector's,
// and the two interleave: for the Runge-Kutta solvers a vector's stage follows
// the state's stage at once, so no stiffnesses are kept.  The state is
// computed R times over by rows that would be idle.
//
// Every component takes the operations of the component rows in their
// order.  The adaptive solver's error sums run over the state's and then
// each vector's terms lane by lane before the row sum, so the rows
// exchange their terms through LDS and every row forms the same sums: the
// results have the same bits, and every decision is the same in all rows
// of an orbit.
#pragma once
#include "fput_crow_rk.h"

namespace chx {

template <int N, int R>
struct CRowSplit : CRowRK<N, 1> {
  using B = CRowRK<N, 1>;
  using O = CRowOrbit<N, 1>;
  using B::dp;
  using B::dq;
  using B::eerr;
  using B::H0;
  using B::lane;
  using B::ld;
  using B::mass;
  using B::p;
  using B::q;
  using B::row;
  using B::slast2;
  using B::smin2;
  using B::st;
  using B::tch;
  using B::tend;
  int v, m;    // this row's vector, the orbit's vectors (v >= m: none)
  int first;   // lane `lane` of the orbit's first row

  __device__ void load(const StepArgs &a, int64_t o, int vectors) {
    B::init_lane();
    m = vectors;
    v = row % R;
    first = (row - v) * 16 + lane;
    // the vector rows of v >= m repeat the last vector and store nothing
    const int64_t k = v < m ? v : m - 1;
    StepArgs b = a;
    b.w = a.w + k * 2 * N * a.pitch;
    b.gm = a.gm + k * a.pitch;
    b.ge = a.ge + k * a.pitch;
    O::load(b, o);
  }
  __device__ void store(const StepArgs &a, int64_t o) const {
    const int64_t P = a.pitch;
    if (mass && v == 0) {
      a.x[lane * P + o] = q;
      a.x[(N + lane) * P + o] = p;
    }
    if (mass && v < m) {
      a.w[((int64_t)v * 2 * N + lane) * P + o] = dq[0];
      a.w[((int64_t)v * 2 * N + N + lane) * P + o] = dp[0];
    }
    if (lane == 0 && v < m) {
      a.gm[v * P + o] = this->gm[0];
      a.ge[v * P + o] = this->ge[0];
    }
    if (lane == 0 && v == 0) {
      a.sc[SC_LD * P + o] = ld;
      a.sc[SC_GPREV * P + o] = this->gprev;
      a.sc[SC_SALI_MIN2 * P + o] = smin2;
      a.sc[SC_SALI_LAST2 * P + o] = slast2;
      a.sc[SC_T_CHAOS * P + o] = tch;
      a.sc[SC_EERR * P + o] = eerr;
      a.sc[SC_T_END * P + o] = tend;
      a.st[o] = st;
    }
  }

  // the 12 stages of the state and of this row's vector, stage by stage
  __device__ __forceinline__ void stages(const StepArgs &a, dop853::Coef cf, double h, bool do_ld,
                                         double (&kq)[12][1], double (&kp)[12][1],
                                         double (&vq)[12][1], double (&vp)[12][1], double &g) {
    using namespace fputrow;
    dop853::static_for<0, 12>([&](auto ic) {
      constexpr int I = decltype(ic)::value;
      const double Yq = q + dop853::stage_sum<I>(cf, kq, 0);
      const double Yp = p + dop853::stage_sum<I>(cf, kp, 0);
      const double Vq = dq[0] + dop853::stage_sum<I>(cf, vq, 0);
      const double Vp = dp[0] + dop853::stage_sum<I>(cf, vp, 0);
      double F, kl, kr;
      O::spring_terms(a, Yq, mass, F, kl, kr);
      if constexpr (dop853::B[I] != 0.0) {
        if (do_ld) g = __builtin_fma(dop853::B[I], mass ? sqrt_ld(Yp) + sqrt_ld(F) : 0.0, g);
      }
      kq[I][0] = h * Yp;
      kp[I][0] = -h * F;
      const double ql = dpp<0x111>(Vq);  // row_shr:1
      const double qr = dpp<0x101>(Vq);  // row_shl:1
      double hq = (kl + kr) * Vq;
      hq = __builtin_fma(-kl, ql, hq);
      hq = __builtin_fma(-kr, qr, hq);
      vq[I][0] = h * Vp;
      vp[I][0] = -h * hq;
    });
  }

  __device__ __forceinline__ void rk_step(const StepArgs &a, double h, bool do_ld) {
    const dop853::Coef cf = dop853::coef();
    double kq[12][1], kp[12][1], vq[12][1], vp[12][1], g = 0.0;
    stages(a, cf, h, do_ld, kq, kp, vq, vp, g);
    q += dop853::final_sum(cf, kq, 0);
    p += dop853::final_sum(cf, kp, 0);
    if (do_ld) ld = __builtin_fma(h, fputrow::row_sum(g), ld);
    dq[0] += dop853::final_sum(cf, vq, 0);
    dp[0] += dop853::final_sum(cf, vp, 0);
  }

  // The scaled error terms of one component (dop853::err_terms before the
  // squares).
  __device__ __forceinline__ static void ratios(const StepArgs &a, dop853::Coef cf, const double (&k)[12][1],
                                                double y, double yn, double sb, double &r5,
                                                double &r3) {
    const double sk = __builtin_fma(
        a.rtol, __builtin_fmax(__builtin_fabs(y), __builtin_fabs(yn)), a.atol);
    r5 = dop853::err5_sum(cf, k, 0) / sk;
    r3 = (sb - dop853::BHH1 * k[0][0] - dop853::BHH2 * k[8][0] - dop853::BHH3 * k[11][0]) / sk;
  }

  // One attempted step of size h (CRowRK::rk_attempt); ex: this wavefront's
  // exchange buffer [4][64] in LDS.
  __device__ __forceinline__ double rk_attempt(const StepArgs &a, double h, bool do_ld,
                                               double (*ex)[64], double &qn, double &pn,
                                               double &dqn, double &dpn, double &ldn) {
    const dop853::Coef cf = dop853::coef();
    double kq[12][1], kp[12][1], vq[12][1], vp[12][1], g = 0.0;
    stages(a, cf, h, do_ld, kq, kp, vq, vp, g);
    const double sq = dop853::final_sum(cf, kq, 0), sp = dop853::final_sum(cf, kp, 0);
    qn = q + sq;
    pn = p + sp;
    const double tq = dop853::final_sum(cf, vq, 0), tp = dop853::final_sum(cf, vp, 0);
    dqn = dq[0] + tq;
    dpn = dp[0] + tp;
    ldn = do_ld ? __builtin_fma(h, fputrow::row_sum(g), ld) : ld;
    double s5q, s3q, s5p, s3p, v5q, v3q, v5p, v3p;
    ratios(a, cf, kq, q, qn, sq, s5q, s3q);
    ratios(a, cf, kp, p, pn, sp, s5p, s3p);
    ratios(a, cf, vq, dq[0], dqn, tq, v5q, v3q);
    ratios(a, cf, vp, dp[0], dpn, tp, v5p, v3p);
    // one wavefront, whose LDS accesses execute in program order
    const int tid = threadIdx.x;
    wave_sync();
    ex[0][tid] = v5q;
    ex[1][tid] = v5p;
    ex[2][tid] = v3q;
    ex[3][tid] = v3p;
    wave_sync();
    double e5 = __builtin_fma(s5p, s5p, __builtin_fma(s5q, s5q, 0.0));
    double e3 = __builtin_fma(s3p, s3p, __builtin_fma(s3q, s3q, 0.0));
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int t = first + 16 * j;
      const double a5 = ex[0][t], b5 = ex[1][t], a3 = ex[2][t], b3 = ex[3][t];
      if (j < m) {
        e5 = __builtin_fma(b5, b5, __builtin_fma(a5, a5, e5));
        e3 = __builtin_fma(b3, b3, __builtin_fma(a3, a3, e3));
      }
    }
    // ghost lanes are no components
    e5 = fputrow::row_sum(mass ? e5 : 0.0);
    e3 = fputrow::row_sum(mass ? e3 : 0.0);
    const double deno = __builtin_fma(0.01, e3, e5);
    if (!(deno > 0.0)) return deno == 0.0 ? 0.0 : deno;  // NaN stays NaN
    return e5 / sqrt((double)(2 * N * (1 + m)) * deno);
  }
  __device__ __forceinline__ static void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // Checkpoint at t (CRowOrbit::checkpoint without a Lyapunov set); returns
  // false when the orbit stops.
  __device__ bool checkpoint(const StepArgs &a, double t) {
    using namespace fputrow;
    tend = t;
    const bool bad = !(__builtin_isfinite(q) && __builtin_isfinite(p));
    if ((__ballot(bad) >> (16 * row)) & 0xFFFFull) {
      st = CHX_ORBIT_NONFINITE;
      return false;
    }
    bool escaped = false;
    if (a.escape_r2 > 0.0) escaped = row_sum(q * q) > a.escape_r2;
    {
      const double r2 = row_sum(__builtin_fma(dq[0], dq[0], dp[0] * dp[0]));
      const double inv = rsqrt_nr(r2);
      dq[0] *= inv;
      dp[0] *= inv;
      grow(this->gm[0], this->ge[0], r2);
    }
    double s2 = 0.0;
    const bool do_sali = (a.ind & CHX_IND_SALI) != 0;
    if (do_sali) {
      const double q0 = __shfl(dq[0], first), p0 = __shfl(dp[0], first);
      const double q1 = __shfl(dq[0], first + 16), p1 = __shfl(dp[0], first + 16);
      const double aq = q0 + q1, ap = p0 + p1;
      const double bq = q0 - q1, bp = p0 - p1;
      const double sp = row_sum(__builtin_fma(aq, aq, ap * ap));
      const double sm = row_sum(__builtin_fma(bq, bq, bp * bp));
      s2 = __builtin_fmin(sp, sm);
      slast2 = s2;
      smin2 = __builtin_fmin(smin2, s2);
      if (s2 < a.thr2 && __builtin_isnan(tch)) tch = t;
    }
    if (a.ind & CHX_IND_ENERGY) {
      const double kk = a.prm[0], al = a.prm[1], be = a.prm[2];
      const double ql = dpp<0x111>(q);
      const double qr = dpp<0x101>(q);
      const double dl = q - ql, dr = qr - q;
      auto spring = [&](double d) {
        const double d2 = d * d;
        return d2 * __builtin_fma(d, __builtin_fma(0.25 * be, d, al * (1.0 / 3.0)), 0.5 * kk);
      };
      double e = (lane <= N) ? spring(dl) : 0.0;
      if (mass) e = __builtin_fma(0.5 * p, p, e);
      if (N == 16 && lane == 15) e += spring(dr);
      eerr = __builtin_fmax(eerr, __builtin_fabs(row_sum(e) - H0));
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

// One 64-thread block is 4 / R orbits; orbits beyond the ensemble or already
// stopped do nothing (all their rows take the same branch).
template <int N, int R>
__global__ void __launch_bounds__(64) fput_split_kernel(const StepArgs a) {
  const int64_t o = (int64_t)blockIdx.x * (4 / R) + (threadIdx.x >> 4) / R;
  if (o >= a.n) return;
  if (a.st[o] != CHX_ORBIT_OK) return;
  CRowSplit<N, R> r;
  r.load(a, o, a.m_s);
  const StepCoef k(a.dt);
  int64_t s = a.s_begin;
  const int64_t K = a.K;
  while (s < a.s_end) {
    int64_t next = (s / K + 1) * K;
    if (next > a.n_total) next = a.n_total;
    r.block(a, k, (int)(next - s));
    s = next;
    if (!r.checkpoint(a, (double)s * a.dt)) break;
  }
  r.store(a, o);
}

template <int N, int R>
__global__ void __launch_bounds__(64) fput_split_rk_kernel(const StepArgs a) {
  const int64_t o = (int64_t)blockIdx.x * (4 / R) + (threadIdx.x >> 4) / R;
  if (o >= a.n) return;
  if (a.st[o] != CHX_ORBIT_OK) return;
  CRowSplit<N, R> r;
  r.load(a, o, a.m_s);
  const bool do_ld = (a.ind & CHX_IND_LD) != 0;
  int64_t s = a.s_begin;
  const int64_t K = a.K;
  while (s < a.s_end) {
    int64_t next = (s / K + 1) * K;
    if (next > a.n_total) next = a.n_total;
    for (int64_t j = s; j < next; ++j) r.rk_step(a, a.dt, do_ld);
    s = next;
    if (!r.checkpoint(a, (double)s * a.dt)) break;
  }
  r.store(a, o);
}

// The loop of fput_crow_rka_kernel, one per orbit.
template <int N, int R>
__global__ void __launch_bounds__(64) fput_split_rka_kernel(const StepArgs a) {
  __shared__ double ex[4][64];
  const int64_t o = (int64_t)blockIdx.x * (4 / R) + (threadIdx.x >> 4) / R;
  if (o >= a.n) return;
  if (a.st[o] != CHX_ORBIT_OK) return;
  CRowSplit<N, R> r;
  r.load(a, o, a.m_s);
  const int64_t P = a.pitch;
  double h = a.sc[SC_H * P + o];
  if (!(h > 0.0)) h = a.dt;  // the first step
  bool rej = a.sc[SC_REJ * P + o] != 0.0;
  double nacc = a.sc[SC_NACC * P + o], nrej = a.sc[SC_NREJ * P + o];
  double emax = a.sc[SC_ERR_MAX * P + o], elast = a.sc[SC_ERR_LAST * P + o];
  const bool do_ld = (a.ind & CHX_IND_LD) != 0;
  int64_t s = a.s_begin;
  const int64_t K = a.K;
  while (s < a.s_end) {
    int64_t next = (s / K + 1) * K;
    if (next > a.n_total) next = a.n_total;
    double t = (double)s * a.dt;
    const double tb = (double)next * a.dt;
    int attempts = 0, fail = CHX_ORBIT_OK;
    while (t < tb) {
      double hh = h;
      bool last = false;
      if (t + 1.01 * hh >= tb) {
        hh = tb - t;
        last = true;
      }
      double qn, pn, dqn, dpn, ldn;
      const double err = r.rk_attempt(a, hh, do_ld, ex, qn, pn, dqn, dpn, ldn);
      const bool lane_bad = !(__builtin_isfinite(qn) && __builtin_isfinite(pn));
      const bool bad = ((__ballot(lane_bad) >> (16 * r.row)) & 0xFFFFull) != 0;
      if (bad || !__builtin_isfinite(err) || !__builtin_isfinite(ldn)) {
        fail = CHX_ORBIT_NONFINITE;
        break;
      }
      if (++attempts > dop853::MAX_ATTEMPTS) {
        fail = CHX_ORBIT_STEP_FAILED;
        break;
      }
      const double qf = sqrt(sqrt(sqrt(err)));
      double fac = qf / dop853::SAFE;
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
        r.q = qn;
        r.p = pn;
        r.dq[0] = dqn;
        r.dp[0] = dpn;
        r.ld = ldn;
        t = last ? tb : t + hh;
      } else {
        h = hh / fac;
        rej = true;
        nrej += 1.0;
      }
    }
    if (fail != CHX_ORBIT_OK) {
      r.st = fail;
      break;
    }
    s = next;
    if (!r.checkpoint(a, tb)) break;
  }
  r.store(a, o);
  if (r.lane == 0 && r.v == 0) {
    a.sc[SC_H * P + o] = h;
    a.sc[SC_REJ * P + o] = rej ? 1.0 : 0.0;
    a.sc[SC_NACC * P + o] = nacc;
    a.sc[SC_NREJ * P + o] = nrej;
    a.sc[SC_ERR_MAX * P + o] = emax;
    a.sc[SC_ERR_LAST * P + o] = elast;
  }
}

}  // namespace chx
