// The windkessel model's Kalman filter (Sec. 3.1.1, Alg. 1 reduced to one
// dimension: every Cholesky factor is a square root), batched over filters,
// in FP64.  Runs over many intervals come in two forms, one wave per filter
// with the intervals spread over its lanes (kf_wave) and one lane per filter:
//   k_kf_run          whole runs over t = 1..T (the exact likelihood)
//   k_kf_proposal     SMC over the parameters with attached Kalman filters:
//                     each proposal's filter over t_{0:i-1}
//   k_kf_advance      every attached filter over t_{i-1:i}
//   k_smc2_accept_kf  the Metropolis-Hastings decision with those filters
//   k_kf_pmmh         marginal Metropolis-Hastings chains on (R, C, Z,
//                     sigma^2) with the exact likelihood
#include <math.h>

#include "pf_device.hpp"
#include "pf_kalman.hpp"

namespace pfk {

// One interval: K predictions m <- a m + c q_{n-1}, V <- a^2 V + sigma_p^2,
// then the correction with y_t; returns ell_t.
__device__ __forceinline__ double kf_interval(const double* th, const KfArgs& A, int t, double& m,
                                              double& V) {
  const double a = th[0], c = th[1], Z = th[2], sp = th[3];
  for (int s = 1; s <= A.K; ++s) {
    const int64_t n = (int64_t)(t - 1) * A.K + s;
    m = a * m + c * A.q[n - 1];
    V = a * a * V + sp * sp;
  }
  const double qn = A.q[(int64_t)t * A.K];
  const double v = A.obs[t - 1] - (m + Z * qn);
  const double S = V + A.R;
  const double e = -0.5 * (log(2.0 * 3.14159265358979323846 * S) + v * v / S);
  const double Kg = V / S;
  m = m + Kg * v;
  V = (1.0 - Kg) * V;
  return e;
}

// ---------------------------------------------------------------- a filter over a wave's lanes
// A run of T intervals by one wave, KF_L consecutive intervals per lane and
// 64 KF_L per pass.  The lane-per-filter form is a chain of T (2 K + a
// logarithm and two divisions) dependent steps, about 0.74 us per interval
// with the scalar loads of the flow on its path, while a batch of hundreds of
// filters fills a few lanes of a few CUs.  The chain breaks into parts that
// do not depend on each other or compose associatively:
//   - K predictions are m <- a^K m + c g_t, V <- a^{2K} V + C2, with
//     g_t = sum_s a^{K-1-s} q_{tK+s} depending on the flow alone and C2 the
//     same for every interval;
//   - prediction and correction take the variance to V' = R P / (P + R),
//     P = a^{2K} V + C2: a fractional-linear map with the same matrix
//     [[R a^{2K}, R C2], [a^{2K}, C2 + R]] at every interval, so a lane's
//     first variance is a power of that matrix applied to the pass's first
//     (powers by squaring; the entries are non-negative, so nothing cancels
//     and each squaring perturbs the map by an ulp of its entries);
//   - given the gains the mean's maps m' = alpha m + beta compose by a wave
//     scan.
//   - the composed maps round a stationary gain the same way at every interval,
//     which adds up over a series.  Its complement is kept in two parts; in
//     series of several passes, where that is not enough, each lane also steps
//     its intervals from the mean that the scan gave it, and a second scan of
//     what that differs by corrects the lanes' first means.
// The logarithms and divisions then run in all lanes at once.  512 chains
// over T = 100, K = 10: 4.7 us an iteration against 74 a lane each (two waves per
// SIMD, still latency: two intervals per lane interleave); 512 likelihoods: 58
// us a call, most of it the copies of the results, against 148.  Both forms'
// arithmetic against 113-bit arithmetic, 500 parameter sets, the likelihood's
// mean relative error, this form / the chain / this form without either
// correction: T = 100, K = 10: 0.97e-15 / 3.6e-15 / 1.3e-15; T = 300: 0.77e-15 /
// 2.1e-15 / 5.1e-15; T = 2,000: 0.44e-15 / 1.6e-15 / 10e-15; K = 1: 3.8e-15 /
// 4.5e-15 / 6.0e-15 at T = 100, 1.3e-15 / 1.7e-15 / 32e-15 at T = 2,000.  Which
// form runs: kf_wave_form.
constexpr int KF_L = 2;
constexpr int KF_PASS = WAVE * KF_L;  // intervals of a pass

// Flow and observations in memory, or staged in LDS with the substeps as
// rows (lanes read consecutive entries).
struct KfSeriesMem {
  const double *qp, *yp;
  int K;
  __device__ __forceinline__ double q(int t, int s) const { return qp[(int64_t)t * K + s]; }
  __device__ __forceinline__ double q_end(int t) const { return qp[(int64_t)(t + 1) * K]; }
  __device__ __forceinline__ double y(int t) const { return yp[t]; }
};
struct KfSeriesLds {
  const double *qp, *yp;
  int ld;  // T + 1
  __device__ __forceinline__ double q(int t, int s) const { return qp[s * ld + t]; }
  __device__ __forceinline__ double q_end(int t) const { return qp[t + 1]; }
  __device__ __forceinline__ double y(int t) const { return yp[t]; }
};

// inclusive scan of the affine maps (a, b): lane l gets the composition of
// lanes 0..l's, first lane applied first
template <int CTRL, int ROWS>
__device__ __forceinline__ void affine_step(double& a, double& b) {
  const double pa = dpp_move<CTRL, ROWS>(a, 1.0), pb = dpp_move<CTRL, ROWS>(b, 0.0);
  b = __builtin_fma(a, pb, b);
  a = a * pa;
}
__device__ __forceinline__ void wave_affine_scan(double& a, double& b) {
  affine_step<0x111, 0xf>(a, b);
  affine_step<0x112, 0xf>(a, b);
  affine_step<0x114, 0xf>(a, b);
  affine_step<0x118, 0xf>(a, b);
  affine_step<0x142, 0xa>(a, b);
  affine_step<0x143, 0xc>(a, b);
}

// The log-likelihood of T intervals from N(m, V), every lane of the wave
// active; th uniform.  ell (or null) receives the T increments; m and V
// become the filtered mean and variance.  The result is the same in every
// lane.  SEVERAL: T may take more than one pass.
template <bool SEVERAL, class Series>
__device__ __forceinline__ double kf_wave(const double* th, int K, int T, double R,
                                          const Series& Q, double& m, double& V,
                                          double* __restrict__ ell) {
  const double a = th[0], c = th[1], Z = th[2], sp = th[3];
  const int lane = threadIdx.x & (WAVE - 1);
  // a^K as a sum of two doubles, and C2 with a^2 as one: the same rounding
  // error at every interval would add up where the substeps' own cancel
  double aK = 1.0, aKl = 0.0, C2 = 0.0;
  const double a2 = a * a, a2l = __builtin_fma(a, a, -a2), sp2 = sp * sp;
  for (int s = 0; s < K; ++s) {
    const double p = aK * a;
    aKl = __builtin_fma(aKl, a, __builtin_fma(aK, a, -p));
    aK = p;
    C2 = __builtin_fma(a2, C2, __builtin_fma(a2l, C2, sp2));
  }
  const double A2 = __builtin_fma(aK, aK, 2.0 * aK * aKl);
  // P[j]: the variance map of KF_L 2^j intervals, scaled by powers of two so
  // that nothing overflows
  const bool stable = __builtin_fabs(a) <= 1.0;
  double P[6][4];
  {
    double M[4] = {R * A2, R * C2, A2, C2 + R};
    const int e0 = -__builtin_amdgcn_frexp_exp((M[0] + M[1]) + (M[2] + M[3]));
#pragma unroll
    for (int p = 0; p < 4; ++p) M[p] = __builtin_ldexp(M[p], e0);
    auto square = [](const double(&x)[4], double(&r)[4]) {
      const double p0 = __builtin_fma(x[0], x[0], x[1] * x[2]);
      const double p1 = x[1] * (x[0] + x[3]);
      const double p2 = x[2] * (x[0] + x[3]);
      const double p3 = __builtin_fma(x[3], x[3], x[1] * x[2]);
      const int e = -__builtin_amdgcn_frexp_exp((p0 + p1) + (p2 + p3));
      r[0] = __builtin_ldexp(p0, e);
      r[1] = __builtin_ldexp(p1, e);
      r[2] = __builtin_ldexp(p2, e);
      r[3] = __builtin_ldexp(p3, e);
    };
    static_assert(KF_L == 2, "the first power is one squaring");
    square(M, P[0]);
#pragma unroll
    for (int j = 1; j < 6; ++j) square(P[j - 1], P[j]);
  }
  double tot = 0.0;
  for (int t0 = 0; t0 < T; t0 += KF_PASS) {
    const int tl = t0 + lane * KF_L;  // this lane's first interval
    double g[KF_L], y[KF_L], qe[KF_L];
#pragma unroll
    for (int e = 0; e < KF_L; ++e) {
      const int t = min(tl + e, T - 1);
      g[e] = 0.0;
      y[e] = Q.y(t);
      qe[e] = Q.q_end(t);
    }
#pragma unroll 4
    for (int s = 0; s < K; ++s)
#pragma unroll
      for (int e = 0; e < KF_L; ++e)
        g[e] = __builtin_fma(a, g[e], Q.q(min(tl + e, T - 1), s));
    // the variance at the lane's first interval
    double vx = V, vy = 1.0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const double nx = __builtin_fma(P[j][0], vx, P[j][1] * vy);
      const double ny = __builtin_fma(P[j][2], vx, P[j][3] * vy);
      const bool on = (lane >> j) & 1;
      vx = on ? nx : vx;
      vy = on ? ny : vy;
    }
    double Vl = vx / vy;
    // no circuit's a = exp(-h/(RC)) exceeds 1; for one that is given all the
    // same the powers' entries may spread beyond the exponent range: step by
    // step
    if (!stable) {
      Vl = V;
      for (int n = 0; n < lane * KF_L; ++n) {
        const double Pv = __builtin_fma(A2, Vl, C2);
        Vl = R * (Pv / (Pv + R));
      }
    }
    double S[KF_L], iS[KF_L], Kg[KF_L];
    double al = 1.0, be = 0.0;
#pragma unroll
    for (int e = 0; e < KF_L; ++e) {
      const bool in = tl + e < T;
      const double Pv = __builtin_fma(A2, Vl, C2);
      S[e] = Pv + R;
      iS[e] = 1.0 / S[e];
      Kg[e] = Pv * iS[e];
      const double rest = R * iS[e], rr = (1.0 - Kg[e]) - rest;  // 1 - Kg, in two parts
      Vl = in ? R * Kg[e] : Vl;
      g[e] = c * g[e];
      const double ae = __builtin_fma(aK, rest, __builtin_fma(aKl, rest, aK * rr));
      const double bb = __builtin_fma(
          rest, g[e], __builtin_fma(Kg[e], __builtin_fma(-Z, qe[e], y[e]), rr * g[e]));
      be = in ? __builtin_fma(ae, be, bb) : be;
      al = in ? ae * al : al;
    }
    double da = al;
    wave_affine_scan(al, be);
    const double mi = __builtin_fma(al, m, be);  // the mean after the lane's intervals
    double ml = wave_prev(mi, m);
    // (several passes) what the lane's intervals, stepped from that mean, make
    // of it, less the scan's: carried on by the same maps, it corrects the
    // lanes' first means
    auto innovation = [&](int e, double mean, double& mp) -> double {
      mp = __builtin_fma(aK, mean, __builtin_fma(aKl, mean, g[e]));
      return __builtin_fma(-Z, qe[e], y[e] - mp);
    };
    if constexpr (SEVERAL) {
      double x = ml, mp;
#pragma unroll
      for (int e = 0; e < KF_L; ++e) {
        const double v = innovation(e, x, mp);
        x = tl + e < T ? __builtin_fma(Kg[e], v, mp) : x;
      }
      double db = x - mi;
      wave_affine_scan(da, db);
      ml += wave_prev(db, 0.0);
    }
    double part = 0.0;
#pragma unroll
    for (int e = 0; e < KF_L; ++e) {
      const bool in = tl + e < T;
      double mp;
      const double v = innovation(e, ml, mp);
      const double le = -0.5 * (log(2.0 * 3.14159265358979323846 * S[e]) + v * v * iS[e]);
      ml = in ? __builtin_fma(Kg[e], v, mp) : ml;
      part += in ? le : 0.0;
      if (ell && in) ell[tl + e] = le;
    }
    tot = tot + wave_sum(part);
    const int last = min(WAVE - 1, (T - 1 - t0) / KF_L);  // the pass's last lane with intervals
    m = lane_value(ml, last);
    V = lane_value(Vl, last);
  }
  return tot;
}

template <bool SEVERAL>
__global__ __launch_bounds__(WAVE) void k_kf_run_wave(KfArgs A, const double* __restrict__ theta,
                                                      double* __restrict__ ll,
                                                      double* __restrict__ ell) {
  const int b = blockIdx.x;
  double th[6];
#pragma unroll
  for (int p = 0; p < 6; ++p) th[p] = theta[(int64_t)b * 8 + p];
  double m = th[4], V = th[5] * th[5];
  const double tot = kf_wave<SEVERAL>(th, A.K, A.T, A.R, KfSeriesMem{A.q, A.obs, A.K}, m, V,
                                      ell + (int64_t)b * A.T);
  if (threadIdx.x == 0) ll[b] = tot;
}

// The proposals' filters (k_kf_proposal), a wave each; i >= 2.
template <bool SEVERAL>
__global__ __launch_bounds__(WAVE) void k_kf_proposal_wave(KfArgs A, Smc2Args S,
                                                           const double* __restrict__ prop_dev,
                                                           double* __restrict__ prop_l,
                                                           double* __restrict__ prop_mV, int i) {
  const int j = blockIdx.x;
  if (!S.inside[j]) return;
  double th[6];
#pragma unroll
  for (int p = 0; p < 6; ++p) th[p] = prop_dev[(int64_t)j * 8 + p];
  double m = th[4], V = th[5] * th[5];
  const double tot =
      kf_wave<SEVERAL>(th, A.K, i - 1, A.R, KfSeriesMem{A.q, A.obs, A.K}, m, V, nullptr);
  if (threadIdx.x == 0) {
    prop_l[j] = tot;
    prop_mV[2 * j] = m;
    prop_mV[2 * j + 1] = V;
  }
}

// ---------------------------------------------------------------- a filter per lane
__global__ void k_kf_run(KfArgs A, const double* __restrict__ theta, double* __restrict__ ll,
                         double* __restrict__ ell) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= A.B) return;
  const double* th = theta + (int64_t)b * 8;
  double m = th[4], V = th[5] * th[5], tot = 0.0;
  for (int t = 1; t <= A.T; ++t) {
    const double e = kf_interval(th, A, t, m, V);
    ell[(int64_t)b * A.T + t - 1] = e;
    tot = tot + e;
  }
  ll[b] = tot;
}

// Proposal filters: from (m0', s0'^2) over t = 1..i-1 for the proposals
// inside the prior box.
__global__ void k_kf_proposal(KfArgs A, Smc2Args S, const double* __restrict__ prop_dev,
                              double* __restrict__ prop_l, double* __restrict__ prop_mV, int i) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= S.B || !S.inside[j]) return;
  const double* th = prop_dev + (int64_t)j * 8;
  double m = th[4], V = th[5] * th[5], lp = 0.0;
  for (int t = 1; t <= i - 1; ++t) lp = lp + kf_interval(th, A, t, m, V);
  prop_l[j] = lp;
  prop_mV[2 * j] = m;
  prop_mV[2 * j + 1] = V;
}

// Accept iff inside and log_alpha <= l' - l (ties accept); an accepted slot
// takes theta', its derived form, l' and the proposal's filter state.
__global__ void k_smc2_accept_kf(Smc2Args S, const double* __restrict__ log_alpha_row,
                                 const double* __restrict__ prop_dev,
                                 const double* __restrict__ prop_l,
                                 const double* __restrict__ prop_mV, int32_t* acc_tr_row) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= S.B) return;
  const int acc = S.inside[j] && (log_alpha_row[j] <= prop_l[j] - S.fs[j].loglik);
  S.accepted[j] = acc;
  if (acc_tr_row) acc_tr_row[j] = acc;
  if (!acc) return;
  S.accepts[j] += 1;
  for (int p = 0; p < S.n_theta; ++p)
    S.raw[(int64_t)j * S.n_theta + p] = S.prop_raw[(int64_t)j * S.n_theta + p];
  for (int p = 0; p < 8; ++p) S.theta_dev[(int64_t)j * 8 + p] = prop_dev[(int64_t)j * 8 + p];
  S.fs[j].loglik = prop_l[j];
  S.fs[j].status = 0;
  S.mV[2 * j] = prop_mV[2 * j];
  S.mV[2 * j + 1] = prop_mV[2 * j + 1];
}

// Every attached filter over t_{i-1:i}: the increment is the new
// theta-log-weight and adds to the likelihood.
__global__ void k_kf_advance(KfArgs A, Smc2Args S, int i) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= S.B) return;
  double m = S.mV[2 * j], V = S.mV[2 * j + 1];
  const double e = kf_interval(S.theta_dev + (int64_t)j * 8, A, i, m, V);
  S.mV[2 * j] = m;
  S.mV[2 * j + 1] = V;
  S.fs[j].loglik = S.fs[j].loglik + e;
  S.fs[j].t = i;
  S.ell_tr_w[(int64_t)j * S.T + i - 1] = e;
}

__global__ void k_kf_init(Smc2Args S) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= S.B) return;
  const double* th = S.theta_dev + (int64_t)j * 8;
  S.mV[2 * j] = th[4];
  S.mV[2 * j + 1] = th[5] * th[5];
}

// ---------------------------------------------------------------- chains on (R, C, Z, sigma^2)

// Phi(x) from the complementary error function (accurate in both tails).
__device__ __forceinline__ double ncdf(double x) { return 0.5 * erfc(-x * 0.70710678118654752440); }

// Model parameters from (R, C, Z, sigma^2) (Sec. 2.1.1): a = exp(-h/(R C)),
// c = R (1 - a), pressure noise sd c sigma, initial N(m0, s0^2); th[8] as
// the filters hold them.
__device__ __forceinline__ void wk_params(const pf_wk_mh& H, double h, const double* x,
                                          double* th) {
  const double a = exp(-h / (x[0] * x[1]));
  const double c = x[0] * (1.0 - a);
  th[0] = a;
  th[1] = c;
  th[2] = x[2];
  th[3] = c * sqrt(x[3]);
  th[4] = H.m0;
  th[5] = H.s0;
}

// ln p(R, C, Z, sigma^2) up to a constant: Gamma densities x^{k-1} e^{-x/s}
// and the Inverse-Gamma density x^{-alpha-1} e^{-beta/x}.
__device__ __forceinline__ double wk_log_prior(const pf_wk_mh& H, const double* x) {
  double lp = 0.0;
  for (int k = 0; k < 3; ++k) lp += (H.prior_shape[k] - 1.0) * log(x[k]) - x[k] / H.prior_scale[k];
  lp += -(H.ig_shape + 1.0) * log(x[3]) - H.ig_scale / x[3];
  return lp;
}

__device__ __forceinline__ double kf_loglik(const KfArgs& A, const double* th) {
  double m = th[4], V = th[5] * th[5], tot = 0.0;
  for (int t = 1; t <= A.T; ++t) tot = tot + kf_interval(th, A, t, m, V);
  return tot;
}

// One chain per wave through every iteration (k_kf_pmmh's steps and order of
// operations).  Lane l works on parameter l mod 4, so the proposals'
// distribution functions, logarithms and inverses of the four parameters are
// evaluated at once; the current state's terms are kept from one iteration to
// the next and follow an acceptance only.  The likelihood is kf_wave, with the
// series staged in LDS when it fits.
template <bool LDS, bool SEVERAL>
__global__ __launch_bounds__(WAVE) void k_kf_pmmh_wave(KfArgs A, pf_wk_mh H, double h,
                                                       int32_t iters,
                                                       const double* __restrict__ theta0,
                                                       const double* __restrict__ prop,
                                                       const double* __restrict__ alpha,
                                                       double* __restrict__ theta_trace,
                                                       double* __restrict__ ll_trace,
                                                       int32_t* __restrict__ accepts,
                                                       double* __restrict__ ll0) {
  extern __shared__ double series[];
  const int c = blockIdx.x, lane = threadIdx.x, k = lane & 3;
  const int T = A.T, K = A.K;
  if constexpr (LDS) {  // rows of T + 1: q_{tK+s} at [s][t], then y
    for (int n = lane; n <= T * K; n += WAVE) {
      const int t = n / K;
      series[(n - t * K) * (T + 1) + t] = A.q[n];
    }
    double* ys = series + (int64_t)K * (T + 1);
    for (int t = lane; t < T; t += WAVE) ys[t] = A.obs[t];
    __syncthreads();
  }
  auto loglik = [&](const double* th) -> double {
    double m = th[4], V = th[5] * th[5];
    if constexpr (LDS)
      return kf_wave<SEVERAL>(th, K, T, A.R,
                              KfSeriesLds{series, series + (int64_t)K * (T + 1), T + 1}, m, V,
                              nullptr);
    else
      return kf_wave<SEVERAL>(th, K, T, A.R, KfSeriesMem{A.q, A.obs, K}, m, V, nullptr);
  };
  // the sum over the parameters in their order
  auto sum4 = [&](double v) -> double {
    double r = 0.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) r += lane_value(v, p);
    return r;
  };
  auto params = [&](double v, double* th) {
    double w[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) w[p] = lane_value(v, p);
    wk_params(H, h, w, th);
  };
  auto prior_term = [&](double v) -> double {
    const double lv = log(v);
    if (k == 3) return -(H.ig_shape + 1.0) * lv - H.ig_scale / v;
    const double sh = k == 0 ? H.prior_shape[0] : k == 1 ? H.prior_shape[1] : H.prior_shape[2];
    const double sc = k == 0 ? H.prior_scale[0] : k == 1 ? H.prior_scale[1] : H.prior_scale[2];
    return (sh - 1.0) * lv - v / sc;
  };
  // this lane's proposal sd (0: fixed); sigma^2 moves by its factor
  const double sd = k == 0 ? H.step_sd[0] : k == 1 ? H.step_sd[1] : k == 2 ? H.step_sd[2] : 0.0;
  const bool gauss = sd > 0.0, ig = k == 3 && H.ig_prop_factor > 0.0;
  double th[8];
  double x = theta0[(int64_t)c * 4 + k];
  params(x, th);
  double ll = loglik(th);
  double lp = sum4(prior_term(x));
  if (ll0 && lane == 0) ll0[c] = ll;
  // Phi(-x/sd) and ln Phi(x/sd) of the current state
  double p0 = gauss ? ncdf(-x / sd) : 0.0;
  double lcx = gauss ? log(ncdf(x / sd)) : 0.0;
  int32_t acc = 0;
  double un = iters > 0 ? prop[(int64_t)c * 4 + k] : 0.5;
  double an = iters > 0 ? alpha[c] : 1.0;
  for (int32_t i = 0; i < iters; ++i) {
    const int64_t row = (int64_t)i * A.B + c;
    const double u = un, al = an;
    if (i + 1 < iters) {  // the next iteration's numbers, on their way meanwhile
      un = prop[(row + A.B) * 4 + k];
      an = alpha[row + A.B];
    }
    double y = x, lq = 0.0, lcy = lcx;
    bool ok = true;
    if (gauss) {
      const double pu = u <= 0.5 ? p0 + u * (1.0 - p0) : (1.0 - u) * (1.0 - p0);
      const double zi = normcdfinv(pu);
      const double z = u <= 0.5 ? zi : -zi;
      y = x + sd * z;
      ok = y > 0.0 && isfinite(y);
      if (ok) {
        lcy = log(ncdf(y / sd));
        lq = lcx - lcy;
      }
    } else if (ig) {
      y = H.ig_prop_factor * x / u;
      ok = y > 0.0 && isfinite(y);
      if (ok) {
        const double r = y / x;
        lq = (2.0 * H.ig_prop_shape + 1.0) * log(r) - H.ig_prop_factor * (r - 1.0 / r);
      }
    }
    if (__ballot(!ok) == 0) {
      params(y, th);
      const double llp = loglik(th);
      const double lpp = sum4(prior_term(y));
      if (log(al) <= (llp - ll) + ((lpp - lp) + sum4(lq))) {
        x = y;
        ll = llp;
        lp = lpp;
        ++acc;
        lcx = lcy;
        if (gauss) p0 = ncdf(-x / sd);
      }
    }
    if (lane < 4) theta_trace[row * 4 + k] = x;
    if (lane == 0) ll_trace[row] = ll;
  }
  if (lane == 0) accepts[c] = acc;
}

// One chain per lane through every iteration (Alg. 3): truncated-Gaussian
// proposals of R, C, Z by inversion on the accurate tail, the
// Inverse-Gamma proposal of sigma^2 from the given Gamma variate, support
// check, exact likelihood, prior and proposal density ratios, acceptance.
__global__ void __launch_bounds__(64) k_kf_pmmh(KfArgs A, pf_wk_mh H, double h, int32_t iters,
                                                const double* __restrict__ theta0,
                                                const double* __restrict__ prop,
                                                const double* __restrict__ alpha,
                                                double* __restrict__ theta_trace,
                                                double* __restrict__ ll_trace,
                                                int32_t* __restrict__ accepts,
                                                double* __restrict__ ll0) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= A.B) return;
  double x[4], y[4], th[8];
  for (int k = 0; k < 4; ++k) x[k] = theta0[(int64_t)c * 4 + k];
  wk_params(H, h, x, th);
  double ll = kf_loglik(A, th);
  double lp = wk_log_prior(H, x);
  if (ll0) ll0[c] = ll;
  int32_t acc = 0;
  for (int32_t i = 0; i < iters; ++i) {
    const int64_t row = (int64_t)i * A.B + c;
    const double* u = prop + row * 4;
    double lq = 0.0;
    bool inside = true;
    for (int k = 0; k < 3; ++k) {
      const double s = H.step_sd[k];
      if (s > 0.0) {
        const double p0 = ncdf(-x[k] / s);
        const double z = (u[k] <= 0.5) ? normcdfinv(p0 + u[k] * (1.0 - p0))
                                        : -normcdfinv((1.0 - u[k]) * (1.0 - p0));
        y[k] = x[k] + s * z;
        if (!(y[k] > 0.0) || !isfinite(y[k]))
          inside = false;
        else
          lq += log(ncdf(x[k] / s)) - log(ncdf(y[k] / s));
      } else {
        y[k] = x[k];
      }
    }
    if (H.ig_prop_factor > 0.0) {
      y[3] = H.ig_prop_factor * x[3] / u[3];
      if (!(y[3] > 0.0) || !isfinite(y[3])) {
        inside = false;
      } else {
        const double r = y[3] / x[3];
        lq += (2.0 * H.ig_prop_shape + 1.0) * log(r) - H.ig_prop_factor * (r - 1.0 / r);
      }
    } else {
      y[3] = x[3];
    }
    if (inside) {
      wk_params(H, h, y, th);
      const double llp = kf_loglik(A, th);
      const double lpp = wk_log_prior(H, y);
      if (log(alpha[row]) <= (llp - ll) + ((lpp - lp) + lq)) {
        for (int k = 0; k < 4; ++k) x[k] = y[k];
        ll = llp;
        lp = lpp;
        ++acc;
      }
    }
    for (int k = 0; k < 4; ++k) theta_trace[row * 4 + k] = x[k];
    ll_trace[row] = ll;
  }
  accepts[c] = acc;
}

// ---------------------------------------------------------------- launchers

static inline unsigned kf_blocks(int n) { return (unsigned)((n + 255) / 256); }

// Which form runs B filters over T intervals of K substeps.  The
// lane-per-filter form is bound by its chain: whatever B (up to 32,768 at
// least) a chain iteration takes about 11 us for the proposals and 0.32 +
// 0.033 K us per interval (K = 10: 13.0 us at T = 3, 23.4 at T = 20, 75 at
// T = 100, 221 at T = 300; T = 100: 46 at K = 1, 109 at K = 20).  The
// wave-per-filter form is bound by issue once its waves fill the SIMDs: per
// chain and iteration about 2.4 ns, plus 1.5 + 0.08 K ns per pass of 128
// intervals (T = 100, K = 10: 6.1 us at 512 chains, 41 at 8,192, 78 at
// 16,384, 152 at 32,768; T = 300: 250 at 32,768).  A plain likelihood run has
// no proposals, in either form, and a wave's own latency shows in the shortest
// ones: 3.2 us against the lane form's 2.1 at T = 1 (one filter, K = 10), 3.0
// against 3.1 at T = 2.  The cheaper estimate wins: at T = 100 and K = 10 the
// wave form up to 16,500 chains.
static inline bool kf_wave_form(int B, int T, int K, bool chains) {
  const double passes = (double)((T + KF_PASS - 1) / KF_PASS);
  const double wave_ns =
      (chains ? 0.0 : 700.0) + B * ((chains ? 2.4 : 0.6) + passes * (1.5 + 0.08 * K));
  const double lane_ns = (chains ? 11e3 : 0.0) + T * (320.0 + 33.0 * K);
  return wave_ns <= lane_ns;
}
// LDS the chains' series may take (a block is one wave; 160 KB per CU)
constexpr size_t KF_LDS_MAX = 64 * 1024;

hipError_t launch_kf_run(const KfArgs& A, const double* theta, double* ll, double* ell,
                         hipStream_t s) {
  if (!kf_wave_form(A.B, A.T, A.K, false))
    hipLaunchKernelGGL(k_kf_run, kf_blocks(A.B), 256, 0, s, A, theta, ll, ell);
  else if (A.T <= KF_PASS)
    hipLaunchKernelGGL(k_kf_run_wave<false>, (unsigned)A.B, WAVE, 0, s, A, theta, ll, ell);
  else
    hipLaunchKernelGGL(k_kf_run_wave<true>, (unsigned)A.B, WAVE, 0, s, A, theta, ll, ell);
  return hipGetLastError();
}

hipError_t launch_kf_init(const Smc2Args& S, hipStream_t s) {
  hipLaunchKernelGGL(k_kf_init, kf_blocks(S.B), 256, 0, s, S);
  return hipGetLastError();
}

hipError_t launch_kf_proposal(const KfArgs& A, const Smc2Args& S, const double* prop_dev,
                              double* prop_l, double* prop_mV, int i, hipStream_t s) {
  if (i < 2 || !kf_wave_form(S.B, i - 1, A.K, false))
    hipLaunchKernelGGL(k_kf_proposal, kf_blocks(S.B), 256, 0, s, A, S, prop_dev, prop_l, prop_mV,
                       i);
  else if (i - 1 <= KF_PASS)
    hipLaunchKernelGGL(k_kf_proposal_wave<false>, (unsigned)S.B, WAVE, 0, s, A, S, prop_dev,
                       prop_l, prop_mV, i);
  else
    hipLaunchKernelGGL(k_kf_proposal_wave<true>, (unsigned)S.B, WAVE, 0, s, A, S, prop_dev,
                       prop_l, prop_mV, i);
  return hipGetLastError();
}

hipError_t launch_smc2_accept_kf(const Smc2Args& S, const double* log_alpha_row,
                                 const double* prop_dev, const double* prop_l,
                                 const double* prop_mV, int32_t* acc_tr_row, hipStream_t s) {
  hipLaunchKernelGGL(k_smc2_accept_kf, kf_blocks(S.B), 256, 0, s, S, log_alpha_row, prop_dev,
                     prop_l, prop_mV, acc_tr_row);
  return hipGetLastError();
}

hipError_t launch_kf_pmmh(const KfArgs& A, const pf_wk_mh& H, double h, int32_t iters,
                          const double* theta0, const double* prop, const double* alpha,
                          double* theta_trace, double* ll_trace, int32_t* accepts, double* ll0,
                          hipStream_t s) {
  const size_t lds = 8 * ((size_t)A.K * ((size_t)A.T + 1) + (size_t)A.T);
  const bool wave = kf_wave_form(A.B, A.T, A.K, true);
#define PF_KF_PMMH(LDS, SEVERAL)                                                                  \
  hipLaunchKernelGGL((k_kf_pmmh_wave<LDS, SEVERAL>), (unsigned)A.B, WAVE, LDS ? lds : 0, s, A, H, \
                     h, iters, theta0, prop, alpha, theta_trace, ll_trace, accepts, ll0)
  const bool fits = lds <= KF_LDS_MAX, several = A.T > KF_PASS;
  if (wave && fits && !several) PF_KF_PMMH(true, false);
  else if (wave && fits) PF_KF_PMMH(true, true);
  else if (wave) PF_KF_PMMH(false, true);
  else
    hipLaunchKernelGGL(k_kf_pmmh, (unsigned)((A.B + 63) / 64), 64, 0, s, A, H, h, iters, theta0,
                       prop, alpha, theta_trace, ll_trace, accepts, ll0);
#undef PF_KF_PMMH
  return hipGetLastError();
}

hipError_t launch_kf_advance(const KfArgs& A, const Smc2Args& S, int i, hipStream_t s) {
  hipLaunchKernelGGL(k_kf_advance, kf_blocks(S.B), 256, 0, s, A, S, i);
  return hipGetLastError();
}

}  // namespace pfk
