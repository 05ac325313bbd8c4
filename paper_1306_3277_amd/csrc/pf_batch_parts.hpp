// Device parts of the batched layout shared by its stepping kernels: one
// particle's interval (propagation and log-weight), and a filter's scan in
// one workgroup (maximum, sums, cumulative weights, stratum counts).
#pragma once
#include "pf_device.hpp"
#include "pf_internal.hpp"

namespace pfk {

__device__ __forceinline__ Key bkey(const KeyArg& k) { return Key{k.lo, k.hi}; }

// ---------------------------------------------------------------- one particle's interval
// Interval t of particle k of filter f (f uniform): the state at column src
// of xp through K substeps to column dst of xn (and of the history's slot xh,
// with HIST); returns the log-weight of the observation.
template <int MODEL, int D, typename Real, bool ACC, bool HIST>
__device__ __forceinline__ double propagate_one(const Real* __restrict__ xp,
                                                Real* __restrict__ xn, Real* __restrict__ xh,
                                                int64_t src, int64_t dst, int64_t k, int f, int t,
                                                uint32_t iter, const BatchArgs& A) {
  const Key key = bkey(A.key);
  const double* th = A.theta + (size_t)f * 8;
  const double* yrow = A.obs + (int64_t)(t - 1) * A.n_obs;
  const int n0 = (t - 1) * A.K;
  double l;
  if constexpr (MODEL == 1) {
    if constexpr (sizeof(Real) == 8) {
      double p = xp[src];
      for (int s = 1; s <= A.K; ++s) {
        const uint4 w = draw(key, TAG_NOISE, 0, iter, (uint32_t)k, (uint32_t)(n0 + s), (uint32_t)f);
        double z0, z1;
        bm_pair_f64(w.x, w.y, z0, z1);
        p = wk_substep_f64(p, th, A.q[n0 + s - 1], z0);
      }
      xn[dst] = p;
      if constexpr (HIST) {
        if (xh) xh[dst] = p;
      }
      const double e = (yrow[0] - (p + th[2] * A.q[(int64_t)t * A.K])) * A.inv_sd;
      l = -0.5 * (e * e) + A.lw_cst;
    } else {
      float p = xp[src];
      double pa = p;  // the accurate form carries the pressure in FP64
      const float a = (float)(th[0] - 1.0), c = (float)th[1], sp = (float)th[3];
      for (int s = 1; s <= A.K; ++s) {
        const uint4 w = draw(key, TAG_NOISE, 0, iter, (uint32_t)k, (uint32_t)(n0 + s), (uint32_t)f);
        float z0, z1;
        bm_pair_f32(w.x, w.y, z0, z1);
        if constexpr (ACC)
          pa = pa + (double)wk_increment_f32((float)pa, a, c, sp, (float)A.q[n0 + s - 1], z0);
        else
          p = wk_substep_f32(p, a, c, sp, (float)A.q[n0 + s - 1], z0);
      }
      if constexpr (ACC) p = (float)pa;
      else pa = p;
      xn[dst] = p;
      if constexpr (HIST) {
        if (xh) xh[dst] = p;
      }
      const double e = (yrow[0] - (pa + th[2] * A.q[(int64_t)t * A.K])) * A.inv_sd;
      l = -0.5 * (e * e) + A.lw_cst;
    }
  } else {
    ObsAhead<D> obs;
    // (held through the substeps of the accurate form, which leave the scalar
    // unit less room, they cost 0.7% more instructions: 95.5 us an interval of
    // 512 filters in one group against 94.4 fetched at their use)
    if constexpr (D <= OBS_AHEAD && !ACC) obs.fetch(yrow, A.obs_pos);
    Real x[D];
#pragma unroll
    for (int i = 0; i < D; ++i) x[i] = xp[(int64_t)i * A.ld + src];
    if constexpr (sizeof(Real) == 8) {
      ModelConsts mc{A.h, A.hh, A.h6, A.inv_sd, A.lw_cst};
      for (int s = 1; s <= A.K; ++s) {
        if constexpr (MODEL == 3)
          l96_substep_stage_f64<D>(x, th[0], th[1], mc, key, TAG_NOISE, iter, (uint32_t)k,
                                   (uint32_t)(n0 + s), (uint32_t)f);
        else
          l96_substep_f64<D>(x, th[0], th[1], mc, key, TAG_NOISE, iter, (uint32_t)k,
                             (uint32_t)(n0 + s), (uint32_t)f);
      }
    } else if constexpr (ACC) {
      double xa[D];
#pragma unroll
      for (int i = 0; i < D; ++i) xa[i] = (double)x[i];
      const L96F32A c = l96_f32a_consts(th[0], th[1], A.h);
      for (int s = 1; s <= A.K; ++s) {
        if constexpr (MODEL == 3)
          l96_substep_stage_f32acc<D>(xa, c, key, TAG_NOISE, iter, (uint32_t)k,
                                      (uint32_t)(n0 + s), (uint32_t)f);
        else
          l96_substep_f32acc<D>(xa, c, key, TAG_NOISE, iter, (uint32_t)k, (uint32_t)(n0 + s),
                                (uint32_t)f);
      }
#pragma unroll
      for (int i = 0; i < D; ++i) x[i] = (Real)xa[i];
      if constexpr (D <= OBS_AHEAD) obs.fetch(yrow, A.obs_pos);
      // the log-weight from the state before it is rounded for storage
      l = l96_logdens<D, double>(xa, obs, yrow, A.obs_pos, A.inv_sd, A.lw_cst);
    } else {
      const L96F32 c = l96_f32_consts(th[0], th[1], A.h);
      for (int s = 1; s <= A.K; ++s) {
        if constexpr (MODEL == 3)
          l96_substep_stage_f32<D>(x, c, key, TAG_NOISE, iter, (uint32_t)k, (uint32_t)(n0 + s),
                                   (uint32_t)f);
        else
          l96_substep_f32<D>(x, c, key, TAG_NOISE, iter, (uint32_t)k, (uint32_t)(n0 + s),
                             (uint32_t)f);
      }
    }
#pragma unroll
    for (int i = 0; i < D; ++i) xn[(int64_t)i * A.ld + dst] = x[i];
    if (HIST && xh) {  // the history's slot, written from the same registers
#pragma unroll
      for (int i = 0; i < D; ++i) xh[(int64_t)i * A.ld + dst] = x[i];
    }
    if constexpr (!ACC || sizeof(Real) == 8) {
      l = l96_logdens<D, Real>(x, obs, yrow, A.obs_pos, A.inv_sd, A.lw_cst);
    }
  }
  return l;
}

// ---------------------------------------------------------------- a filter's scan
__device__ __forceinline__ int stage_slot(int i) { return i ^ ((i >> 4) & 15); }

// The ancestors in LDS (the stage, once its weights are read): one padding
// word after every 16, so that lanes reading or writing their own runs of
// P consecutive entries hit distinct banks (8,704 words for 8192 entries).
__device__ __forceinline__ int anc_slot(int i) { return i + (i >> 4); }

// A lane's weights e^{lw - M} over its run [i0, i1) of P <= CNT particles,
// their in-lane prefix sums, sum of squares and last positive index.  The
// body is straight-line over CNT slots (weights past the run are 0 and add
// nothing), so the exponentials interleave; P is the same for every lane,
// so the choice of CNT (the smallest power of two >= P) is a uniform branch.
template <int CNT, int MAXP>
__device__ __forceinline__ void lane_weights(const double* stage, int N, double M, bool finite,
                                             int P, int i0, int i1, double (&loc)[MAXP],
                                             double& run, double& run2, int& cand) {
  if constexpr (CNT > 1) {
    if (P <= CNT / 2) {
      lane_weights<CNT / 2, MAXP>(stage, N, M, finite, P, i0, i1, loc, run, run2, cand);
      return;
    }
  }
  double lv[CNT];
#pragma unroll
  for (int e = 0; e < CNT; ++e) lv[e] = stage[stage_slot(min(i0 + e, N - 1))];
#pragma unroll
  for (int e = 0; e < CNT; ++e) {
    const double we = exp_nonpos(lv[e] - M);  // exp(-inf) = 0
    const double w = (finite && e < P && i0 + e < i1) ? we : 0.0;
    cand = (w > 0.0) ? i0 + e : cand;
    run += w;
    run2 += w * w;
    loc[e] = run;
  }
}

// A lane's counts over its run of P particles, four side by side (more would
// hold more registers than the propagation running beside it can spare), the
// count before its first particle and the count of the whole filter.
// cum(e): particle e's cumulative weight.
template <int MAXP, class Cum>
__device__ __forceinline__ void lane_counts(int P, int i0, int i1, double vprev, double S,
                                            double invS, double u, int N, Cum cum,
                                            int32_t (&cnt)[MAXP], int32_t& before,
                                            int32_t& total) {
  constexpr int G = MAXP < 4 ? MAXP : 4;
  const int n = i1 - i0;
  {
    const double W[2] = {S, vprev};
    int32_t c[2];
    stratum_counts(W, S, invS, u, N, n > 0 ? 2 : 1, c);
    total = c[0];
    before = c[1];
  }
#pragma unroll
  for (int g = 0; g < MAXP; g += G) {
    if (g < P) {
      double W[G];
      int32_t c[G];
#pragma unroll
      for (int e = 0; e < G; ++e) W[e] = cum(g + e);
      stratum_counts(W, S, invS, u, N, n - g, c);
#pragma unroll
      for (int e = 0; e < G; ++e) cnt[g + e] = c[e];
    }
  }
}

// What a workgroup knows of its filter after the scan.  Thread tid owns the P
// consecutive particles [i0, i1).
template <int MAXP>
struct BatchScan {
  double M, S, S2;      // maximum, sum and sum of squares of exp(lw - M)
  double u;             // the resampling uniform
  double vprev, vlast;  // cumulative weights before the run and at its end
  double loc[MAXP];     // in-lane prefix sums
  int P, i0, i1;
  int jstar;            // the filter's last particle of positive weight
  bool finite;
  __device__ __forceinline__ double cum(int e) const {
    return (i0 + e == i1 - 1) ? vlast : fmin(vprev + loc[e], vlast);
  }
};
template <int NT>
struct ScanLds {
  double xa[NT / WAVE], xs[NT / WAVE], xb[NT / WAVE];
  int xi[NT / WAVE];
  double u;
};

// The scan of a filter's N <= NT MAXP log-weights by a workgroup of NT
// threads; `stage` holds NT MAXP doubles and is free again afterwards.  first()
// runs in thread 0 while the weights load and gives the uniform.
template <int NT, int MAXP, class First>
__device__ __forceinline__ void batch_scan(const double* __restrict__ lw, int N, double* stage,
                                           ScanLds<NT>& X, First first, BatchScan<MAXP>& o) {
  constexpr int NW = NT / WAVE;
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  // (1) coalesced load to the stage and the maximum; the loads are issued
  // together (indices past the filter read its last element and are
  // dropped), so their latencies overlap
  double m = -INFINITY;
  {
    double v[MAXP];
#pragma unroll
    for (int r = 0; r < MAXP; ++r)
      if (r * NT < N) v[r] = lw[min((int)threadIdx.x + r * NT, N - 1)];
    // the resampling uniform, drawn while the loads are in flight and
    // published with the first exchange
    if (threadIdx.x == 0) X.u = first();
#pragma unroll
    for (int r = 0; r < MAXP; ++r) {
      const int i = (int)threadIdx.x + r * NT;
      if (r * NT < N && i < N) {
        const double x = (v[r] == v[r]) ? v[r] : -INFINITY;  // NaN counts as zero weight
        stage[stage_slot(i)] = x;
        m = fmax(m, x);
      }
    }
  }
  m = wave_max(m);
  if (lane == 0) X.xa[wv] = m;
  __syncthreads();  // 1
  o.u = X.u;
  double M = X.xa[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmax(M, X.xa[w]);
  const bool finite = (M > -INFINITY) && (M < INFINITY);
  o.M = M;
  o.finite = finite;
  // (2) this lane's run: weights, in-lane prefix, square sum, last positive
  const int P = o.P = (N + NT - 1) / NT;
  const int i0 = o.i0 = min(N, (int)threadIdx.x * P), i1 = o.i1 = min(N, i0 + P);
  double run = 0.0, run2 = 0.0;
  int cand = -1;
  lane_weights<MAXP, MAXP>(stage, N, M, finite, P, i0, i1, o.loc, run, run2, cand);
  // one exchange: scan of the lanes' sums, total of squares, last positive
  // The scan's partial sums are rounded along different trees, so one
  // lane's may fall an ulp below the lane before: a running maximum makes
  // them non-decreasing, held past the filter's last particle (lanes with no
  // particles take -inf there), so that a wave's total is its last
  // particle's.
  const double incl = wave_incl_scan(run);
  const double inclm = wave_incl_max_scan((i1 > i0) ? incl : -INFINITY);
  const double s2w = wave_sum(run2);
  const int cw = wave_max_i(cand);
  // (the lane sums go to their own array, so no barrier separates them from
  // the maxima read above; the stage is reused only after this exchange)
  if (lane == WAVE - 1) X.xs[wv] = (inclm > -INFINITY) ? inclm : 0.0;
  if (lane == 0) {
    X.xb[wv] = s2w;
    X.xi[wv] = cw;
  }
  __syncthreads();  // 3
  // S: the waves' totals added in order; base: the same sum over the waves
  // before this one (the same operations, so the same bits)
  double base = 0.0, S = 0.0, S2 = 0.0;
  int jstar = -1;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w == wv) base = S;
    S += X.xs[w];
    S2 += X.xb[w];
    jstar = max(jstar, X.xi[w]);
  }
  // The cumulative weights: lane l's last particle has V_l = base + its
  // running total; before its first particle stands V_{l-1}, which the lane
  // before computes from the same two values (at a wave's first lane it is
  // base, the previous wave's last V); the particles between take
  // min(V_{l-1} + in-lane prefix, V_l).  Each value lies in [V_{l-1}, V_l]
  // (the prefixes are non-negative), so the sequence never decreases across
  // lanes and waves, and the filter's last particle has exactly S.
  // (the lane move runs in every lane, outside the select: a lane whose
  // source lane is switched off would read nothing)
  const double inprev = wave_prev(inclm, 0.0);
  o.vprev = (lane == 0) ? base : base + inprev;
  o.vlast = base + inclm;
  o.S = S;
  o.S2 = S2;
  o.jstar = jstar;
}

}  // namespace pfk
