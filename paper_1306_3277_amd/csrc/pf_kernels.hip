// Plain-layout kernels of the gfx950 bootstrap particle filter (Alg. 2):
//   K1 propagate + weight   one particle per lane, K substeps in registers,
//                           log-weight, per-block (max, sum, sum of squares)
//   K2 combine              (filters of more than FUSE_NB blocks) one
//                           workgroup: global max, FP64 block offsets,
//                           likelihood increment, ESS, resampling uniform
//   K3 combine + scan +     (smaller filters combine the block partials in
//      marks                every K3 block instead of K2) FP64 block scan
//                           of exp(lw - M); for each particle the number of
//                           strata its cumulative weight covers, and a mark
//                           (its index) on the first stratum it owns
//   K4 tile gather          per tile of 256 outputs, a running maximum over
//                           the marks names every output's ancestor (the
//                           work per lane does not depend on the weights),
//                           then the ancestors' states are copied; only
//                           where the resampled set itself is wanted, K1
//                           names and gathers its ancestors the same way
// plus the stateless resampler's kernels, initialisation and the
// synthetic-data simulator.  The state is kept in 64-particle tiles (pidx).
#include <math.h>

#include "pf_device.hpp"
#include "pf_internal.hpp"

namespace pfk {

__device__ __forceinline__ Key key_of(const KeyArg& k) { return Key{k.lo, k.hi}; }

// ---------------------------------------------------------------- init
template <int MODEL, int D, typename Real>
__global__ __launch_bounds__(K1_NT) void k_init(Real* __restrict__ x, PlainArgs A) {
  const int64_t j = (int64_t)blockIdx.x * K1_NT + threadIdx.x;
  if (j >= A.N) return;
  const Key key = key_of(A.key);
  const uint32_t iter = A.fs->iter;
  const int64_t col = A.off + j;
  if (MODEL == 1) {
    double z0, z1;
    const uint4 w = draw(key, TAG_INIT, 0, iter, (uint32_t)j, 0, A.b);
    bm_pair_f64(w.x, w.y, z0, z1);
    x[col] = (Real)(A.theta[4] + A.theta[5] * z0);
  } else {
#pragma unroll
    for (int blk = 0; blk < D / 4; ++blk) {
      double z[4];
      normals4_f64(draw(key, TAG_INIT, blk, iter, (uint32_t)j, 0, A.b), z);
#pragma unroll
      for (int m = 0; m < 4; ++m) x[pidx(col, 4 * blk + m, D)] = (Real)z[m];
    }
  }
}

__global__ void k_reset(FilterState* fs, double* ell, double* ess, int B, int T, uint32_t iter) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)B * T) {
    ell[i] = 0.0;
    ess[i] = 0.0;
  }
  if (i < B) {
    FilterState f;
    f.loglik = 0.0;
    f.M = 0.0;
    f.S = 0.0;
    f.u = 0.0;
    f.ell = 0.0;
    f.ess = 0.0;
    f.t = 0;
    f.status = 0;
    f.iter = iter;
    f.pad = 0;
    f.lprev = 0.0;
    f.carry = 0;
    f.tk = 0;
    f.cn1 = 0;
    f.amode = AMODE_IDENTITY;
    fs[i] = f;
  }
}

// ---------------------------------------------------------------- combine
// The collective over the block partials (max, sum, sum of squares of the
// 256-particle K1 blocks).  Offsets of the blocks' cumulative weights: K1
// block i owns [off_i, off_{i+1}), off_nb = S.  They are summed
// sequentially within each lane's chunk of partials and scanned across the
// lanes; an exact running maximum then makes them non-decreasing whatever
// the rounding, so the cumulative weights built on them are monotone.
//
// Two forms.  A filter of at most FUSE_NB blocks has every K3 block combine
// all of its partials itself, each wave in the same order and with the same
// code as if a workgroup of COMB_NT lanes did, so that all obtain the same bits
// with no extra launch and no communication between blocks (a block's waves
// sharing the scans took five barriers, 6,450 of the block's 13,500 cycles at
// 256 partials).  A larger filter has one K2 workgroup combine them once and
// store the offsets, before K3.
struct Combined {
  double M, S, S2, lo, hi;
};

// The wave's lane l stands for lanes l, l + 64, l + 128 and l + 192 (its rows)
// of a combining workgroup of COMB_NT lanes, each of which owns `chunk`
// consecutive partials.  lo, hi: the offsets of partials k1b and k1b + span (S
// at the end).  Up to 64 partials fill one row, up to COMB_NT all four with a
// partial each; beyond, the block's waves share the exponentials through LDS
// (two barriers) and each scans them all (16 exponentials per lane took
// 10,500 cycles at 780 partials).
constexpr int COMB_NT = 256;
constexpr int COMB_PER = 4;  // partials per lane, at most
static_assert(FUSE_NB <= COMB_PER * COMB_NT, "partials per lane");
struct CombineLds {
  double T[FUSE_NB + FUSE_NB / 16];  // T_i at i + i/16 (padded against bank conflicts)
  double xm[COMB_NT / WAVE], xs2[COMB_NT / WAVE];
};

// The scan, from the lanes' totals T[r][c] of partials (64 r + lane) chunk + c.
template <int ROWS, int CH>
__device__ __forceinline__ void combine_scan(const double (&T)[ROWS][CH], int nb, int chunk,
                                             int k1b, int span, Combined& o) {
  const int lane = threadIdx.x & (WAVE - 1);
  double pre[ROWS], tot[ROWS], S = 0.0;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    double loc = 0.0;
#pragma unroll
    for (int c = 0; c < CH; ++c) loc += T[r][c];
    const double incl = wave_incl_scan(loc);
    pre[r] = incl - loc;
    tot[r] = last_lane(incl);
  }
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
#pragma unroll
    for (int q = 0; q < r; ++q) pre[r] += tot[q];
    S += tot[r];
  }
  // each lane's last offset; an exact running maximum over earlier lanes
  // makes the offsets non-decreasing whatever the rounding of the scan
  double vprev[ROWS], vall = -INFINITY;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    double last = -INFINITY, run = pre[r];
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (c < chunk && (r * WAVE + lane) * chunk + c < nb) {
        last = run;
        run += T[r][c];
      }
    const double vin = wave_incl_max_scan(last);
    vprev[r] = fmax(wave_prev(vin, -INFINITY), vall);
    vall = fmax(vall, last_lane(vin));
  }
  o.S = fmax(S, vall);
  // the offset of partial i, from the lane that owns it
  auto offset = [&](int i) -> double {
    if (i >= nb) return o.S;
    const int q = CH == 1 ? i : i / chunk, c0 = CH == 1 ? 0 : i - q * chunk, r0 = q / WAVE;
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      double run = pre[r];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (r == r0 && c == c0) v = fmax(run, vprev[r]);
        run += T[r][c];
      }
    }
    return lane_value(v, q & (WAVE - 1));
  };
  o.lo = offset(k1b);
  o.hi = offset(k1b + span);
}

// nb <= 64 ROWS partials, each wave for itself.  between() runs while they
// load.  S2 only if want2.
template <int ROWS, class Between>
__device__ __forceinline__ Combined combine_wave(const double* __restrict__ P, int nb, int k1b,
                                                 int span, bool want2, Between between) {
  const int lane = threadIdx.x & (WAVE - 1);
  double pm[ROWS], ps[ROWS], p2[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int i = min(r * WAVE + lane, nb - 1);
    pm[r] = P[3 * i];
    ps[r] = P[3 * i + 1];
    p2[r] = want2 ? P[3 * i + 2] : 0.0;
  }
  between();
  double m = -INFINITY;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    pm[r] = r * WAVE + lane < nb ? pm[r] : -INFINITY;
    m = fmax(m, pm[r]);
  }
  Combined o;
  const double M = wave_max(m);
  const bool finite = (M > -INFINITY) && (M < INFINITY);
  o.M = finite ? M : -INFINITY;
  // block totals T_i = s_i exp(m_i - M) (0 without a finite maximum or weight)
  double T[ROWS][1];
  o.S2 = 0.0;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const double e = exp_nonpos(pm[r] - M);
    const double sc = finite ? e : 0.0;
    T[r][0] = ps[r] * sc;
    p2[r] = p2[r] * (sc * sc);
  }
  if (want2) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) o.S2 += wave_sum(p2[r]);
  }
  combine_scan<ROWS, 1>(T, nb, 1, k1b, span, o);
  return o;
}

// 64 < nb <= FUSE_NB partials, the block's waves together.
template <class Between>
__device__ __forceinline__ Combined combine_block(const double* __restrict__ P, int nb, int k1b,
                                                  int span, bool want2, CombineLds& X,
                                                  Between between) {
  constexpr int NW = COMB_NT / WAVE, ROWS = NW;
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  double pm[COMB_PER], ps[COMB_PER], p2[COMB_PER];
#pragma unroll
  for (int k = 0; k < COMB_PER; ++k) {
    const int i = min((int)threadIdx.x + k * COMB_NT, nb - 1);
    pm[k] = P[3 * i];
    ps[k] = P[3 * i + 1];
    p2[k] = want2 ? P[3 * i + 2] : 0.0;
  }
  between();
  double m = -INFINITY;
#pragma unroll
  for (int k = 0; k < COMB_PER; ++k) {
    pm[k] = (int)threadIdx.x + k * COMB_NT < nb ? pm[k] : -INFINITY;
    m = fmax(m, pm[k]);
  }
  m = wave_max(m);
  if (lane == 0) X.xm[wv] = m;
  __syncthreads();
  double M = X.xm[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmax(M, X.xm[w]);
  Combined o;
  const bool finite = (M > -INFINITY) && (M < INFINITY);
  o.M = finite ? M : -INFINITY;
  double loc2 = 0.0;
#pragma unroll
  for (int k = 0; k < COMB_PER; ++k) {
    const int i = (int)threadIdx.x + k * COMB_NT;
    const double e = exp_nonpos(pm[k] - M);
    const double sc = finite ? e : 0.0;
    if (i < FUSE_NB) X.T[i + (i >> 4)] = i < nb ? ps[k] * sc : 0.0;
    if (i < nb) loc2 += p2[k] * (sc * sc);
  }
  if (want2) {
    const double s2w = wave_sum(loc2);
    if (lane == 0) X.xs2[wv] = s2w;
  }
  __syncthreads();
  o.S2 = 0.0;
  if (want2) {
#pragma unroll
    for (int w = 0; w < NW; ++w) o.S2 += X.xs2[w];
  }
  const int chunk = (nb + COMB_NT - 1) / COMB_NT;
  double T[ROWS][COMB_PER];
#pragma unroll
  for (int r = 0; r < ROWS; ++r)
#pragma unroll
    for (int c = 0; c < COMB_PER; ++c) {
      const int i = (r * WAVE + lane) * chunk + c;
      T[r][c] = (c < chunk && i < nb) ? X.T[i + (i >> 4)] : 0.0;
    }
  combine_scan<ROWS, COMB_PER>(T, nb, chunk, k1b, span, o);
  return o;
}

template <class Between>
__device__ __forceinline__ Combined combine(const double* __restrict__ P, int nb, int k1b,
                                            int span, bool want2, CombineLds& X,
                                            Between between) {
  if (nb <= WAVE) return combine_wave<1>(P, nb, k1b, span, want2, between);
  if (nb <= COMB_NT) return combine_wave<COMB_NT / WAVE>(P, nb, k1b, span, want2, between);
  return combine_block(P, nb, k1b, span, want2, X, between);
}

// K2 (filters of more than FUSE_NB blocks): one workgroup combines the
// partials and stores the offsets; a wave of its own beside them does the
// filter's bookkeeping (likelihood increment, ESS, trigger, resampling uniform,
// traces, interval counter) in step with the exchanges.  A lane sums a chunk of
// consecutive partials.  Up to K2_NT * KC of them come in, and their offsets go
// out, through LDS: a lane that reads and writes its own chunk in memory
// touches a line per access (192 and 64 B apart).  4,096 partials: 9.7 -> 7.5 us
// (one workgroup: latencies and a wave's FP64 chains; the partials alone, cold,
// take 2 us).
__global__ __launch_bounds__(K2_NT + WAVE) void k_combine(const double* __restrict__ part,
                                                          double* __restrict__ boff,
                                                          PlainArgs A) {
  constexpr int NW = K2_NT / WAVE;
  constexpr int KC = 8;  // block terms cached per lane (nb <= 4096 stays in registers)
  __shared__ double xm[NW], xs[NW], xs2[NW], xv[NW];
  // staged partials, then offsets; a pad per chunk spreads the lanes over the banks
  __shared__ double stage[K2_NT * (3 * KC + 1)];
  const int nb = A.nblk;
  const double* P = part + 3 * A.boff0;
  double* bo = boff + A.boff0 + A.b;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid / WAVE;
  const int chunk = (nb + K2_NT - 1) / K2_NT;
  const bool staged = chunk <= KC;
  if (wv == NW) {  // the bookkeeping wave
    FilterState* fst = A.fs;
    const int t = fst->tk;  // the interval K1 just propagated
    const double loglik0 = fst->loglik;
    const double lprev0 = fst->lprev;
    const int carry0 = fst->carry;
    const double u =
        A.mode == 2
            ? fst->u
            : u01_f64(draw(key_of(A.key), TAG_RESAMPLE, 0, fst->iter, 0, (uint32_t)t, A.b).x);
    // the factor's normaliser: ln N after a resampling, else the carried
    // weights' ln sum exp
    const double lprev = carry0 ? lprev0 : log((double)A.N);
    if (staged) __syncthreads();
    __syncthreads();  // exchange 1
    double M = xm[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmax(M, xm[w]);
    const bool finite = (M > -INFINITY) && (M < INFINITY);
    __syncthreads();  // exchange 2
    double S = 0.0, S2 = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      S += xs[w];
      S2 += xs2[w];
    }
    double L = M + log(S), ess = (S * S) / S2;
    __syncthreads();  // exchange 3
    double vall = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) vall = fmax(vall, xv[w]);
    const double Sf = fmax(S, vall);
    if (Sf != S) {  // rounding put the last block's offset above the total
      L = M + log(Sf);
      ess = (Sf * Sf) / S2;
    }
    if (lane == 0) {
      double ell = -INFINITY;
      int carry = 0;
      if (finite && Sf > 0.0) {
        ell = L - lprev;
        carry = !(ess < A.rs.ess_frac * (double)A.N);  // resample when ESS < ess_frac N
        fst->lprev = L;
      } else {
        ess = 0.0;
        fst->status = 4;
      }
      bo[nb] = Sf;
      fst->carry = carry;
      fst->loglik = loglik0 + ell;
      fst->M = finite ? M : -INFINITY;
      fst->S = Sf;
      fst->ell = ell;
      fst->ess = ess;
      fst->u = u;
      A.ell_tr[t - 1] = ell;
      A.ess_tr[t - 1] = ess;
      fst->t = t;
    }
    if (staged) __syncthreads();
    return;
  }
  const int i0 = min(nb, tid * chunk), i1 = min(nb, i0 + chunk);
  // the lane's first KC partials (indices past its chunk reread the last block
  // and are masked below)
  double pm[KC], ps[KC], p2[KC];
  if (staged) {
    double q[3 * KC];
#pragma unroll
    for (int e = 0; e < 3 * KC; ++e) q[e] = P[min(tid + e * K2_NT, 3 * nb - 1)];
#pragma unroll
    for (int e = 0; e < 3 * KC; ++e) {
      const int i = tid + e * K2_NT;
      stage[i + i / (3 * KC)] = q[e];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < KC; ++e) {
      const int i = min(i0 + e, nb - 1), c = 3 * i + i / KC;
      pm[e] = stage[c];
      ps[e] = stage[c + 1];
      p2[e] = stage[c + 2];
    }
  } else {
#pragma unroll
    for (int e = 0; e < KC; ++e) {
      const int i = min(i0 + e, nb - 1);
      pm[e] = P[3 * i];
      ps[e] = P[3 * i + 1];
      p2[e] = P[3 * i + 2];
    }
  }
  // exchange 1: the global maximum
  double m = -INFINITY;
#pragma unroll
  for (int e = 0; e < KC; ++e) {
    pm[e] = i0 + e < i1 ? pm[e] : -INFINITY;
    m = fmax(m, pm[e]);
  }
  for (int i = i0 + KC; i < i1; ++i) m = fmax(m, P[3 * i]);
  m = wave_max(m);
  if (lane == 0) xm[wv] = m;
  __syncthreads();
  double M = xm[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmax(M, xm[w]);
  const bool finite = (M > -INFINITY) && (M < INFINITY);
  // block totals T_i = s_i exp(m_i - M), summed sequentially within the lane;
  // the first KC of a lane's terms stay in registers (unrolled, fixed
  // indices), any further ones are recomputed
  auto term = [&](int i, double& T2) -> double {
    const double mb = P[3 * i];
    T2 = 0.0;
    if (!(finite && mb > -INFINITY)) return 0.0;
    const double sc = exp_nonpos(mb - M);
    T2 = P[3 * i + 2] * (sc * sc);
    return P[3 * i + 1] * sc;
  };
  double Tc[KC];
  double loc = 0.0, loc2 = 0.0;
#pragma unroll
  for (int e = 0; e < KC; ++e) {
    // (past the chunk, without a weight or a finite maximum: 0)
    const double x = exp_nonpos(pm[e] - M);
    const double sc = finite && pm[e] > -INFINITY ? x : 0.0;
    Tc[e] = ps[e] * sc;
    loc += Tc[e];
    loc2 += p2[e] * (sc * sc);
  }
  for (int i = i0 + KC; i < i1; ++i) {
    double T2;
    loc += term(i, T2);
    loc2 += T2;
  }
  // exchange 2: scan of the lanes' sums, total of squares
  const double incl = wave_incl_scan(loc, lane);
  const double s2w = wave_sum(loc2);
  if (lane == WAVE - 1) xs[wv] = incl;
  if (lane == 0) xs2[wv] = s2w;
  __syncthreads();
  double pre = incl - loc;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w < wv) pre += xs[w];
  // this lane's last offset; an exact running maximum over earlier lanes
  // makes the offsets non-decreasing whatever the rounding of the scan
  double last = -INFINITY;
  double off[KC];
  double run = pre;
#pragma unroll
  for (int e = 0; e < KC; ++e) {
    off[e] = run;
    if (i0 + e < i1) {
      last = run;
      run += Tc[e];
    }
  }
  const double run8 = run;
  for (int i = i0 + KC; i < i1; ++i) {
    double T2;
    last = run;
    run += term(i, T2);
  }
  const double vin = wave_incl_max_scan(last, lane);
  const double vup = wave_prev(vin, -INFINITY);
  if (lane == WAVE - 1) xv[wv] = vin;
  __syncthreads();  // exchange 3
  double vw = -INFINITY;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w < wv) vw = fmax(vw, xv[w]);
  const double vprev = (lane == 0) ? vw : fmax(vup, vw);
  if (staged) {
#pragma unroll
    for (int e = 0; e < KC; ++e) {
      const int i = i0 + e;
      if (i < i1) stage[i + i / KC] = fmax(off[e], vprev);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < KC; ++e) {
      const int i = tid + e * K2_NT;
      if (i < nb) bo[i] = stage[i + i / KC];
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < KC; ++e)
    if (i0 + e < i1) bo[i0 + e] = fmax(off[e], vprev);
  run = run8;
  for (int i = i0 + KC; i < i1; ++i) {
    double T2;
    bo[i] = fmax(run, vprev);
    run += term(i, T2);
  }
}


// ---------------------------------------------------------------- K1
// A K1 block's partials from its lanes' log-weights: the maximum, the sum and
// the sum of squares of exp(lw - max), valid in thread 0.  The waves' sums are
// added in order; two exchanges (a reduction of its own for each of the three
// took six barriers, 1,850 cycles).  `red` is LDS of 3 K1_NT / WAVE doubles.
__device__ __forceinline__ void block_partials(double lc, double* red, double& m, double& s1,
                                               double& s2) {
  constexpr int NW = K1_NT / WAVE;
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
  const double mw = wave_max(lc);
  if (lane == 0) red[w] = mw;
  __syncthreads();
  m = red[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) m = fmax(m, red[i]);
  // (without a finite maximum lc - m is -inf or NaN and the weight 0)
  const double e = exp_nonpos(lc - m);
  const double a = wave_sum(e), b = wave_sum(e * e);
  if (lane == 0) {
    red[NW + w] = a;
    red[2 * NW + w] = b;
  }
  __syncthreads();
  s1 = s2 = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    s1 += red[NW + i];
    s2 += red[2 * NW + i];
  }
}

// The particle output j continues in this interval (plain layout, every
// thread of a K1 block calls it: it has a barrier): the identity, the
// ancestor array, or, after a systematic or stratified collective, the
// running maximum of the marks over the block's tile (one tile of K4_TILE =
// K1_NT outputs per block) started from the tile's owner, as the tile
// gather forms it; those marks are cleared for the next collective and the
// ancestors written out.  Outputs past the filter's strata (rounding) go to
// the last particle of positive weight.
__device__ __forceinline__ int64_t plain_ancestor(int64_t j, int32_t* __restrict__ marks_all,
                                                  const int32_t* __restrict__ owner_all,
                                                  const int32_t* __restrict__ jc_all,
                                                  int32_t* __restrict__ anc,
                                                  const PlainArgs& A, int32_t* wtop,
                                                  int32_t* s_js) {
  const int64_t N = A.N;
  int32_t* marks = marks_all + A.off;
  // the mark and the tile's owner are fetched beside the filter's scalars,
  // wanted or not: one latency instead of two
  const int32_t mark = j < N ? marks[j] : -1;
  const int32_t own = owner_all[A.own0 + blockIdx.x];
  const int32_t amode = A.fs->amode;
  const int64_t cn1 = A.fs->cn1;
  if (amode == AMODE_IDENTITY) return j;
  if (amode == AMODE_ARRAY) return j < N ? (int64_t)anc[A.off + j] : j;
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int64_t k0 = (int64_t)blockIdx.x * K1_NT;
  if (threadIdx.x < WAVE) {
    int found = -1;
    if (k0 + K1_NT > cn1 && cn1 < N) {
      const int nb3 = (int)((N + K3_SPAN - 1) / K3_SPAN);
      for (int base = nb3 - 1; base >= 0 && found < 0; base -= WAVE) {
        const int i = base - (int)threadIdx.x;
        found = wave_max_i(i >= 0 ? jc_all[A.own0 + i] : -1);
      }
    }
    if (threadIdx.x == 0) *s_js = found;
  }
  const int32_t run = max(k0 < cn1 ? own : -1, mark);
  if (j < N) marks[j] = -1;
  const int32_t incl = wave_incl_max_scan_i(run, lane);
  if (lane == WAVE - 1) wtop[wv] = incl;
  __syncthreads();
  int32_t excl = -1;
#pragma unroll
  for (int w = 0; w < K1_NT / WAVE; ++w)
    if (w < wv) excl = max(excl, wtop[w]);
  if (j >= N) return j;
  int32_t a = j < cn1 ? max(excl, incl) : *s_js;
  if (a < 0 || a >= N) {  // never expected; flagged, and kept in bounds
    atomicOr(&A.fs->pad, 1);
    a = 0;
  }
  anc[A.off + j] = a;
  return a;
}

template <int MODEL, int D, typename Real, bool ACC = false>
__global__ __launch_bounds__(K1_NT) void k_propagate_weight(Real* __restrict__ xa,
                                                            Real* __restrict__ xb,
                                                            double* __restrict__ lw,
                                                            double* __restrict__ part,
                                                            int32_t* __restrict__ marks,
                                                            const int32_t* __restrict__ owner,
                                                            const int32_t* __restrict__ jc,
                                                            int32_t* __restrict__ anc,
                                                            PlainArgs A) {
  __shared__ double red[3 * K1_NT / WAVE];
  __shared__ int32_t wtop[K1_NT / WAVE];
  __shared__ int32_t s_js;
  const int64_t j = (int64_t)blockIdx.x * K1_NT + threadIdx.x;
  const int t = A.fs->t + 1;
  const uint32_t iter = A.fs->iter;
  const Key key = key_of(A.key);
  // interval t gathers buffer (t - 1) % 2 and writes buffer t % 2
  const Real* __restrict__ xcur = ((t - 1) & 1) ? xb : xa;
  Real* __restrict__ xprop = (t & 1) ? xb : xa;
  const double* __restrict__ yrow = A.obs + (int64_t)(t - 1) * A.n_obs;
  const int64_t src = A.off + plain_ancestor(j, marks, owner, jc, anc, A, wtop, &s_js);
  double l = -INFINITY;
  if (j < A.N) {
    const int64_t col = A.off + j;
    const int n0 = (t - 1) * A.K;
    if constexpr (MODEL == 1) {
      if constexpr (sizeof(Real) == 8) {
        double p = xcur[src];
        for (int s = 1; s <= A.K; ++s) {
          const uint4 w = draw(key, TAG_NOISE, 0, iter, (uint32_t)j, (uint32_t)(n0 + s), A.b);
          double z0, z1;
          bm_pair_f64(w.x, w.y, z0, z1);
          p = wk_substep_f64(p, A.theta, A.q[n0 + s - 1], z0);
        }
        xprop[col] = p;
        const double e = (yrow[0] - (p + A.theta[2] * A.q[(int64_t)t * A.K])) * A.inv_sd;
        l = -0.5 * (e * e) + A.lw_cst;
      } else {
        float p = xcur[src];
        double pa = p;  // the accurate form carries the pressure in FP64
        const float a = (float)(A.theta[0] - 1.0), c = (float)A.theta[1], sp = (float)A.theta[3];
        for (int s = 1; s <= A.K; ++s) {
          const uint4 w = draw(key, TAG_NOISE, 0, iter, (uint32_t)j, (uint32_t)(n0 + s), A.b);
          float z0, z1;
          bm_pair_f32(w.x, w.y, z0, z1);
          if constexpr (ACC) {
            pa = pa + (double)wk_increment_f32((float)pa, a, c, sp, (float)A.q[n0 + s - 1], z0);
          } else {
            p = wk_substep_f32(p, a, c, sp, (float)A.q[n0 + s - 1], z0);
          }
        }
        if constexpr (ACC) p = (float)pa;
        else pa = p;
        xprop[col] = p;
        const double e = (yrow[0] - (pa + A.theta[2] * A.q[(int64_t)t * A.K])) * A.inv_sd;
        l = -0.5 * (e * e) + A.lw_cst;
      }
    } else {
      Real x[D];
#pragma unroll
      for (int i = 0; i < D; ++i) x[i] = xcur[pidx(src, i, D)];
      ObsAhead<D> obs;  // on its way beside the state
      if constexpr (D <= OBS_AHEAD) obs.fetch(yrow, A.obs_pos);
      if constexpr (sizeof(Real) == 8) {
        const double F = A.theta[0], sq = A.theta[1];
        ModelConsts mc{A.h, A.hh, A.h6, A.inv_sd, A.lw_cst};
        for (int s = 1; s <= A.K; ++s) {
          if constexpr (MODEL == 3)
            l96_substep_stage_f64<D>(x, F, sq, mc, key, TAG_NOISE, iter, (uint32_t)j,
                                     (uint32_t)(n0 + s), A.b);
          else
            l96_substep_f64<D>(x, F, sq, mc, key, TAG_NOISE, iter, (uint32_t)j,
                               (uint32_t)(n0 + s), A.b);
        }
      } else if constexpr (ACC) {
        double xa[D];
#pragma unroll
        for (int i = 0; i < D; ++i) xa[i] = (double)x[i];
        const L96F32A c = l96_f32a_consts(A.theta[0], A.theta[1], A.h);
        for (int s = 1; s <= A.K; ++s) {
          if constexpr (MODEL == 3)
            l96_substep_stage_f32acc<D>(xa, c, key, TAG_NOISE, iter, (uint32_t)j,
                                        (uint32_t)(n0 + s), A.b);
          else
            l96_substep_f32acc<D>(xa, c, key, TAG_NOISE, iter, (uint32_t)j, (uint32_t)(n0 + s),
                                  A.b);
        }
#pragma unroll
        for (int i = 0; i < D; ++i) xprop[pidx(col, i, D)] = (Real)xa[i];
        // the log-weight from the state before it is rounded for storage
        l = l96_logdens<D, double>(xa, obs, yrow, A.obs_pos, A.inv_sd, A.lw_cst);
      } else {
        const L96F32 c = l96_f32_consts(A.theta[0], A.theta[1], A.h);
        for (int s = 1; s <= A.K; ++s) {
          if constexpr (MODEL == 3)
            l96_substep_stage_f32<D>(x, c, key, TAG_NOISE, iter, (uint32_t)j, (uint32_t)(n0 + s),
                                     A.b);
          else
            l96_substep_f32<D>(x, c, key, TAG_NOISE, iter, (uint32_t)j, (uint32_t)(n0 + s), A.b);
        }
      }
      if constexpr (!ACC || sizeof(Real) == 8) {
#pragma unroll
        for (int i = 0; i < D; ++i) xprop[pidx(col, i, D)] = x[i];
        l = l96_logdens<D, Real>(x, obs, yrow, A.obs_pos, A.inv_sd, A.lw_cst);
      }
    }
    // weights kept from a step that did not resample carry over
    if (A.fs->carry) l = lw[col] + l;
    lw[col] = l;
  }
  // a NaN log-weight counts as zero weight
  const double lc = (l == l) ? l : -INFINITY;
  double m, s1, s2;
  block_partials(lc, red, m, s1, s2);
  if (threadIdx.x == 0) {
    double* p = part + 3 * (A.boff0 + blockIdx.x);
    p[0] = m;
    p[1] = s1;
    p[2] = s2;
    // the interval K3 processes (it must not read the counter it advances)
    if (blockIdx.x == 0) A.fs->tk = t;
  }
}

// The stateless resampler's first kernel: block partials (max, sum, sum of
// squares of exp(lw - max)) of caller-given FP64 log-weights, the reduction
// K1 ends with; each block also clears its marks, and block 0 starts the
// scalars that the scan reads (u, interval 1).  Launch-bound calls: three
// launches for the clearing and the scalars took as long as this kernel (5.7
// us of 10^6 weights' 34, more than half of the kernel time of a small set's).
__global__ __launch_bounds__(K1_NT) void k_lw_partials(const double* __restrict__ lw,
                                                       double* __restrict__ part,
                                                       int32_t* __restrict__ marks, double u,
                                                       PlainArgs A) {
  __shared__ double red[3 * K1_NT / WAVE];
  const int64_t j = (int64_t)blockIdx.x * K1_NT + threadIdx.x;
  const double l = j < A.N ? lw[j] : -INFINITY;
  if (j < A.N) marks[j] = -1;
  const double lc = (l == l) ? l : -INFINITY;  // a NaN log-weight counts as zero weight
  double m, s1, s2;
  block_partials(lc, red, m, s1, s2);
  if (threadIdx.x == 0) {
    double* p = part + 3 * (int64_t)blockIdx.x;
    p[0] = m;
    p[1] = s1;
    p[2] = s2;
    if (blockIdx.x == 0) {
      FilterState f = {};
      f.u = u;
      f.tk = 1;
      *A.fs = f;
    }
  }
}

__global__ void k_set_u(FilterState* fs, double u) {
  if (threadIdx.x == 0 && blockIdx.x == 0) fs->u = u;
}

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------- K3
// W_j = boff[blk] + (block-local inclusive scan of exp(lw - M)), made
// non-decreasing by an exact running maximum and capped by boff[blk+1]; then
// c_j = #{k : (u + k) S < N W_j}, the number of strata owned by particles
// 0..j, so particle j owns strata [c_{j-1}, c_j).  Each particle that owns
// any marks the first of them with its index (one store per particle, no
// loop over its offspring); the owner of every K4 tile's first stratum is
// stored by the particle whose strata cover it, so K4 can name every
// stratum's owner from its tile's marks alone.  At a block edge the strata
// between the block's last count and g = count(boff[blk+1]) belong to the
// next block's first particle; the block's last lane records them, because
// only it knows that count.  Strata past the last particle's count (rounding
// overflow) go to the last particle of positive weight (jstar).
// FUSED: the block's waves combine the partials themselves, and (but in mode
// 1) the launch has one block more, the first, that does the filter's
// bookkeeping: its two logarithms and division, on another CU's time.
template <bool FUSED>
__global__ __launch_bounds__(K3_NT) void k_scan_mark(const double* __restrict__ lw,
                                                     const double* __restrict__ part,
                                                     const double* __restrict__ boff,
                                                     int32_t* __restrict__ marks_all,
                                                     int32_t* __restrict__ owner_all,
                                                     int32_t* __restrict__ jc_all,
                                                     PlainArgs A) {
  constexpr int NW = K3_NT / WAVE;
  __shared__ double xsum[NW], xvmax[NW];
  __shared__ int xcand[NW];
  __shared__ CombineLds X;
  const int blk = (int)blockIdx.x - (FUSED && A.mode != 1 ? 1 : 0);
  const int32_t N = (int32_t)A.N;
  FilterState* fst = A.fs;
  const Key key = key_of(A.key);
  if (FUSED && blk < 0) {
    int32_t t;
    double lprev, u;
    const Combined cb = combine(part + 3 * A.boff0, A.nblk, 0, 1, true, X, [&] {
      t = fst->tk;  // the interval K1 just propagated
      lprev = fst->carry ? fst->lprev : log((double)N);
      // mode 0 draws the resampling uniform, mode 2 has it in the scalars
      u = A.mode == 0 ? u01_f64(draw(key, TAG_RESAMPLE, 0, fst->iter, 0, (uint32_t)t, A.b).x)
                      : fst->u;
    });
    const bool pos = (cb.M > -INFINITY) && (cb.M < INFINITY) && (cb.S > 0.0);
    const double ess = pos ? (cb.S * cb.S) / cb.S2 : 0.0;
    if (threadIdx.x != 0) return;
    // likelihood increment (the normaliser is ln N after a resampling, else
    // the carried weights' ln sum exp), ESS, trigger (resample when ESS <
    // ess_frac N), uniform, traces, and the interval counter
    double ell;
    if (pos) {
      const double L = cb.M + log(cb.S);
      ell = L - lprev;
      fst->lprev = L;
    } else {
      ell = -INFINITY;
      fst->status = 4;
    }
    fst->carry = pos && !(ess < A.rs.ess_frac * (double)N);
    fst->loglik = fst->loglik + ell;
    fst->M = cb.M;
    fst->S = cb.S;
    fst->ell = ell;
    fst->ess = ess;
    fst->u = u;
    A.ell_tr[t - 1] = ell;
    A.ess_tr[t - 1] = ess;
    fst->t = t;
    return;
  }
  // no cumulative weights needed
  if (A.rs.scheme == RS_METROPOLIS || A.rs.scheme == RS_REJECTION) return;
  const int32_t jb = blk * K3_SPAN;
  const int32_t j0 = jb + (int)threadIdx.x * K3_PER;
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  // the lane's K3_PER consecutive log-weights, loaded first so that they
  // arrive while the partials are combined (past the end they reread the
  // last weight)
  double lv[K3_PER];
#pragma unroll
  for (int e = 0; e < K3_PER; ++e) lv[e] = lw[A.off + min((int64_t)j0 + e, (int64_t)N - 1)];
  const int k1b = blk * (K3_SPAN / K1_NT);  // first K1 block of this block
  double M, S, u, lo_off, hi_off;
  bool pos, carry;
  int32_t t_now;
  uint32_t it_now;
  if constexpr (FUSED) {
    const Combined cb = combine(
        part + 3 * A.boff0, A.nblk, k1b, K3_SPAN / K1_NT, A.rs.ess_frac < INFINITY, X, [&] {
          t_now = fst->tk;
          it_now = fst->iter;
          // modes 1 and 2 take the uniform already in the filter's scalars
          // (1 redraws only the ancestors)
          u = A.mode == 0
                  ? u01_f64(draw(key, TAG_RESAMPLE, 0, it_now, 0, (uint32_t)t_now, A.b).x)
                  : fst->u;
        });
    M = cb.M;
    S = cb.S;
    lo_off = cb.lo;
    hi_off = cb.hi;
    pos = (M > -INFINITY) && (M < INFINITY) && (S > 0.0);
    carry = pos && A.rs.ess_frac < INFINITY && !((S * S) / cb.S2 < A.rs.ess_frac * (double)N);
  } else {
    // K2 has combined the partials and done the bookkeeping
    t_now = fst->tk;
    it_now = fst->iter;
    M = fst->M;
    S = fst->S;
    u = fst->u;
    pos = (M > -INFINITY) && (M < INFINITY) && (S > 0.0);
    carry = fst->carry;
    const double* bo = boff + A.boff0 + A.b;
    lo_off = bo[k1b];
    hi_off = bo[min(k1b + K3_SPAN / K1_NT, A.nblk)];
  }
  // a step that keeps its weights (ESS above the trigger) or has none
  // positive gives every particle one offspring: itself
  const bool finite = pos && !carry;
  const double invS = 1.0 / S;
  // in-lane sequential prefix of K3_PER consecutive weights, and the lane's
  // last particle of positive weight (for the rare case where rounding
  // leaves the final strata without an owner)
  double loc[K3_PER];
  double run = 0.0;
  int cand = -1;
#pragma unroll
  for (int e = 0; e < K3_PER; ++e) {
    const bool in = j0 + e < N && lv[e] == lv[e];
    const double we = exp_nonpos((in ? lv[e] : -INFINITY) - M);
    const double w = finite ? we : 0.0;
    cand = w > 0.0 ? j0 + e : cand;
    run += w;
    loc[e] = run;
  }
  // exchange 1: the lanes' sums scanned across the block (and the block's
  // candidate, which only lane 0 needs)
  const double incl = wave_incl_scan(run);
  const int cw = wave_max_i(cand);
  if (lane == WAVE - 1) xsum[wv] = incl;
  if (lane == 0) xcand[wv] = cw;
  __syncthreads();
  double pre = incl - run;
#pragma unroll
  for (int q = 0; q < NW; ++q)
    if (q < wv) pre += xsum[q];
  double V[K3_PER];
#pragma unroll
  for (int e = 0; e < K3_PER; ++e) V[e] = lo_off + (pre + loc[e]);
  // exchange 2: an exact running maximum over earlier lanes keeps W
  // non-decreasing across lanes whatever the rounding of the tree scan;
  // capped by the next offset
  const double vin = wave_incl_max_scan(V[K3_PER - 1]);
  const double vup = wave_prev(vin, -INFINITY);
  if (lane == WAVE - 1) xvmax[wv] = vin;
  __syncthreads();
  double vw = -INFINITY;
#pragma unroll
  for (int q = 0; q < NW; ++q)
    if (q < wv) vw = fmax(vw, xvmax[q]);
  const double vprev = lane > 0 ? fmax(vup, vw) : (wv > 0 ? vw : lo_off);
  // W[e + 1]: particle e's cumulative weight; W[0]: the one before the lane's
  // first (the previous lane's last, or this block's offset); then the next
  // block's offset.  Their stratum counts c: particle e owns the strata
  // [c[e], c[e + 1]), and those up to c[K3_PER + 1] below the next block's
  // first count belong to its first particle: this block's last lane records
  // them, because only it knows its own last count.
  double W[K3_PER + 2];
  W[0] = fmin(vprev, hi_off);
#pragma unroll
  for (int e = 0; e < K3_PER; ++e) W[e + 1] = fmin(fmax(V[e], vprev), hi_off);
  W[K3_PER + 1] = hi_off;
  if (A.rs.scheme == RS_MULTINOMIAL) {
#pragma unroll
    for (int e = 0; e < K3_PER; ++e)
      if (j0 + e < N) A.wcum[j0 + e] = W[e + 1];
    // the ends of every 16 and every 256 of them
    const int32_t jl = j0 < N ? lane_last(j0, N) : 0;  // the lane's last particle
    double wl = W[1];
#pragma unroll
    for (int e = 1; e < K3_PER; ++e) wl = jl == j0 + e ? W[e + 1] : wl;
    if (j0 < N && (jl % 16 == 15 || jl == N - 1)) A.w16[jl / 16] = wl;
    if (j0 < N && (jl % 256 == 255 || jl == N - 1)) A.w256[jl / 256] = wl;
  }
  // the lane before the next block, if there is one
  const bool ends = threadIdx.x == K3_NT - 1 && (int64_t)jb + K3_SPAN < N;
  int32_t c[K3_PER + 2];
  if (!finite) {
#pragma unroll
    for (int e = 0; e <= K3_PER; ++e) c[e] = j0 + e;
    c[K3_PER + 1] = c[K3_PER];
  } else if (A.rs.scheme == RS_STRATIFIED) {
    auto count = [&](double w) -> int32_t {
      return stratum_count_strat(w, S, invS, N, key, t_now, A.b, it_now);
    };
#pragma unroll
    for (int e = 0; e <= K3_PER; ++e) c[e] = j0 < N ? count(W[e]) : 0;
    c[K3_PER + 1] = ends ? count(hi_off) : 0;
  } else {
    stratum_counts(W, S, invS, u, N, j0 < N ? (ends ? K3_PER + 2 : K3_PER + 1) : 0, c);
  }
  if (A.rs.scheme != RS_MULTINOMIAL) {
    int32_t* marks = marks_all + A.off;
    int32_t* owner = owner_all + A.own0;
    if (blk == 0 && threadIdx.x == 0) fst->amode = AMODE_MARKS;  // for the next propagation
    // ranges [rlo, rhi) of particle j0 + e (e = K3_PER: the next block's first)
    int32_t rlo[K3_PER + 1], rhi[K3_PER + 1];
#pragma unroll
    for (int e = 0; e <= K3_PER; ++e) {
      const bool in = e < K3_PER ? j0 + e < N : ends;
      rlo[e] = in ? c[e] : 0;
      rhi[e] = in ? c[e + 1] : 0;
      if (rlo[e] < rhi[e]) marks[rlo[e]] = j0 + e;
    }
    // Tile q's first stratum q K4_TILE lies in at most one range.  A range
    // covering at most two tile starts is stored by its lane; a longer one
    // (a particle owning many strata) by the whole wave, strided over the
    // lanes, so no lane loops over hundreds of tiles.
#pragma unroll
    for (int e = 0; e <= K3_PER; ++e) {
      const int32_t first = (int32_t)(((uint32_t)rlo[e] + (K4_TILE - 1)) / K4_TILE);
      const int32_t last = rhi[e] > rlo[e] ? (rhi[e] - 1) / K4_TILE : first - 1;
      if (__ballot(first <= last) == 0) continue;
      const bool big = last - first + 1 > 2;
      if (!big)
        for (int32_t q = first; q <= last; ++q) owner[q] = j0 + e;
      uint64_t mask = __ballot(big);
      while (mask) {
        const int src = __ffsll((unsigned long long)mask) - 1;
        mask &= mask - 1;
        const int32_t bj = __builtin_amdgcn_readlane(j0 + e, src);
        const int32_t bq0 = __builtin_amdgcn_readlane(first, src);
        const int32_t bq1 = __builtin_amdgcn_readlane(last, src);
        for (int64_t q = (int64_t)bq0 + lane; q <= bq1; q += WAVE) owner[q] = bj;
      }
    }
  }
  if (j0 < N && N - j0 <= K3_PER) {  // the lane of the last particle
    int32_t cn1 = c[1];
#pragma unroll
    for (int e = 1; e < K3_PER; ++e) cn1 = j0 + e == N - 1 ? c[e + 1] : cn1;
    fst->cn1 = cn1;
  }
  if (threadIdx.x == 0) {
    int cb = xcand[0];
#pragma unroll
    for (int q = 1; q < NW; ++q) cb = max(cb, xcand[q]);
    jc_all[A.own0 + blk] = cb;
  }
}

// ---------------------------------------------------------------- K4
// The resampled set, on demand (the stepping path never runs this: the next
// propagation gathers through the pending ancestors itself).  One block per
// tile of K4_TILE outputs: with marks pending, a running maximum over the
// tile's marks (which it clears), started from the owner of the tile's
// first stratum, names each output's ancestor (outputs past the strata take
// the last particle of positive weight); with the identity or the ancestor
// array pending, those.  The ancestors are written out, and with buffers
// given, buffer t % 2 (t = fs->t) is gathered through them into buffer
// (t + 1) % 2.
template <int D, typename Real>
__global__ __launch_bounds__(K4_NT) void k_tile_gather(int32_t* __restrict__ marks_all,
                                                       const int32_t* __restrict__ owner_all,
                                                       const int32_t* __restrict__ jc_all,
                                                       Real* __restrict__ xa,
                                                       Real* __restrict__ xb,
                                                       int32_t* __restrict__ anc,
                                                       PlainArgs A) {
  static_assert(K4_PER == 1 && K4_NT == K1_NT, "one output per lane, one tile per block");
  __shared__ int32_t wtop[K4_NT / WAVE];
  __shared__ int32_t s_js;
  const int64_t k = (int64_t)blockIdx.x * K4_TILE + threadIdx.x;
  const int64_t a = plain_ancestor(k, marks_all, owner_all, jc_all, anc, A, wtop, &s_js);
  if (k >= A.N) return;
  anc[A.off + k] = (int32_t)a;
  if (xa == nullptr) return;
  const int t = A.fs->t;
  const Real* __restrict__ xprop = (t & 1) ? xb : xa;
  Real* __restrict__ xout = (t & 1) ? xa : xb;
  const int64_t src = A.off + a, dst = A.off + k;
  if constexpr (D > 0) {
#pragma unroll
    for (int i = 0; i < D; ++i) xout[pidx(dst, i, D)] = xprop[pidx(src, i, D)];
  } else {
    for (int i = 0; i < A.d; ++i) xout[pidx(dst, i, A.d)] = xprop[pidx(src, i, A.d)];
  }
}

// The stateless resampler's last kernel: the ancestors named by the marks of
// its scan, a wave per tile and four outputs per lane (the tile gather's
// block per tile has two barriers' latency for one output per lane, and clears
// marks that the next call's first kernel clears): 10^6 weights, 5.75 -> 3.65 us.
__global__ __launch_bounds__(K4_NT) void k_name_ancestors(const int32_t* __restrict__ marks,
                                                          const int32_t* __restrict__ owner,
                                                          const int32_t* __restrict__ jc,
                                                          int32_t* __restrict__ anc, PlainArgs A) {
  constexpr int PER = K4_TILE / WAVE;
  static_assert(PER == 4, "a lane's outputs are one 16-byte access");
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t N = A.N;
  const int64_t tile = (int64_t)blockIdx.x * (K4_NT / WAVE) + threadIdx.x / WAVE;
  const int64_t k0 = tile * K4_TILE, k = k0 + lane * PER;
  if (k0 >= N) return;
  const bool whole = k0 + K4_TILE <= N && (((uintptr_t)marks | (uintptr_t)anc) & 15) == 0;
  int32_t v[PER];
  if (whole) {
    const int4 q = *(const int4*)(marks + k);
    v[0] = q.x, v[1] = q.y, v[2] = q.z, v[3] = q.w;
  } else {
#pragma unroll
    for (int e = 0; e < PER; ++e) v[e] = k + e < N ? marks[k + e] : -1;
  }
  const int32_t own = owner[tile];
  const int64_t cn1 = A.fs->cn1;
  int32_t js = -1;
  if (k0 + K4_TILE > cn1 && cn1 < N) {  // strata past the last particle's count
    const int nb3 = (int)((N + K3_SPAN - 1) / K3_SPAN);
    for (int base = nb3 - 1; base >= 0 && js < 0; base -= WAVE) {
      const int i = base - lane;
      js = wave_max_i(i >= 0 ? jc[i] : -1);
    }
  }
#pragma unroll
  for (int e = 1; e < PER; ++e) v[e] = max(v[e], v[e - 1]);
  const int32_t incl = wave_incl_max_scan_i(v[PER - 1]);
  const int32_t up = __shfl_up(incl, 1);
  const int32_t before = max(k0 < cn1 ? own : -1, lane > 0 ? up : -1);
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    v[e] = k + e < cn1 ? max(before, v[e]) : js;
    if (k + e < N && (v[e] < 0 || v[e] >= N)) {  // never expected; kept in bounds
      atomicOr(&A.fs->pad, 1);
      v[e] = 0;
    }
  }
  if (whole) {
    *(int4*)(anc + k) = make_int4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (k + e < N) anc[k + e] = v[e];
  }
}

__global__ void k_set_amode(FilterState* fs, int n, int32_t v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) fs[i].amode = v;
}

// ---------------------------------------------------------------- Metropolis resampling
// A resampler without the collective over the weights: output k starts at
// particle k and takes A.rs.steps Metropolis moves with uniform proposals,
// reading the FP64 log-weights directly (a NaN counts as -inf).  A step that
// keeps its weights, or has none positive, gives the identity.
__global__ __launch_bounds__(K1_NT) void k_metropolis(const double* __restrict__ lw,
                                                      int32_t* __restrict__ anc, PlainArgs A) {
  const int64_t k = (int64_t)blockIdx.x * K1_NT + threadIdx.x;
  if (k >= A.N) return;
  const FilterState* f = A.fs;
  const bool draw_rs = (f->M > -INFINITY) && (f->M < INFINITY) && (f->S > 0.0) && !f->carry;
  const double* l = lw + A.off;
  const int32_t N = (int32_t)A.N;
  int32_t j = (int32_t)k;
  if (draw_rs) {
    const Key key = key_of(A.key);
    const int32_t t = f->t;
    const uint32_t it = f->iter;
    double lj = l[j];
    lj = (lj == lj) ? lj : -INFINITY;
    for (int s = 1; s <= A.rs.steps; s += 2) {
      const uint4 w = metro_draw(key, t, A.b, it, (int32_t)k, s);
      int32_t jp = metro_index(w.x, N);
      double lp = l[jp];
      lp = (lp == lp) ? lp : -INFINITY;
      if (ln_u_leq(w.y, lp - lj)) {
        j = jp;
        lj = lp;
      }
      if (s + 1 <= A.rs.steps) {
        jp = metro_index(w.z, N);
        lp = l[jp];
        lp = (lp == lp) ? lp : -INFINITY;
        if (ln_u_leq(w.w, lp - lj)) {
          j = jp;
          lj = lp;
        }
      }
    }
  }
  anc[A.off + k] = j;
  if (k == 0) A.fs->amode = AMODE_ARRAY;
}

// ---------------------------------------------------------------- rejection resampling
// Needs the largest log-weight (from the step's reduction) but no scan:
// output k tries candidates, k first, then uniform draws, until one passes
// ln u <= lw_j - M.  A step that keeps its weights, or has none positive,
// gives the identity.
__global__ __launch_bounds__(K1_NT) void k_rejection(const double* __restrict__ lw,
                                                     int32_t* __restrict__ anc, PlainArgs A) {
  const int64_t k = (int64_t)blockIdx.x * K1_NT + threadIdx.x;
  if (k >= A.N) return;
  const FilterState* f = A.fs;
  const double M = f->M;
  const bool draw_rs = (M > -INFINITY) && (M < INFINITY) && (f->S > 0.0) && !f->carry;
  const double* l = lw + A.off;
  int32_t j = (int32_t)k;
  if (draw_rs)
    j = reject_ancestor(key_of(A.key), f->t, A.b, f->iter, (int32_t)k, (int32_t)A.N, M,
                        [&](int32_t i) { return l[i]; });
  anc[A.off + k] = j;
  if (k == 0) A.fs->amode = AMODE_ARRAY;
}

// Multinomial resampling, as Alg. 2 writes it: output k takes
// a_k = min{j : W_j > u_k S} for an independent uniform u_k, by search of the
// cumulative weights K3 left (exactly non-decreasing); rounding overflow goes
// to the last positive weight (found by K3).  A step that keeps its weights, or
// has none positive, gives the identity.
// The search is a chain of dependent loads, scattered over the outputs: in the
// weights alone log2 N of them.  K3 also leaves the last weight of every 16
// and of every 256, so a block takes the lowest of these levels that has at most
// MULTI_NB entries (past 262,144 particles even samples of the highest) into
// LDS, searches it there and goes down by whole nodes of 16, a line each.
// 100,003 particles: 9.15 -> 7.15 us.  An interval of d = 4 filters, K = 2, of
// 1,000 / 65,536 / 10^6 particles: 12.6 / 18.7 / 109 us where the search of the
// weights took 14.0 / 20.7 / 137; seven values a round in the weights alone gave
// 12.3 / 19.1 / 186.
// The first of the n non-decreasing values at W + lo that is above thr (lo + n:
// none).
__device__ __forceinline__ int32_t first_above(const double* W, int32_t lo, int32_t n,
                                               double thr) {
  for (int32_t hi = lo + n; lo < hi;) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    const bool up = !(W[mid] > thr);
    lo = up ? mid + 1 : lo;
    hi = up ? hi : mid;
  }
  return lo;
}

// The same for n from 1 to 16, in one round.  Reads 16 values.
__device__ __forceinline__ int32_t node_above(const double* __restrict__ W, int32_t lo, int32_t n,
                                              double thr) {
  typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));
  d2 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = *(const d2*)(W + lo + 2 * i);
  int c = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) c += i < n && !(v[i / 2][i % 2] > thr) ? 1 : 0;
  return lo + c;
}

__global__ __launch_bounds__(K1_NT) void k_multinomial(const int32_t* __restrict__ jc_all,
                                                       int32_t* __restrict__ anc, PlainArgs A) {
  __shared__ double ends[MULTI_NB];
  const int32_t N = (int32_t)A.N;
  const int32_t k = (int32_t)(blockIdx.x * K1_NT + threadIdx.x);
  const auto [n16, level, nt, per, ns] = multi_levels(N);
  const double* top = level == 0 ? A.wcum : level == 1 ? A.w16 : A.w256;
  // sample i: the end of the level's entries [i per, (i + 1) per)
  double e[MULTI_NB / K1_NT];
#pragma unroll
  for (int q = 0; q < MULTI_NB / K1_NT; ++q)
    e[q] = top[min(((int)threadIdx.x + q * K1_NT + 1) * per, nt) - 1];
  const FilterState* f = A.fs;
  const double S = f->S;
  const bool draw_rs = (f->M > -INFINITY) && (f->M < INFINITY) && (S > 0.0) && !f->carry;
  const double thr = multi_u(key_of(A.key), f->t, A.b, f->iter, k) * S;
#pragma unroll
  for (int q = 0; q < MULTI_NB / K1_NT; ++q) ends[threadIdx.x + q * K1_NT] = e[q];
  __syncthreads();
  if (k >= N) return;
  int32_t a = k;
  if (draw_rs) {
    int32_t j = first_above(ends, 0, ns, thr);
    if (j < ns) {  // the sample is above thr: every level below has such an entry
      if (per > 1) j = first_above(top, j * per, min((j + 1) * per, nt) - 1 - j * per, thr);
      if (level == 2) j = node_above(A.w16, 16 * j, min(16, n16 - 16 * j), thr);
      if (level >= 1) j = node_above(A.wcum, 16 * j, min(16, N - 16 * j), thr);
      a = j;
    } else {
      int32_t js = -1;
      for (int i = (N - 1) / K3_SPAN; i >= 0 && js < 0; --i) js = jc_all[A.own0 + i];
      a = js >= 0 ? js : 0;
    }
  }
  anc[A.off + k] = a;
  if (k == 0) A.fs->amode = AMODE_ARRAY;
}

// ---------------------------------------------------------------- simulator
template <int MODEL, int D>
__global__ void k_simulate(double* __restrict__ out, PlainArgs A, double obs_sd) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const Key key = key_of(A.key);
  double x[D];
  if (MODEL == 1) {
    double z0, z1;
    const uint4 w = draw(key, TAG_DATA, 0, 0, 0, 0, 0);
    bm_pair_f64(w.x, w.y, z0, z1);
    x[0] = A.theta[4] + A.theta[5] * z0;
  } else {
    for (int blk = 0; blk < D / 4; ++blk) {
      double z[4];
      normals4_f64(draw(key, TAG_DATA, blk, 0, 0, 0, 0), z);
      for (int m = 0; m < 4; ++m) x[4 * blk + m] = z[m];
    }
  }
  for (int i = 0; i < D; ++i) out[i] = x[i];
  double* obs = out + (int64_t)(A.T + 1) * D;
  ModelConsts mc{A.h, A.hh, A.h6, A.inv_sd, A.lw_cst};
  for (int t = 1; t <= A.T; ++t) {
    for (int s = 1; s <= A.K; ++s) {
      const int n = (t - 1) * A.K + s;
      if (MODEL == 1) {
        double z0, z1;
        const uint4 w = draw(key, TAG_DATA, 0, 0, 0, (uint32_t)n, 0);
        bm_pair_f64(w.x, w.y, z0, z1);
        x[0] = wk_substep_f64(x[0], A.theta, A.q[n - 1], z0);
      } else {
        if constexpr (MODEL == 3)
          l96_substep_stage_f64<D>(x, A.theta[0], A.theta[1], mc, key, TAG_DATA, 0, 0,
                                   (uint32_t)n, 0);
        else
          l96_substep_f64<D>(x, A.theta[0], A.theta[1], mc, key, TAG_DATA, 0, 0, (uint32_t)n, 0);
      }
    }
    for (int i = 0; i < D; ++i) out[(int64_t)t * D + i] = x[i];
    for (int o = 0; o < A.n_obs; ++o) {
      double z[4];
      normals4_f64(draw(key, TAG_OBS, (uint32_t)(o / 4), 0, 0, (uint32_t)t, 0), z);
      const double mu = (MODEL == 1) ? x[0] + A.theta[2] * A.q[(int64_t)t * A.K]
                                     : x[A.obs_idx[o]];
      obs[(int64_t)(t - 1) * A.n_obs + o] = mu + obs_sd * z[o % 4];
    }
  }
}

// ---------------------------------------------------------------- launchers
static inline unsigned nblocks(int64_t n, int nt) { return (unsigned)((n + nt - 1) / nt); }

#define PF_L96_DIMS(X) X(4) X(8) X(16) X(32) X(40)

hipError_t launch_init(int model, int d, int prec, void* x, const PlainArgs& a, hipStream_t s) {
  const unsigned g = nblocks(a.N, K1_NT);
  if (model == 1) {
    if (prec == 0)
      hipLaunchKernelGGL((k_init<1, 1, double>), g, K1_NT, 0, s, (double*)x, a);
    else
      hipLaunchKernelGGL((k_init<1, 1, float>), g, K1_NT, 0, s, (float*)x, a);
    return hipGetLastError();
  }
  switch (d) {
#define X(DD)                                                                          \
  case DD:                                                                             \
    if (prec == 0)                                                                     \
      hipLaunchKernelGGL((k_init<2, DD, double>), g, K1_NT, 0, s, (double*)x, a);      \
    else                                                                               \
      hipLaunchKernelGGL((k_init<2, DD, float>), g, K1_NT, 0, s, (float*)x, a);        \
    break;
    PF_L96_DIMS(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_reset(FilterState* fs, double* ell, double* ess, int B, int T, uint32_t iter,
                        hipStream_t s) {
  const int64_t n = (int64_t)B * T > B ? (int64_t)B * T : B;
  hipLaunchKernelGGL(k_reset, nblocks(n, 256), 256, 0, s, fs, ell, ess, B, T, iter);
  return hipGetLastError();
}

hipError_t launch_propagate(int model, int d, int prec, void* xa, void* xb, void* lw,
                            double* part, int32_t* marks, const int32_t* owner,
                            const int32_t* jc, int32_t* anc, const PlainArgs& a, hipStream_t s) {
  const unsigned g = (unsigned)a.nblk;
  if (model == 1) {
    if (prec == 0)
      hipLaunchKernelGGL((k_propagate_weight<1, 1, double>), g, K1_NT, 0, s,
                         (double*)xa, (double*)xb, (double*)lw, part, marks, owner, jc, anc, a);
    else if (prec == 1)
      hipLaunchKernelGGL((k_propagate_weight<1, 1, float>), g, K1_NT, 0, s,
                         (float*)xa, (float*)xb, (double*)lw, part, marks, owner, jc, anc, a);
    else
      hipLaunchKernelGGL((k_propagate_weight<1, 1, float, true>), g, K1_NT, 0, s,
                         (float*)xa, (float*)xb, (double*)lw, part, marks, owner, jc, anc, a);
    return hipGetLastError();
  }
  switch (d * 4 + model) {
#define X(DD)                                                                             \
  case DD * 4 + 2:                                                                        \
    if (prec == 0)                                                                        \
      hipLaunchKernelGGL((k_propagate_weight<2, DD, double>), g, K1_NT, 0, s,             \
                         (double*)xa, (double*)xb, (double*)lw, part, marks, owner, jc, anc, a);      \
    else if (prec == 1)                                                                   \
      hipLaunchKernelGGL((k_propagate_weight<2, DD, float>), g, K1_NT, 0, s,              \
                         (float*)xa, (float*)xb, (double*)lw, part, marks, owner, jc, anc, a);        \
    else                                                                                  \
      hipLaunchKernelGGL((k_propagate_weight<2, DD, float, true>), g, K1_NT, 0, s,        \
                         (float*)xa, (float*)xb, (double*)lw, part, marks, owner, jc, anc, a);        \
    break;                                                                                \
  case DD * 4 + 3:                                                                        \
    if (prec == 0)                                                                        \
      hipLaunchKernelGGL((k_propagate_weight<3, DD, double>), g, K1_NT, 0, s,             \
                         (double*)xa, (double*)xb, (double*)lw, part, marks, owner, jc, anc, a);      \
    else if (prec == 1)                                                                   \
      hipLaunchKernelGGL((k_propagate_weight<3, DD, float>), g, K1_NT, 0, s,              \
                         (float*)xa, (float*)xb, (double*)lw, part, marks, owner, jc, anc, a);        \
    else                                                                                  \
      hipLaunchKernelGGL((k_propagate_weight<3, DD, float, true>), g, K1_NT, 0, s,        \
                         (float*)xa, (float*)xb, (double*)lw, part, marks, owner, jc, anc, a);        \
    break;
    PF_L96_DIMS(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_set_u(FilterState* fs, double u, hipStream_t s) {
  hipLaunchKernelGGL(k_set_u, 1, 64, 0, s, fs, u);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill_i32, nblocks(n, 256), 256, 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_lw_partials(const double* lw, double* part, int32_t* marks, double u,
                              const PlainArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_lw_partials, nblocks(a.N, K1_NT), K1_NT, 0, s, lw, part, marks, u, a);
  return hipGetLastError();
}

hipError_t launch_name_ancestors(const int32_t* marks, const int32_t* owner, const int32_t* jc,
                                 int32_t* anc, const PlainArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_name_ancestors, nblocks(a.N, K4_TILE * (K4_NT / WAVE)), K4_NT, 0, s, marks,
                     owner, jc, anc, a);
  return hipGetLastError();
}

hipError_t launch_tile_anc(int32_t* marks, const int32_t* owner, const int32_t* jc, int32_t* anc,
                           const PlainArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_tile_gather<0, float>), nblocks(a.N, K4_TILE), K4_NT, 0, s, marks, owner,
                     jc, (float*)nullptr, (float*)nullptr, anc, a);
  return hipGetLastError();
}

hipError_t launch_set_amode(FilterState* fs, int n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_set_amode, (unsigned)((n + 255) / 256), 256, 0, s, fs, n, v);
  return hipGetLastError();
}

hipError_t launch_combine(const double* part, double* boff, const PlainArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_combine, 1, K2_NT + WAVE, 0, s, part, boff, a);
  return hipGetLastError();
}

hipError_t launch_scan_mark(const double* lw, const double* part, const double* boff,
                            int32_t* marks, int32_t* owner, int32_t* jc, const PlainArgs& a,
                            hipStream_t s) {
  const unsigned g = nblocks(a.N, K3_SPAN);
  if (a.nblk <= FUSE_NB)
    hipLaunchKernelGGL(k_scan_mark<true>, g + (a.mode != 1 ? 1 : 0), K3_NT, 0, s, lw, part, boff, marks, owner, jc, a);
  else
    hipLaunchKernelGGL(k_scan_mark<false>, g, K3_NT, 0, s, lw, part, boff, marks, owner, jc, a);
  return hipGetLastError();
}

hipError_t launch_tile_gather(int model, int d, int prec, int32_t* marks, const int32_t* owner,
                              const int32_t* jc, void* xa, void* xb, int32_t* anc,
                              const PlainArgs& a, hipStream_t s) {
  const unsigned g = nblocks(a.N, K4_TILE);
  const int dd = model == 1 ? 1 : d;
  switch (dd) {
#define X(DD)                                                                               \
  case DD:                                                                                  \
    if (prec == 0)                                                                          \
      hipLaunchKernelGGL((k_tile_gather<DD, double>), g, K4_NT, 0, s, marks, owner, jc,      \
                         (double*)xa, (double*)xb, anc, a);                                 \
    else                                                                                    \
      hipLaunchKernelGGL((k_tile_gather<DD, float>), g, K4_NT, 0, s, marks, owner, jc,       \
                         (float*)xa, (float*)xb, anc, a);                                   \
    break;
    X(1) PF_L96_DIMS(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_metropolis_anc(const double* lw, int32_t* anc, const PlainArgs& a,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_metropolis, nblocks(a.N, K1_NT), K1_NT, 0, s, lw, anc, a);
  return hipGetLastError();
}

hipError_t launch_rejection_anc(const double* lw, int32_t* anc, const PlainArgs& a,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_rejection, nblocks(a.N, K1_NT), K1_NT, 0, s, lw, anc, a);
  return hipGetLastError();
}

hipError_t launch_multinomial_anc(const int32_t* jc, int32_t* anc,
                                  const PlainArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_multinomial, nblocks(a.N, K1_NT), K1_NT, 0, s, jc, anc, a);
  return hipGetLastError();
}

hipError_t launch_simulate(int model, int d, double* out, const PlainArgs& a, double obs_sd,
                           hipStream_t s) {
  if (model == 1) {
    hipLaunchKernelGGL((k_simulate<1, 1>), 1, 64, 0, s, out, a, obs_sd);
    return hipGetLastError();
  }
  switch (d * 4 + model) {
#define X(DD)                                                                      \
  case DD * 4 + 2:                                                                 \
    hipLaunchKernelGGL((k_simulate<2, DD>), 1, 64, 0, s, out, a, obs_sd);          \
    break;                                                                         \
  case DD * 4 + 3:                                                                 \
    hipLaunchKernelGGL((k_simulate<3, DD>), 1, 64, 0, s, out, a, obs_sd);          \
    break;
    PF_L96_DIMS(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace pfk
