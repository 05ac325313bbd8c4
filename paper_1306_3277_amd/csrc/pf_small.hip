// Filters of at most SMALL_MAXN particles, one workgroup each, everything of
// an interval in registers and LDS:
//   k_small_systematic  the resampling collective on caller-given weights
//                       (pf_systematic): one launch
//   k_small_noise       the random numbers of many intervals of every
//                       windkessel filter, over the whole device
//   k_small_run         those intervals of a windkessel filter in one launch
//
// The multi-kernel plain layout spends two launches per interval on such a
// filter and each of its kernels runs on one to sixteen of the 256 CUs,
// waiting on memory: 17.6 us per interval for 1,024 windkessel particles,
// 3.4 of them between kernels.  In one workgroup an interval needs no launch
// and no exchange through memory, but one CU's lanes for the normals, three
// quarters of the propagation's instructions; those depend on nothing but
// their counters, so a launch over the whole device draws them beforehand.
//
// Both keep the plain kernels' arithmetic: the sums over 256-particle blocks
// by 64-particle waves, the block totals and offsets, the scan over
// 1,024-particle spans of four particles per lane, with the same operands in
// the same order, so that weights, counts, ancestors and likelihoods have the
// same bits as theirs (eager steps, which stop between the two kernels, still
// run those).
#include <math.h>

#include "pf_device.hpp"
#include "pf_internal.hpp"

namespace pfk {

// Wave w of a workgroup holds the 256-particle block w, row r of its lanes
// the block's wave r (particle 256 w + 64 r + lane); as a scan lane, thread
// tid holds particles 4 tid .. 4 tid + 3.  NQ: 1,024-particle spans.
constexpr int ROWS = 4;
static_assert(K1_NT == ROWS * WAVE && K3_PER == ROWS && K3_SPAN == 4 * K1_NT, "block shapes");
static_assert(SMALL_MAXN == 4 * K3_SPAN, "spans of the largest workgroup");

template <int NQ>
struct SmallLds {
  double lw[NQ * K3_SPAN];       // log-weights; the multinomial form's cumulative weights
  int32_t marks[NQ * K3_SPAN];   // first strata, -1 between collectives
  double part[4 * NQ][3];        // the blocks' maximum, sum and sum of squares
  double xsum[4 * NQ], xvmax[4 * NQ];
  int32_t xcand[4 * NQ], xtop[4 * NQ];
  int32_t cn1;
};

struct SmallOut {
  double M, S, S2;  // as the plain combine gives them (M not yet masked by finite)
  bool finite, pos, carry;
};

__device__ __forceinline__ double lane_val(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// The collective over one workgroup's log-weights l (row layout; particles
// past N are ignored): likelihood sums, the resampling decision and, for
// every output of the rows, its ancestor.  `between` runs after the first
// barrier, while the arithmetic hides what it starts.
template <int NQ, class Between>
__device__ __forceinline__ SmallOut small_collective(SmallLds<NQ>& X, const double (&l)[ROWS],
                                                     int N, double u, const ResampleArgs& rs,
                                                     Key key, int32_t t, uint32_t b,
                                                     uint32_t iter, int32_t* pad,
                                                     int32_t (&anc)[ROWS], Between between) {
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
  const int base = w * K1_NT + lane;
  const int nb = (N + K1_NT - 1) / K1_NT;
  // the block's maximum and sums (as the plain propagation ends)
  double lc[ROWS], m = -INFINITY;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int j = base + r * WAVE;
    lc[r] = (j < N && l[r] == l[r]) ? l[r] : -INFINITY;
    m = fmax(m, lc[r]);
    X.lw[j] = l[r];
  }
  m = wave_max(m);
  {
    const bool fin = m > -INFINITY && m < INFINITY;
    double e[ROWS], s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) e[r] = fin ? exp_nonpos(lc[r] - m) : 0.0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) s1 += wave_sum(e[r]);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) s2 += wave_sum(e[r] * e[r]);
    if (lane == 0) {
      X.part[w][0] = m;
      X.part[w][1] = s1;
      X.part[w][2] = s2;
    }
  }
  __syncthreads();  // 1
  between();
  // every wave combines the blocks (lane i: block i) as a plain scan block does
  SmallOut o;
  double lo_off, hi_off;
  {
    const bool in = lane < nb;
    const double mb = in ? X.part[in ? lane : 0][0] : -INFINITY;
    const double M = wave_max(mb);
    o.finite = M > -INFINITY && M < INFINITY;
    double T = 0.0, T2 = 0.0;
    if (in && o.finite && mb > -INFINITY) {
      const double sc = exp_nonpos(mb - M);
      T = X.part[lane][1] * sc;
      T2 = X.part[lane][2] * (sc * sc);
    }
    const double incl = wave_incl_scan(T);
    o.S2 = wave_sum(T2);
    const double pre = incl - T;
    const double vin = wave_incl_max_scan(in ? pre : -INFINITY);
    const double off = fmax(pre, wave_prev(vin, -INFINITY));
    o.M = M;
    o.S = fmax(last_lane(incl), last_lane(vin));
    const int k1b = w & ~3, k1e = k1b + 4;
    lo_off = lane_val(off, k1b);
    hi_off = k1e < nb ? lane_val(off, k1e) : o.S;
  }
  const double M = o.M, S = o.S;
  o.pos = o.finite && S > 0.0;
  const double ess = o.pos ? (S * S) / o.S2 : 0.0;
  o.carry = o.pos && !(ess < rs.ess_frac * (double)N);
  const bool draws = o.pos && !o.carry;
  const bool marked = rs.scheme == RS_SYSTEMATIC || rs.scheme == RS_STRATIFIED;
  if (!draws) {  // every particle is its own offspring
#pragma unroll
    for (int r = 0; r < ROWS; ++r) anc[r] = base + r * WAVE;
    __syncthreads();  // the next collective's stores come after these reads
    return o;
  }
  if (rs.scheme == RS_METROPOLIS || rs.scheme == RS_REJECTION) {
#pragma unroll 1
    for (int r = 0; r < ROWS; ++r) {
      const int k = base + r * WAVE;
      int j = k;
      if (k < N && rs.scheme == RS_METROPOLIS) {
        auto read = [&](int i) -> double {
          const double x = X.lw[i];
          return x == x ? x : -INFINITY;
        };
        double lj = read(j);
        for (int s = 1; s <= rs.steps; s += 2) {
          const uint4 q = metro_draw(key, t, b, iter, k, s);
          int jp = metro_index(q.x, N);
          double lp = read(jp);
          if (ln_f64(u01_f64(q.y)) <= lp - lj) {
            j = jp;
            lj = lp;
          }
          if (s + 1 <= rs.steps) {
            jp = metro_index(q.z, N);
            lp = read(jp);
            if (ln_f64(u01_f64(q.w)) <= lp - lj) {
              j = jp;
              lj = lp;
            }
          }
        }
      } else if (k < N) {
        j = reject_ancestor(key, t, b, iter, k, N, M, [&](int i) { return X.lw[i]; });
      }
#pragma unroll
      for (int q = 0; q < ROWS; ++q) anc[q] = q == r ? j : anc[q];
    }
    __syncthreads();
    return o;
  }
  // the scan lane's weights (as the plain scan forms them)
  const int j0 = ROWS * tid;
  double loc[ROWS], run = 0.0;
  int cand = -1;
#pragma unroll
  for (int e = 0; e < ROWS; ++e) {
    const double lv = X.lw[j0 + e];
    const double we = (j0 + e < N && lv == lv) ? exp_nonpos(lv - M) : 0.0;
    if (we > 0.0) cand = j0 + e;
    run += we;
    loc[e] = run;
  }
  const double incl = wave_incl_scan(run);
  const int cw = wave_max_i(cand);
  if (lane == WAVE - 1) X.xsum[w] = incl;
  if (lane == 0) X.xcand[w] = cw;
  __syncthreads();  // 2
  const int wv = w & 3, w0 = w & ~3;  // this wave within its span, the span's first wave
  double pre = incl - run;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (q < wv) pre += X.xsum[w0 + q];
  double V[ROWS];
#pragma unroll
  for (int e = 0; e < ROWS; ++e) V[e] = lo_off + (pre + loc[e]);
  const double vin = wave_incl_max_scan(V[ROWS - 1]);
  const double vup = wave_prev(vin, -INFINITY);
  if (lane == WAVE - 1) X.xvmax[w] = vin;
  __syncthreads();  // 3
  double vw = -INFINITY;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (q < wv) vw = fmax(vw, X.xvmax[w0 + q]);
  const double vprev = lane > 0 ? fmax(vup, vw) : (wv > 0 ? vw : lo_off);
  double W[ROWS];
#pragma unroll
  for (int e = 0; e < ROWS; ++e) W[e] = fmin(fmax(V[e], vprev), hi_off);
  if (marked) {
    const double invS = 1.0 / S;
    const bool strat = rs.scheme == RS_STRATIFIED;
    auto count = [&](double v) -> int32_t {
      return strat ? stratum_count_strat(v, S, invS, N, key, t, b, iter)
                   : stratum_count(v, S, invS, u, N);
    };
    // the count before the lane's first particle is the previous lane's last
    // count, of the same clamped value
    int cprev = j0 < N ? count(fmin(vprev, hi_off)) : 0;
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
      const int j = j0 + e;
      if (j < N) {
        const int c = count(W[e]);
        if (cprev < c) X.marks[cprev] = j;
        cprev = c;
        if (j == N - 1) {
          X.cn1 = c;
        } else if (e == ROWS - 1 && (j & (K3_SPAN - 1)) == K3_SPAN - 1) {
          // strata below the next span's first count belong to its first particle
          if (c < count(hi_off)) X.marks[c] = j + 1;
        }
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < ROWS; ++e)
      if (j0 + e < N) X.lw[j0 + e] = W[e];
  }
  __syncthreads();  // 4
  // the last particle of positive weight takes what rounding leaves over
  auto last_positive = [&]() -> int {
    int js = -1;
    for (int q = 0; q < 4 * NQ; ++q) js = max(js, X.xcand[q]);
    return js;
  };
  if (!marked) {  // multinomial: search of the cumulative weights
#pragma unroll 1
    for (int r = 0; r < ROWS; ++r) {
      const int k = base + r * WAVE;
      int a = k;
      if (k < N) {
        const double thr = multi_u(key, t, b, iter, k) * S;
        int lo = 0, hi = N;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (X.lw[mid] > thr) hi = mid;
          else lo = mid + 1;
        }
        a = lo < N ? lo : max(0, last_positive());
      }
#pragma unroll
      for (int q = 0; q < ROWS; ++q) anc[q] = q == r ? a : anc[q];
    }
    __syncthreads();
    return o;
  }
  // owners: a running maximum of the marks over the strata
  int mk[ROWS], top = -1;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int k = base + r * WAVE;
    const int v = X.marks[k];
    X.marks[k] = -1;
    mk[r] = max(wave_incl_max_scan_rows(v), top);
    top = __builtin_amdgcn_readlane(mk[r], WAVE - 1);
  }
  if (lane == 0) X.xtop[w] = top;
  __syncthreads();  // 5
  int before = -1;
#pragma unroll
  for (int q = 0; q < 4 * NQ; ++q)
    if (q < w) before = max(before, X.xtop[q]);
  const int cn1 = X.cn1;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int k = base + r * WAVE;
    int a = max(before, mk[r]);
    if (k >= cn1 && k < N) a = last_positive();
    if (k < N && (a < 0 || a >= N)) {  // never expected; flagged, and kept in bounds
      if (pad) atomicOr(pad, 1);
      a = 0;
    }
    anc[r] = a;
  }
  return o;
}

// ---------------------------------------------------------------- pf_systematic
template <int NQ>
__global__ __launch_bounds__(K3_NT* NQ) void k_small_systematic(const double* __restrict__ lw,
                                                                int N, double u,
                                                                int32_t* __restrict__ anc,
                                                                double* __restrict__ stats) {
  __shared__ SmallLds<NQ> X;
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
  const int base = w * K1_NT + lane;
  double l[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    l[r] = lw[min(base + r * WAVE, N - 1)];
    X.marks[base + r * WAVE] = -1;
  }
  int32_t a[ROWS];
  const ResampleArgs rs{RS_SYSTEMATIC, 0, INFINITY};
  const SmallOut o = small_collective<NQ>(X, l, N, u, rs, Key{0, 0}, 0, 0, 0, nullptr, a, [] {});
#pragma unroll
  for (int r = 0; r < ROWS; ++r)
    if (base + r * WAVE < N) anc[base + r * WAVE] = a[r];
  if (threadIdx.x == 0) {
    const double lprev = log((double)N);
    stats[0] = o.pos ? (o.M + log(o.S)) - lprev : -INFINITY;
    stats[1] = o.pos ? (o.S * o.S) / o.S2 : 0.0;
  }
}

hipError_t launch_small_systematic(const double* lw, int n, double u, int32_t* anc, double* stats,
                                   hipStream_t s) {
  if (n < 1 || n > SMALL_MAXN) return hipErrorInvalidValue;
  if (n <= K3_SPAN)
    hipLaunchKernelGGL(k_small_systematic<1>, 1, K3_NT, 0, s, lw, n, u, anc, stats);
  else if (n <= 2 * K3_SPAN)
    hipLaunchKernelGGL(k_small_systematic<2>, 1, 2 * K3_NT, 0, s, lw, n, u, anc, stats);
  else
    hipLaunchKernelGGL(k_small_systematic<4>, 1, 4 * K3_NT, 0, s, lw, n, u, anc, stats);
  return hipGetLastError();
}

}  // namespace pfk
