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
// waiting on memory: 10.8 us per interval for 1,024 windkessel particles in
// FP64 (17.6 before its kernels' chains were shortened), 3.4 of them between
// kernels.  In one workgroup an interval needs no launch
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

// The collective over one workgroup's log-weights l (row layout; particles
// past N are ignored): likelihood sums, the resampling decision and, for
// every output of the rows, its ancestor.  `between` runs after the first
// barrier, while the arithmetic hides what it starts.
// SYS: systematic resampling (any scheme otherwise: a kernel with all of
// them spends most of its registers on their constants).
template <int NQ, bool SYS, class Between>
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
    X.lw[j] = lc[r];  // a NaN is a weight of 0 to every scheme
  }
  m = wave_max(m);
  {
    // (without a finite maximum lc - m is -inf or NaN and the weight 0)
    double e[ROWS], s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) e[r] = exp_nonpos(lc[r] - m);
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
    lo_off = lane_value(off, k1b);
    hi_off = k1e < nb ? lane_value(off, k1e) : o.S;
  }
  const double M = o.M, S = o.S;
  o.pos = o.finite && S > 0.0;
  const double ess = o.pos ? (S * S) / o.S2 : 0.0;
  o.carry = o.pos && !(ess < rs.ess_frac * (double)N);
  const bool draws = o.pos && !o.carry;
  const bool marked = SYS || rs.scheme == RS_SYSTEMATIC || rs.scheme == RS_STRATIFIED;
  if (!draws) {  // every particle is its own offspring
#pragma unroll
    for (int r = 0; r < ROWS; ++r) anc[r] = base + r * WAVE;
    __syncthreads();  // the next collective's stores come after these reads
    return o;
  }
  if (!SYS && (rs.scheme == RS_METROPOLIS || rs.scheme == RS_REJECTION)) {
#pragma unroll 1
    for (int r = 0; r < ROWS; ++r) {
      const int k = base + r * WAVE;
      int j = k;
      if (k < N && rs.scheme == RS_METROPOLIS) {
        double lj = X.lw[j];
        for (int s = 1; s <= rs.steps; s += 2) {
          const uint4 q = metro_draw(key, t, b, iter, k, s);
          int jp = metro_index(q.x, N);
          double lp = X.lw[jp];
          if (ln_u_leq(q.y, lp - lj)) {
            j = jp;
            lj = lp;
          }
          if (s + 1 <= rs.steps) {
            jp = metro_index(q.z, N);
            lp = X.lw[jp];
            if (ln_u_leq(q.w, lp - lj)) {
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
    const double we = exp_nonpos(X.lw[j0 + e] - M);  // 0 past N
    cand = we > 0.0 ? j0 + e : cand;
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
    const bool strat = !SYS && rs.scheme == RS_STRATIFIED;
    auto count = [&](double v) -> int32_t {
      return strat ? stratum_count_strat(v, S, invS, N, key, t, b, iter)
                   : stratum_count(v, S, invS, u, N);
    };
    // c[e + 1]: the count of the lane's particle e; c[0]: the one before its
    // first, the previous lane's last, of the same clamped value
    const double v[ROWS + 1] = {fmin(vprev, hi_off), W[0], W[1], W[2], W[3]};
    int32_t c[ROWS + 1];
    if (strat) {
#pragma unroll
      for (int e = 0; e <= ROWS; ++e) c[e] = count(v[e]);
    } else {
      stratum_counts(v, S, invS, u, N, j0 < N ? ROWS + 1 : 0, c);
    }
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
      const int j = j0 + e;
      if (j < N && c[e] < c[e + 1]) X.marks[c[e]] = j;
    }
    const int jl = j0 + ROWS - 1;
    if (j0 < N && jl >= N - 1) {  // the lane of the last particle
      X.cn1 = N - 1 == j0 ? c[1] : N - 1 == j0 + 1 ? c[2] : N - 1 == j0 + 2 ? c[3] : c[4];
    } else if (jl < N && (jl & (K3_SPAN - 1)) == K3_SPAN - 1) {
      // strata below the next span's first count belong to its first particle
      if (c[ROWS] < count(hi_off)) X.marks[c[ROWS]] = jl + 1;
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
  const SmallOut o = small_collective<NQ, true>(X, l, N, u, rs, Key{0, 0}, 0, 0, 0, nullptr, a, [] {});
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

// ---------------------------------------------------------------- windkessel runs
// One interval's record: the resampling uniform, Z q(t), y(t), then c q of
// its K substeps (FP32 forms: the FP32 product), each as the multi-kernel
// path forms it.
constexpr int REC_HEAD = 3;

// The random numbers of n intervals from every filter's counter on: sigma_p z
// (FP64; the FP32 forms keep z, which enters a fused multiply-add), and the
// intervals' records.  Every filter has W = small_width(max_n) numbers, whole
// 256-particle blocks but in a filter of a single row; within a block a lane's
// four rows lie together: nz[((i K + s) B + b) W + 256 block + 4 lane + row].
// One lane per particle and interval (numbers past a filter's end are not
// drawn); bound by the normals' FP64 instructions (1,024 particles, 100
// intervals of K = 10: 13.4 us for all of them).
template <typename Real>
__global__ __launch_bounds__(K1_NT) void k_small_noise(PlainArgs A,
                                                       const int64_t* __restrict__ offs,
                                                       Real* __restrict__ nz,
                                                       double* __restrict__ rec, int n, int W) {
  const int i = blockIdx.y, b = blockIdx.z;
  const int N = (int)(offs[b + 1] - offs[b]);
  const FilterState* fs = A.fs + b;
  const uint32_t iter = fs->iter;
  const int t = fs->t + 1 + i;
  const int n0 = (t - 1) * A.K;
  const double* th = A.theta + (size_t)b * 8;
  const Key key{A.key.lo, A.key.hi};
  if (blockIdx.x == 0) {
    double* o = rec + ((int64_t)b * n + i) * (A.K + REC_HEAD);
    for (int s = threadIdx.x; s < A.K + REC_HEAD; s += K1_NT) {
      double v;
      if (s == 0)
        v = u01_f64(draw(key, TAG_RESAMPLE, 0, iter, 0, (uint32_t)t, (uint32_t)b).x);
      else if (s == 1)
        v = th[2] * A.q[(int64_t)t * A.K];
      else if (s == 2)
        v = A.obs[t - 1];
      else if constexpr (sizeof(Real) == 8)
        v = th[1] * A.q[n0 + s - REC_HEAD];
      else
        v = (double)((float)th[1] * (float)A.q[n0 + s - REC_HEAD]);
      o[s] = v;
    }
  }
  // thread 4 lane + row of the block
  const int j = blockIdx.x * K1_NT + (threadIdx.x & 3) * WAVE + (threadIdx.x >> 2);
  if (j >= N) return;
  const int64_t step = (int64_t)gridDim.z * W;
  Real* o = nz + (int64_t)i * A.K * step + (int64_t)b * W + blockIdx.x * K1_NT + threadIdx.x;
  for (int s = 1; s <= A.K; ++s, o += step) {
    const uint4 w = draw(key, TAG_NOISE, 0, iter, (uint32_t)j, (uint32_t)(n0 + s), (uint32_t)b);
    if constexpr (sizeof(Real) == 8) {
      double z0, z1;
      bm_pair_f64(w.x, w.y, z0, z1);
      *o = th[3] * z0;
    } else {
      float z0, z1;
      bm_pair_f32(w.x, w.y, z0, z1);
      *o = z0;
    }
  }
}

// n intervals of one filter per workgroup, from the ancestors pending as the
// identity or the array; leaves what the multi-kernel path leaves, with the
// ancestors in the array.  Bound by the chain of an interval: the substeps'
// dependent adds, two exponentials, five barriers.  The next interval's
// numbers are loaded during the collective, and the likelihood's logarithms
// wait for 64 intervals to be taken by 64 lanes.  1,024 particles, K = 10,
// FP64: 5.3 us an interval (10.8 on the multi-kernel path's graphs).
template <typename Real, bool ACC, int NQ, bool SYS>
__global__ __launch_bounds__(K3_NT* NQ) void k_small_run(Real* __restrict__ xa,
                                                         Real* __restrict__ xb,
                                                         double* __restrict__ lw,
                                                         int32_t* __restrict__ anc_all,
                                                         PlainArgs A,
                                                         const int64_t* __restrict__ offs,
                                                         const Real* __restrict__ nz,
                                                         const double* __restrict__ rec, int n,
                                                         int W) {
  constexpr int NT = K3_NT * NQ;
  // substeps loaded ahead, as many as the registers leave room for
  constexpr int AHEAD = NQ == 4 ? 4 : 12;
  typedef Real Row4 __attribute__((ext_vector_type(ROWS)));
  constexpr int RING = WAVE;
  __shared__ SmallLds<NQ> X;
  __shared__ Real xs[2][NQ * K3_SPAN];
  __shared__ double recL[2][SMALL_MAXK + REC_HEAD];
  __shared__ double rM[RING], rS[RING], rS2[RING];
  __shared__ int32_t rflag[RING];  // 1: a positive weight, 2: weights kept
  const int b = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int base = wave * K1_NT + lane;
  const int64_t off = offs[b];
  const int N = (int)(offs[b + 1] - off), K = A.K;
  FilterState* fs = A.fs + b;
  const int t0 = fs->t;
  const uint32_t iter = fs->iter;
  const int amode = fs->amode;
  // marks are the caller's to write out first: flagged, not run past silently
  if (tid == 0 && amode == AMODE_MARKS) atomicOr(&fs->pad, 1);
  bool carry = fs->carry != 0;
  const double* th = A.theta + (size_t)b * 8;
  const Key key{A.key.lo, A.key.hi};
  const double a64 = th[0];
  const float am1 = (float)(th[0] - 1.0), sp = (float)th[3];
  // this wave's block of numbers, from the lane's on (a wave or a lane past the
  // filter's reads the last)
  const int64_t step = (int64_t)gridDim.x * W;
  nz += (int64_t)b * W + min(wave, (W - 1) / K1_NT) * K1_NT + ROWS * min(lane, W / ROWS - 1);
  rec += (int64_t)b * n * (K + REC_HEAD);
  double* ell_tr = A.ell_tr + (int64_t)b * A.T;
  double* ess_tr = A.ess_tr + (int64_t)b * A.T;
  uint32_t jr[ROWS];
  Real p[ROWS];
  double l[ROWS];
  int32_t anc[ROWS];
  const Real* x0 = (t0 & 1) ? xb : xa;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    jr[r] = min(base + r * WAVE, N - 1);
    X.marks[base + r * WAVE] = -1;
    const int a = amode == AMODE_ARRAY ? anc_all[off + jr[r]] : (int)jr[r];
    p[r] = x0[off + a];
    l[r] = carry ? lw[off + jr[r]] : 0.0;
    anc[r] = base + r * WAVE;
  }
  Row4 zn[AHEAD];
  auto load_ahead = [&](int i) {
    const Real* zi = nz + (int64_t)i * K * step;
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
      if (s < K) zn[s] = *(const Row4*)(zi + s * step);
  };
  load_ahead(0);
  if (tid < K + REC_HEAD) recL[0][tid] = rec[tid];
  __syncthreads();
  // the running scalars, held by wave 0
  double loglik = fs->loglik, lprev = fs->lprev, ell_last = 0.0, ess_last = 0.0;
  bool carry_before = carry, none = false;
  SmallOut o{};
  for (int i = 0; i < n; ++i) {
    const int par = i & 1;
    const double* R = recL[par];
    const bool more = i + 1 < n;
    double rn = 0.0;
    if (more && tid < K + REC_HEAD) rn = rec[(int64_t)(i + 1) * (K + REC_HEAD) + tid];
    double pa[ROWS];  // the accurate form carries the pressure in FP64
#pragma unroll
    for (int r = 0; r < ROWS; ++r) pa[r] = (double)p[r];
    auto substep = [&](double cq, const Row4& z) {
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        if constexpr (sizeof(Real) == 8)
          p[r] = (a64 * p[r] + cq) + z[r];
        else if constexpr (ACC)
          pa[r] = pa[r] + (double)fmaf(sp, z[r], fmaf(am1, (float)pa[r], (float)cq));
        else
          p[r] = p[r] + fmaf(sp, z[r], fmaf(am1, p[r], (float)cq));
      }
    };
    {
      const double head = R[min(lane, SMALL_MAXK - 1) + REC_HEAD];  // c q of substep `lane`
#pragma unroll
      for (int s = 0; s < AHEAD; ++s)
        if (s < K) substep(lane_value(head, s), zn[s]);
      const Real* zi = nz + (int64_t)i * K * step;
      for (int s0 = AHEAD; s0 < K; s0 += 4) {
        Row4 z[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) z[s] = *(const Row4*)(zi + min(s0 + s, K - 1) * step);
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (s0 + s < K) substep(R[REC_HEAD + s0 + s], z[s]);
      }
    }
    const double u = R[0], zq = R[1], y = R[2];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      if constexpr (ACC) p[r] = (Real)pa[r];
      else pa[r] = (double)p[r];
      const double e = (y - (pa[r] + zq)) * A.inv_sd;
      const double ln = -0.5 * (e * e) + A.lw_cst;
      l[r] = carry ? l[r] + ln : ln;
      xs[par][base + r * WAVE] = p[r];
    }
    o = small_collective<NQ, SYS>(X, l, N, u, A.rs, key, t0 + 1 + i, (uint32_t)b, iter, &fs->pad, anc,
                             [&] {
                               if (tid < K + REC_HEAD) recL[par ^ 1][tid] = rn;
                               if (more) load_ahead(i + 1);
                             });
    carry = o.carry;
    if (more)
#pragma unroll
      for (int r = 0; r < ROWS; ++r)
        if (base + r * WAVE < N) p[r] = xs[par][anc[r]];
    // the bookkeeping of up to 64 intervals at once, by wave 0
    if (tid < WAVE) {
      const int k = i & (RING - 1);
      if (tid == 0) {
        rM[k] = o.M;
        rS[k] = o.S;
        rS2[k] = o.S2;
        rflag[k] = (o.pos ? 1 : 0) | (o.carry ? 2 : 0);
      }
      if (k == RING - 1 || !more) {
        __builtin_amdgcn_wave_barrier();
        const bool in = lane <= k;
        const int fl = in ? rflag[lane] : 0;
        const double S = in ? rS[lane] : 1.0;
        const bool pos = fl & 1;
        const double L = pos ? rM[in ? lane : 0] + log(S) : 0.0;
        // the factor's normaliser: ln N after a resampling, else the carried
        // weights' ln sum exp
        const double Lp = wave_prev(L, lprev);
        const int kept = dpp_move_i<0x138, 0xf>(fl, carry_before ? 2 : 0) & 2;
        const double ell = pos ? L - (kept ? Lp : log((double)N)) : -INFINITY;
        const double ess = pos ? (S * S) / rS2[in ? lane : 0] : 0.0;
        if (in) {
          ell_tr[t0 + i - k + lane] = ell;
          ess_tr[t0 + i - k + lane] = ess;
        }
        none = none || __ballot(in && !pos) != 0;
        for (int q = 0; q <= k; ++q) loglik = loglik + lane_value(ell, q);
        lprev = lane_value(L, k);
        ell_last = lane_value(ell, k);
        ess_last = lane_value(ess, k);
        carry_before = o.carry;
      }
    }
  }
  const int t = t0 + n;
  Real* xn = (t & 1) ? xb : xa;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int j = base + r * WAVE;
    if (j < N) {
      xn[off + j] = p[r];
      lw[off + j] = l[r];
      anc_all[off + j] = anc[r];
    }
  }
  if (tid == 0) {
    fs->loglik = loglik;
    fs->M = o.finite ? o.M : -INFINITY;
    fs->S = o.S;
    fs->u = recL[(n - 1) & 1][0];
    fs->ell = ell_last;
    fs->ess = ess_last;
    fs->t = t;
    if (none) fs->status = 4;
    fs->lprev = lprev;
    fs->carry = o.carry;
    fs->tk = t;
    fs->cn1 = 0;
    fs->amode = AMODE_ARRAY;
  }
}

template <typename Real, bool ACC>
static void small_run(int nq, int W, int B, void* xa, void* xb, double* lw, int32_t* anc,
                      const PlainArgs& a, const int64_t* off, const void* nz, const double* rec,
                      int n, hipStream_t s) {
#define PF_SMALL(Q, SYS)                                                                       \
  hipLaunchKernelGGL((k_small_run<Real, ACC, Q, SYS>), (unsigned)B, K3_NT* Q, 0, s, (Real*)xa, \
                     (Real*)xb, lw, anc, a, off, (const Real*)nz, rec, n, W)
  const bool sys = a.rs.scheme == RS_SYSTEMATIC;
  if (nq == 1) {
    if (sys) PF_SMALL(1, true);
    else PF_SMALL(1, false);
  } else if (nq == 2) {
    if (sys) PF_SMALL(2, true);
    else PF_SMALL(2, false);
  } else {
    if (sys) PF_SMALL(4, true);
    else PF_SMALL(4, false);
  }
#undef PF_SMALL
}

hipError_t launch_small_run(int prec, int B, int max_n, void* xa, void* xb, double* lw,
                            int32_t* anc, const PlainArgs& a, const int64_t* off, void* nz,
                            double* rec, int n, hipStream_t s) {
  if (max_n < 1 || max_n > SMALL_MAXN || a.K > SMALL_MAXK || n < 1 || B < 1 || B > 65535 ||
      n > 65535)
    return hipErrorInvalidValue;
  const int W = small_width(max_n);
  const dim3 g((unsigned)((max_n + K1_NT - 1) / K1_NT), (unsigned)n, (unsigned)B);
  if (prec == 0)
    hipLaunchKernelGGL(k_small_noise<double>, g, K1_NT, 0, s, a, off, (double*)nz, rec, n, W);
  else
    hipLaunchKernelGGL(k_small_noise<float>, g, K1_NT, 0, s, a, off, (float*)nz, rec, n, W);
  const int nq = max_n <= K3_SPAN ? 1 : max_n <= 2 * K3_SPAN ? 2 : 4;
  if (prec == 0) small_run<double, false>(nq, W, B, xa, xb, lw, anc, a, off, nz, rec, n, s);
  else if (prec == 1) small_run<float, false>(nq, W, B, xa, xb, lw, anc, a, off, nz, rec, n, s);
  else small_run<float, true>(nq, W, B, xa, xb, lw, anc, a, off, nz, rec, n, s);
  return hipGetLastError();
}

}  // namespace pfk
