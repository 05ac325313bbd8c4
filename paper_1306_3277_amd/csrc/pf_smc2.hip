// SMC over the parameters with a particle filter attached to every
// theta-particle (Sec. 3.2.2, Alg. 4; SMC^2 when the filter is Alg. 2), on
// top of the batched layout: theta-particle j owns filter slot j.
//
//   k_theta_resample    one workgroup: theta-weights v_j = ell_j of the last
//                       interval, their max, FP64 sums and scan, ESS, the
//                       evidence factor, systematic theta-ancestors by binary
//                       search of the scan, and the move of parameters,
//                       likelihood and status to the new slots.
//   k_filter_gather     whole-filter copies (systematic selection when the
//                       particle counts differ) of the slots whose ancestor
//                       is another slot, into the spare state buffer.
//   k_smc2_start        the copies become the slots' particles; random-walk
//                       proposals inside the prior box, written as the
//                       proposal handle's derived parameters; the proposal
//                       filters' initial states and scalars.
//   k_smc2_finish       Metropolis-Hastings decision per theta-particle
//                       (Alg. 3, eq. mh) after the proposal filters ran;
//                       accepted slots take the proposal filter's particles.
//   k_smc2_propose      the proposals alone (attached Kalman filters).
//
// A time's work besides the filters is small (a few MB of copies, B decisions)
// and was nine launches of 3 to 11 us with 2 us between them; what needs no
// other workgroup's result shares a launch, so it is four.  64 theta-particles
// of 2,048: 48 -> 24 us of kernels a time, 15.6 -> 14.7 ms for 40 times.
#include <math.h>

#include "pf_device.hpp"
#include "pf_smc2.hpp"

namespace pfk {

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ double block_max_1024(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l == 0) red[w] = v;
  __syncthreads();
  double r = red[0];
  for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = fmax(r, red[i]);
  __syncthreads();
  return r;
}

__device__ __forceinline__ double block_sum_1024(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) r += red[i];
  __syncthreads();
  return r;
}

// Whole-filter copy index: destination particle k of n_dst takes source
// particle floor((k + w 2^-32) n_src / n_dst) (systematic selection on equal
// weights), exact in 64-bit integers for counts up to 2^13.
__device__ __forceinline__ int64_t copy_index(int64_t k, int64_t n_src, int64_t n_dst,
                                              uint32_t w) {
  const uint64_t num = (((uint64_t)k << 32) | (uint64_t)w) * (uint64_t)n_src;
  return (int64_t)(num / ((uint64_t)n_dst << 32));
}

// ---------------------------------------------------------------- theta layer

// One workgroup, a lane per theta-particle up to SMC2_NT lanes, and a wave more
// for the evidence where they leave room.  v_j = ell_tr[j*T + col].  Writes the
// theta-ESS and adds ln(sum exp v) - ln B to *evid.  With draw != 0 also
// draws a[k] = min{j : B W_j > (u + k) S} (W the inclusive scan of
// exp(v - max)), falling back to the last positive weight, and moves the
// parameters (raw and derived), likelihood and status of slot a[k] to slot
// k.  If no theta-weight is positive the ancestors are the identity and
// *numeric is set.
__global__ __launch_bounds__(SMC2_NT) void k_theta_resample(Smc2Args S, int32_t col, double u,
                                                            int32_t draw, int32_t* anc_tr_row,
                                                            double* ess_out) {
  __shared__ double W[SMC2_MAXB];
  __shared__ double red[SMC2_NT / 64];
  __shared__ int ired[SMC2_NT / 64];
  const int B = S.B;
  const int tid = threadIdx.x;
  // this lane's contiguous range of theta-particles
  const int nt = blockDim.x, nw = nt >> 6;
  const int per = (B + nt - 1) / nt;
  const int j0 = tid * per, j1 = min(B, j0 + per);
  double m = -INFINITY;
  for (int j = j0; j < j1; ++j) {
    const double v = S.ell_tr[(int64_t)j * S.T + col];
    if (v > m) m = v;
  }
  const double M = block_max_1024(m, red);
  const bool numeric = !(M > -INFINITY) || !(M < INFINITY);
  double acc = 0.0, acc2 = 0.0;
  int jstar = -1;
  if (!numeric) {
    for (int j = j0; j < j1; ++j) {
      const double w = exp_nonpos(S.ell_tr[(int64_t)j * S.T + col] - M);
      acc = acc + w;
      acc2 = acc2 + w * w;
      W[j] = acc;  // local inclusive scan, offset below
      if (w > 0.0) jstar = j;
    }
  }
  // exclusive scan of the lanes' sums (sequential over the wave sums)
  double x = acc;
  const int lane = tid & 63, wv = tid >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const double y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) red[wv] = x;
  int js = jstar;
  for (int o = 32; o > 0; o >>= 1) js = max(js, __shfl_xor(js, o));
  if (lane == 0) ired[wv] = js;
  __syncthreads();
  double base = 0.0;
  for (int i = 0; i < wv; ++i) base += red[i];
  double total = 0.0;
  int jst = -1;
  for (int i = 0; i < nw; ++i) {
    total += red[i];
    jst = max(jst, ired[i]);
  }
  const double excl = base + x - acc;
  if (!numeric)
    for (int j = j0; j < j1; ++j) W[j] += excl;
  __syncthreads();  // every lane has read red before it is reused
  const double S2 = block_sum_1024(acc2, red);  // its barriers also order the W writes
  if (tid == nt - 64) {  // (the last wave: with up to 960 lanes, one without a particle)
    *S.numeric = *S.numeric | (numeric ? 1 : 0);
    if (numeric) {
      *ess_out = 0.0;
      *S.evid = -INFINITY;
    } else {
      *ess_out = (total * total) / S2;
      *S.evid = *S.evid + ((M + log(total)) - log((double)B));
    }
  }
  if (!draw) return;
  // ancestors by binary search of the scan
  const double Bd = (double)B;
  int own = tid;  // the first slot's ancestor
  for (int k = tid; k < B; k += nt) {
    int a = k;
    if (!numeric) {
      const double thr = (u + (double)k) * total;
      int lo = 0, hi = B;  // first j with B W_j > thr, or B
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (Bd * W[mid] > thr) hi = mid;
        else lo = mid + 1;
      }
      a = lo < B ? lo : jst;
    }
    S.a[k] = a;
    if (k == tid) own = a;
    if (anc_tr_row) anc_tr_row[k] = a;
  }
  if (per == 1) {  // every slot's values wait in its lane's registers
    double dev[8], raw[8], ll = 0.0, mv[2] = {0.0, 0.0};
    int32_t st = 0;
    const bool in = tid < B;
    if (in) {
#pragma unroll
      for (int p = 0; p < 8; ++p) dev[p] = S.theta_dev[(int64_t)own * 8 + p];
#pragma unroll
      for (int p = 0; p < 8; ++p)
        if (p < S.n_theta) raw[p] = S.raw[(int64_t)own * S.n_theta + p];
      ll = S.fs[own].loglik;
      st = S.fs[own].status;
      if (S.mV) {
        mv[0] = S.mV[2 * own];
        mv[1] = S.mV[2 * own + 1];
      }
    }
    __syncthreads();
    if (in) {
#pragma unroll
      for (int p = 0; p < 8; ++p) S.theta_dev[(int64_t)tid * 8 + p] = dev[p];
#pragma unroll
      for (int p = 0; p < 8; ++p)
        if (p < S.n_theta) S.raw[(int64_t)tid * S.n_theta + p] = raw[p];
      S.fs[tid].loglik = ll;
      S.fs[tid].status = st;
      if (S.mV) {
        S.mV[2 * tid] = mv[0];
        S.mV[2 * tid + 1] = mv[1];
      }
    }
    return;
  }
  // snapshot the slots' parameters, likelihoods and status, then move them
  for (int j = tid; j < B; j += nt) {
    for (int p = 0; p < 8; ++p) S.snap_dev[(int64_t)j * 8 + p] = S.theta_dev[(int64_t)j * 8 + p];
    for (int p = 0; p < S.n_theta; ++p)
      S.snap_raw[(int64_t)j * S.n_theta + p] = S.raw[(int64_t)j * S.n_theta + p];
    S.snap_ll[j] = S.fs[j].loglik;
    S.snap_st[j] = S.fs[j].status;
    if (S.mV) {
      S.snap_mV[2 * j] = S.mV[2 * j];
      S.snap_mV[2 * j + 1] = S.mV[2 * j + 1];
    }
  }
  __syncthreads();
  for (int j = tid; j < B; j += nt) {
    const int s = S.a[j];
    for (int p = 0; p < 8; ++p) S.theta_dev[(int64_t)j * 8 + p] = S.snap_dev[(int64_t)s * 8 + p];
    for (int p = 0; p < S.n_theta; ++p)
      S.raw[(int64_t)j * S.n_theta + p] = S.snap_raw[(int64_t)s * S.n_theta + p];
    S.fs[j].loglik = S.snap_ll[s];
    S.fs[j].status = S.snap_st[s];
    if (S.mV) {
      S.mV[2 * j] = S.snap_mV[2 * s];
      S.mV[2 * j + 1] = S.snap_mV[2 * s + 1];
    }
  }
}

// Pass 1 of the whole-filter copies: slot f whose theta-ancestor s differs
// takes s's equally weighted particles, i.e. the propagated states at s's
// pending ancestors, written to the spare buffer.
template <typename Real>
__global__ __launch_bounds__(BATCH_NT) void k_filter_gather(const Real* __restrict__ xcur,
                                                            Real* __restrict__ xspare,
                                                            const int32_t* __restrict__ anc,
                                                            BatchArgs A, Smc2Args S,
                                                            const uint32_t* __restrict__ w) {
  const int f = A.chunk_f[blockIdx.x];
  const int s = S.a[f];
  if (s == f) return;
  const int64_t off = A.off[f], n = A.off[f + 1] - off;
  const int64_t k = (int64_t)A.chunk_k[blockIdx.x] + threadIdx.x;
  if (k >= n) return;
  const int64_t soff = A.off[s], sn = A.off[s + 1] - soff;
  const int64_t p = copy_index(k, sn, n, w[f]);
  const int64_t src = soff + anc[soff + p];
  for (int i = 0; i < A.d; ++i) xspare[(int64_t)i * A.ld + off + k] = xcur[(int64_t)i * A.ld + src];
}

// Slot j's proposal: theta' = theta + step_sd z on the moved parameters (two
// roundings, no contraction); returns whether every moved parameter lies
// within [lo, hi].  dev: the derived parameters of theta' (or of theta when
// outside: that slot's proposal run is then unused).
__device__ __forceinline__ int propose(const Smc2Args& S, const double* __restrict__ z_row, int j,
                                       double (&th)[8], double (&dev)[8]) {
  const int nt = S.n_theta;
  int inside = 1;
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    th[p] = 0.0;
    if (p < nt) {
      th[p] = S.raw[(int64_t)j * nt + p];
      if (S.step_sd[p] != 0.0) {
        const double step = __dmul_rn(S.step_sd[p], z_row[(int64_t)j * nt + p]);
        th[p] = __dadd_rn(th[p], step);
        if (!(th[p] >= S.lo[p] && th[p] <= S.hi[p])) inside = 0;
      }
    }
  }
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    if (!inside) dev[p] = S.theta_dev[(int64_t)j * 8 + p];
    else if (S.model == 1) dev[p] = p < 6 ? th[p] : 0.0;
    else dev[p] = p == 0 ? th[0] : p == 1 ? __dmul_rn(th[1], S.sqrt_h) : 0.0;
  }
  return inside;
}

__device__ __forceinline__ void store_proposal(const Smc2Args& S, int j, int inside,
                                               const double (&th)[8], const double (&dev)[8],
                                               double* __restrict__ prop_dev) {
#pragma unroll
  for (int p = 0; p < 8; ++p)
    if (p < S.n_theta) S.prop_raw[(int64_t)j * S.n_theta + p] = th[p];
  S.inside[j] = inside;
#pragma unroll
  for (int p = 0; p < 8; ++p) prop_dev[(int64_t)j * 8 + p] = dev[p];
}

__global__ void k_smc2_propose(Smc2Args S, const double* __restrict__ z_row,
                               double* __restrict__ prop_dev) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= S.B) return;
  double th[8], dev[8];
  const int inside = propose(S, z_row, j, th, dev);
  store_proposal(S, j, inside, th, dev, prop_dev);
}

// A block per chunk of a slot's particles.  With `copied`, a slot whose
// theta-ancestor is another takes its copied particles from the spare buffer
// as its equally weighted set.  Every block forms its slot's proposal (the
// block of the first chunk stores it, and the likelihood the decision
// compares with) and draws its part of the proposal filter's initial state,
// as an initialisation of that handle at iteration `iter` would; the blocks
// together clear its traces.
template <int MODEL, int D, typename Real>
__global__ __launch_bounds__(BATCH_NT) void k_smc2_start(Real* __restrict__ xcur,
                                                         const Real* __restrict__ xspare,
                                                         int32_t* __restrict__ anc,
                                                         const double* __restrict__ z_row,
                                                         SmcProposal P, uint32_t iter, int copied,
                                                         BatchArgs A, Smc2Args S) {
  const int f = A.chunk_f[blockIdx.x];
  const int64_t off = A.off[f], n = A.off[f + 1] - off;
  const int k0 = A.chunk_k[blockIdx.x];
  const int64_t k = (int64_t)k0 + threadIdx.x;
  for (int64_t i = (int64_t)blockIdx.x * BATCH_NT + threadIdx.x; i < (int64_t)S.B * S.T;
       i += (int64_t)gridDim.x * BATCH_NT) {
    P.ell_tr[i] = 0.0;
    P.ess_tr[i] = 0.0;
  }
  double th[8], dev[8];
  const int inside = propose(S, z_row, f, th, dev);
  if (k0 == 0 && threadIdx.x == 0) {
    store_proposal(S, f, inside, th, dev, P.theta_dev);
    S.snap_ll[f] = S.fs[f].loglik;
    FilterState o = {};
    o.iter = iter;
    o.amode = AMODE_IDENTITY;
    P.fs[f] = o;
  }
  if (k >= n) return;
  if (copied && S.a[f] != f) {
    Real v[D];
#pragma unroll
    for (int i = 0; i < D; ++i) v[i] = xspare[(int64_t)i * A.ld + off + k];
#pragma unroll
    for (int i = 0; i < D; ++i) xcur[(int64_t)i * A.ld + off + k] = v[i];
    anc[off + k] = (int32_t)k;
  }
  Real* x = (Real*)P.x;
  P.anc[off + k] = (int32_t)k;
  const Key key{A.key.lo, A.key.hi};
  if constexpr (MODEL == 1) {
    double z0, z1;
    const uint4 w = draw(key, TAG_INIT, 0, iter, (uint32_t)k, 0, (uint32_t)f);
    bm_pair_f64(w.x, w.y, z0, z1);
    x[off + k] = (Real)(dev[4] + dev[5] * z0);
  } else {
#pragma unroll
    for (int blk = 0; blk < D / 4; ++blk) {
      double z[4];
      normals4_f64(draw(key, TAG_INIT, blk, iter, (uint32_t)k, 0, (uint32_t)f), z);
#pragma unroll
      for (int m = 0; m < 4; ++m) x[(int64_t)(4 * blk + m) * A.ld + off + k] = (Real)z[m];
    }
  }
}

// Accept iff inside and log_alpha <= l' - l (ties accept).  Every block of a
// slot's chunks decides for itself, from values none of them changes.  An
// accepted slot takes theta', its derived form, l', the proposal filter's
// status and its equally weighted particles.
template <int D, typename Real>
__global__ __launch_bounds__(BATCH_NT) void k_smc2_finish(
    Real* __restrict__ xcur, int32_t* __restrict__ anc,
    const double* __restrict__ log_alpha_row, int32_t* __restrict__ acc_tr_row,
    double* __restrict__ theta_tr_row, SmcProposal P, BatchArgs A, Smc2Args S) {
  const int f = A.chunk_f[blockIdx.x];
  const int64_t off = A.off[f], n = A.off[f + 1] - off;
  const int k0 = A.chunk_k[blockIdx.x];
  const int64_t k = (int64_t)k0 + threadIdx.x;
  const double l_new = P.fs[f].loglik;
  const int32_t st_new = P.fs[f].status;
  const double lp = st_new ? -INFINITY : l_new;
  const int acc = S.inside[f] && (log_alpha_row[f] <= lp - S.snap_ll[f]);
  if (k0 == 0 && threadIdx.x == 0) {
    acc_tr_row[f] = acc;
    const int64_t r0 = (int64_t)f * S.n_theta;
    for (int p = 0; p < S.n_theta; ++p) {
      const double v = acc ? S.prop_raw[r0 + p] : S.raw[r0 + p];
      if (acc) S.raw[r0 + p] = v;
      theta_tr_row[r0 + p] = v;
    }
    if (acc) {
      S.accepts[f] += 1;
      for (int p = 0; p < 8; ++p) S.theta_dev[(int64_t)f * 8 + p] = P.theta_dev[(int64_t)f * 8 + p];
      S.fs[f].loglik = l_new;
      S.fs[f].status = st_new;
    }
  }
  if (!acc || k >= n) return;
  const Real* px = (const Real*)P.x;
  const int64_t src = off + P.anc[off + k];
  Real v[D];
#pragma unroll
  for (int i = 0; i < D; ++i) v[i] = px[(int64_t)i * A.ld + src];
#pragma unroll
  for (int i = 0; i < D; ++i) xcur[(int64_t)i * A.ld + off + k] = v[i];
  anc[off + k] = (int32_t)k;
}

// ---------------------------------------------------------------- launchers

hipError_t launch_theta_resample(const Smc2Args& S, int32_t col, double u, int32_t draw,
                                 int32_t* anc_tr_row, double* ess_out, hipStream_t s) {
  if (S.B < 1 || S.B > SMC2_MAXB) return hipErrorInvalidValue;
  // (B <= SMC2_NT: a lane each, and a wave for the evidence)
  const int nt = min(SMC2_NT, (S.B + 127) / 64 * 64);
  hipLaunchKernelGGL(k_theta_resample, 1, nt, 0, s, S, col, u, draw, anc_tr_row, ess_out);
  return hipGetLastError();
}

hipError_t launch_filter_gather(int prec, const void* xcur, void* xspare, const int32_t* anc,
                                const BatchArgs& A, const Smc2Args& S, const uint32_t* w,
                                hipStream_t s) {
  const unsigned g = (unsigned)A.n_chunks;
  if (g == 0) return hipSuccess;
  if (prec == 0)
    hipLaunchKernelGGL(k_filter_gather<double>, g, BATCH_NT, 0, s, (const double*)xcur,
                       (double*)xspare, anc, A, S, w);
  else
    hipLaunchKernelGGL(k_filter_gather<float>, g, BATCH_NT, 0, s, (const float*)xcur,
                       (float*)xspare, anc, A, S, w);
  return hipGetLastError();
}

hipError_t launch_smc2_propose(const Smc2Args& S, const double* z_row, double* prop_dev,
                               hipStream_t s) {
  const unsigned g = (unsigned)((S.B + 255) / 256);
  hipLaunchKernelGGL(k_smc2_propose, g, 256, 0, s, S, z_row, prop_dev);
  return hipGetLastError();
}

template <int MODEL, int D>
static void start_d(int prec, unsigned g, hipStream_t s, void* xcur, const void* xspare,
                    int32_t* anc, const double* z_row, const SmcProposal& P, uint32_t iter,
                    int copied, const BatchArgs& A, const Smc2Args& S) {
  if (prec == 0)
    hipLaunchKernelGGL((k_smc2_start<MODEL, D, double>), g, BATCH_NT, 0, s, (double*)xcur,
                       (const double*)xspare, anc, z_row, P, iter, copied, A, S);
  else
    hipLaunchKernelGGL((k_smc2_start<MODEL, D, float>), g, BATCH_NT, 0, s, (float*)xcur,
                       (const float*)xspare, anc, z_row, P, iter, copied, A, S);
}

template <int D>
static void finish_d(int prec, unsigned g, hipStream_t s, void* xcur, int32_t* anc,
                     const double* la, int32_t* acc_tr_row, double* theta_tr_row,
                     const SmcProposal& P, const BatchArgs& A, const Smc2Args& S) {
  if (prec == 0)
    hipLaunchKernelGGL((k_smc2_finish<D, double>), g, BATCH_NT, 0, s, (double*)xcur, anc, la,
                       acc_tr_row, theta_tr_row, P, A, S);
  else
    hipLaunchKernelGGL((k_smc2_finish<D, float>), g, BATCH_NT, 0, s, (float*)xcur, anc, la,
                       acc_tr_row, theta_tr_row, P, A, S);
}

hipError_t launch_smc2_start(int model, int d, int prec, void* xcur, const void* xspare,
                             int32_t* anc, const double* z_row, const SmcProposal& P,
                             uint32_t iter, int copied, const BatchArgs& A, const Smc2Args& S,
                             hipStream_t s) {
  const unsigned g = (unsigned)A.n_chunks;
  if (g == 0) return hipSuccess;
  switch (model == 1 ? 1 : d) {
#define X(M, DD) \
  case DD: start_d<M, DD>(prec, g, s, xcur, xspare, anc, z_row, P, iter, copied, A, S); break;
    X(1, 1) X(2, 4) X(2, 8) X(2, 16) X(2, 32) X(2, 40)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_smc2_finish(int d, int prec, void* xcur, int32_t* anc,
                              const double* log_alpha_row, int32_t* acc_tr_row,
                              double* theta_tr_row, const SmcProposal& P, const BatchArgs& A,
                              const Smc2Args& S, hipStream_t s) {
  const unsigned g = (unsigned)A.n_chunks;
  if (g == 0) return hipSuccess;
  switch (d) {
#define X(DD) \
  case DD:    \
    finish_d<DD>(prec, g, s, xcur, anc, log_alpha_row, acc_tr_row, theta_tr_row, P, A, S); break;
    X(1) X(4) X(8) X(16) X(32) X(40)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace pfk
