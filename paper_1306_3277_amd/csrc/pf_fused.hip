// Fused intervals of the batched layout, for filters of up to a few thousand
// particles: one launch per interval instead of two.  A launch boundary costs
// about 2 us here, the collective is a chain of a few us that leaves the chip
// idle, and both stood in every interval (64 filters of 2,048 particles: 11 us
// of propagation in an interval of 29).
//
// The collective cannot hand its ancestors to other workgroups inside a
// launch (a device-scope hand-off costs more than the boundary), so every
// workgroup that propagates NT of a filter's particles first runs the whole
// filter's collective for itself, from the log-weights the previous launch
// left: the same code as the batched collective, so the same bits in each.  It
// needs the ancestors of its own outputs only, by binary search of the
// stratum counts in LDS; they reach memory only if a history records them.
// The log-weights alternate between two buffers, since workgroups of one
// launch still read the old ones when others have written theirs, and the
// filters' interval counters advance at the end of the run (the last
// collective is the batched layout's own).
#include <math.h>

#include "pf_batch_parts.hpp"

namespace pfk {

template <int MODEL, int D, typename Real, bool ACC, int NT>
__global__ __launch_bounds__(NT) void k_batch_fused(Real* __restrict__ xa, Real* __restrict__ xb,
                                                    const double* __restrict__ lw_in,
                                                    double* __restrict__ lw, BatchArgs A) {
  constexpr int MAXP = FUSED_PER;
  __shared__ double stage[NT * MAXP];
  __shared__ ScanLds<NT> X;
  const FilterSlot slot = A.fused[blockIdx.x];
  const int f = slot.f, N = slot.n, k0 = slot.pad;
  if (N == 0) return;  // the table's padding
  const int64_t off = slot.off;
  FilterState* fs = A.fs + f;
  const int t = fs->t + 1 + A.step;  // the interval propagated; the collective is t - 1's
  const uint32_t iter = fs->iter;
  const bool keeper = k0 == 0;  // this workgroup does the filter's bookkeeping
  double lprev = 0.0;
  BatchScan<MAXP> sc;
  batch_scan<NT, MAXP>(
      lw_in + off, N, stage, X,
      [&]() -> double {
        if (keeper) lprev = fs->carry ? fs->lprev : log((double)N);
        return u01_f64(draw(bkey(A.key), TAG_RESAMPLE, 0, iter, 0, (uint32_t)(t - 1),
                            (uint32_t)f).x);
      },
      sc);
  const double M = sc.M, S = sc.S;
  const bool ok = sc.finite && S > 0.0;
  const double ess = ok ? (S * S) / sc.S2 : 0.0;
  const bool carry = ok && A.rs.ess_frac < INFINITY && !(ess < A.rs.ess_frac * (double)N);
  const int k = k0 + (int)threadIdx.x;
  int a = k;
  if (sc.finite && !carry) {
    int32_t cnt[MAXP], before, total;
    lane_counts<MAXP>(sc.P, sc.i0, sc.i1, sc.vprev, S, 1.0 / S, sc.u, N,
                      [&](int e) { return sc.cum(e); }, cnt, before, total);
    int32_t* counts = reinterpret_cast<int32_t*>(stage);
#pragma unroll
    for (int e = 0; e < MAXP; ++e)
      if (e < sc.P && sc.i0 + e < sc.i1) counts[anc_slot(sc.i0 + e)] = cnt[e];
    __syncthreads();
    // output k's ancestor: the first particle whose count exceeds k
    int lo = 0;
    for (int len = N; len > 0;) {
      const int half = len >> 1;
      const bool up = counts[anc_slot(min(lo + half, N - 1))] <= k;
      lo = up ? lo + half + 1 : lo;
      len = up ? len - half - 1 : half;
    }
    a = k < total ? lo : sc.jstar;
    if (k < N && (a < 0 || a >= N)) {  // never expected; flagged, and kept in bounds
      a = 0;
      atomicOr(&fs->pad, 1);
    }
  }
  if (k < N) {
    // the state written by interval s lies in buffer s % 2
    const Real* xp = ((t - 1) & 1) ? xb : xa;
    Real* xn = (t & 1) ? xb : xa;
    Real* xh = A.hx ? (Real*)A.hx + (int64_t)t * (MODEL == 1 ? 1 : D) * A.ld : nullptr;
    if (A.ha) A.ha[(int64_t)(t - 2) * A.ld + off + k] = a;
    double l = propagate_one<MODEL, D, Real, ACC, true>(xp, xn, xh, off + a, off + k, k, f, t,
                                                        iter, A);
    if (carry) l = lw_in[off + k] + l;
    lw[off + k] = l;
  }
  if (keeper && threadIdx.x == 0) {
    double ell;
    if (ok) {
      const double L = M + log(S);
      ell = L - lprev;
      fs->lprev = L;
    } else {
      ell = -INFINITY;
      fs->status = 4;
    }
    fs->carry = carry;
    fs->loglik = fs->loglik + ell;
    fs->M = sc.finite ? M : -INFINITY;
    fs->S = S;
    fs->ell = ell;
    fs->ess = ess;
    A.ell_tr[(size_t)f * A.T + t - 2] = ell;
    A.ess_tr[(size_t)f * A.T + t - 2] = ess;
    fs->u = sc.u;
  }
}

// ---------------------------------------------------------------- launchers

template <int MODEL, int D, typename Real, bool ACC = false>
static void launch_fused(int nt, unsigned g, hipStream_t s, void* xa, void* xb,
                         const double* lw_in, double* lw, const BatchArgs& a) {
  if (nt == 256)
    hipLaunchKernelGGL((k_batch_fused<MODEL, D, Real, ACC, 256>), g, 256, 0, s, (Real*)xa,
                       (Real*)xb, lw_in, lw, a);
  else if constexpr (sizeof(Real) == 4)  // (an FP64 propagation is never better off so)
    hipLaunchKernelGGL((k_batch_fused<MODEL, D, Real, ACC, 512>), g, 512, 0, s, (Real*)xa,
                       (Real*)xb, lw_in, lw, a);
}

hipError_t launch_batched_fused(int model, int d, int prec, int nt, void* xa, void* xb,
                                const double* lw_in, double* lw, const BatchArgs& a,
                                int nentries, hipStream_t s) {
  if (nentries <= 0) return hipSuccess;
  if (lw_in == lw || a.step < 1 || (nt != 256 && (nt != 512 || prec == 0)))
    return hipErrorInvalidValue;
  const unsigned g = (unsigned)nentries;
#define PF_FUSED(M, DD)                                                              \
  do {                                                                               \
    if (prec == 0) launch_fused<M, DD, double>(nt, g, s, xa, xb, lw_in, lw, a);      \
    else if (prec == 1) launch_fused<M, DD, float>(nt, g, s, xa, xb, lw_in, lw, a);  \
    else launch_fused<M, DD, float, true>(nt, g, s, xa, xb, lw_in, lw, a);           \
  } while (0)
  switch (model == 1 ? 1 : d * 4 + model) {
    case 1: PF_FUSED(1, 1); break;
    case 4 * 4 + 2: PF_FUSED(2, 4); break;
    case 8 * 4 + 2: PF_FUSED(2, 8); break;
    case 16 * 4 + 2: PF_FUSED(2, 16); break;
    case 4 * 4 + 3: PF_FUSED(3, 4); break;
    case 8 * 4 + 3: PF_FUSED(3, 8); break;
    case 16 * 4 + 3: PF_FUSED(3, 16); break;
    default: return hipErrorInvalidValue;
  }
#undef PF_FUSED
  return hipGetLastError();
}

}  // namespace pfk
