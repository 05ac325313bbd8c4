// The FP64 normals' building blocks and the resamplers' logarithm decision
// (pf_device.hpp) against the plain IEEE expressions that they stand for, at
// every 32-bit word.  normals_check fills out[0..5] with the words at which ln,
// the radius, sin and cos differ, the words (paired with 40,503 w + 12,345) at
// which a stage-noise quotient differs, and the words whose FP32 logarithm
// leaves the decision's margin of 2e-5; out[6] is the largest distance
// |0.69314718 log2f(u) - ln u| as the bits of a double.
#include "pf_device.hpp"

namespace {
using namespace pfk;

__device__ double ref_u(uint32_t w) { return ((double)w + 0.5) * 0x1p-32; }

__device__ double ref_ln(double x) {
  const uint64_t bits = (uint64_t)__double_as_longlong(x);
  int e = (int)((bits >> 52) & 0x7ff) - 1022;
  double f = __longlong_as_double((long long)((bits & 0x000fffffffffffffULL) | 0x3fe0000000000000ULL));
  if (f < 0x1.6a09e667f3bcdp-1) {
    f = f + f;
    e = e - 1;
  }
  const double s = (f - 1.0) / (f + 1.0);
  const double s2 = s * s;
  double p = 1.0 / 21.0;
  for (int k = 19; k >= 1; k -= 2) p = p * s2 + 1.0 / (double)k;
  const double lnf = (2.0 * s) * p;
  const double de = (double)e;
  return de * 0x1.62e42feep-1 + (de * 0x1.a39ef35793c76p-33 + lnf);
}

__device__ void ref_sincos(double u, double& s_out, double& c_out) {
  const double v = 4.0 * u;
  const double kf = __builtin_floor(v + 0.5);
  const double f = v - kf;
  const int k = ((int)kf) & 3;
  const double p = f * 0x1.921fb54442d18p0, p2 = p * p;
  double sp = -1.0 / 121645100408832000.0;
  sp = sp * p2 + 1.0 / 355687428096000.0;
  sp = sp * p2 - 1.0 / 1307674368000.0;
  sp = sp * p2 + 1.0 / 6227020800.0;
  sp = sp * p2 - 1.0 / 39916800.0;
  sp = sp * p2 + 1.0 / 362880.0;
  sp = sp * p2 - 1.0 / 5040.0;
  sp = sp * p2 + 1.0 / 120.0;
  sp = sp * p2 - 1.0 / 6.0;
  sp = sp * p2 + 1.0;
  sp = sp * p;
  double cp = -1.0 / 6402373705728000.0;
  cp = cp * p2 + 1.0 / 20922789888000.0;
  cp = cp * p2 - 1.0 / 87178291200.0;
  cp = cp * p2 + 1.0 / 479001600.0;
  cp = cp * p2 - 1.0 / 3628800.0;
  cp = cp * p2 + 1.0 / 40320.0;
  cp = cp * p2 - 1.0 / 720.0;
  cp = cp * p2 + 1.0 / 24.0;
  cp = cp * p2 - 1.0 / 2.0;
  cp = cp * p2 + 1.0;
  const bool odd = (k & 1) != 0;
  const double s0 = odd ? cp : sp, c0 = odd ? -sp : cp;
  const bool neg = (k & 2) != 0;
  s_out = neg ? -s0 : s0;
  c_out = neg ? -c0 : c0;
}

__device__ bool differ(double a, double b) {
  return __double_as_longlong(a) != __double_as_longlong(b);
}

constexpr int PER = 1024;  // words per thread

__global__ __launch_bounds__(256) void k_check(unsigned long long* out, double h, double sq) {
  const uint32_t w0 = (blockIdx.x * 256u + threadIdx.x) * (uint32_t)PER;
  unsigned long long bad[6] = {};
  double far = 0.0;
  const double inv_h = 1.0 / h;
  for (int i = 0; i < PER; ++i) {
    const uint32_t w = w0 + (uint32_t)i, w2 = 40503u * w + 12345u;
    const double l = ln_f64(u01_f64(w)), rl = ref_ln(ref_u(w));
    bad[0] += differ(l, rl);
    bad[1] += differ(sqrt_mid(-2.0 * l), __builtin_sqrt(-2.0 * rl));
    double s, c, rs, rc;
    sincos2pi_f64(w, s, c);
    ref_sincos(ref_u(w), rs, rc);
    bad[2] += differ(s, rs);
    bad[3] += differ(c, rc);
    double z0, z1;
    bm_pair_f64(w, w2, z0, z1);
    bad[4] += differ(div_by(sq * z0, h, inv_h), (sq * z0) / h) ||
              differ(div_by(sq * z1, h, inv_h), (sq * z1) / h);
    const double d =
        __builtin_fabs((double)(0.69314718f * __builtin_amdgcn_logf(u01_f32(w))) - rl);
    bad[5] += !(d < 2e-5);
    far = fmax(far, d);
  }
  for (int k = 0; k < 6; ++k)
    if (bad[k]) atomicAdd(&out[k], bad[k]);
  atomicMax(&out[6], (unsigned long long)__double_as_longlong(far));
}
}  // namespace

extern "C" int normals_check(double h, double sq, unsigned long long* out) {
  unsigned long long* d = nullptr;
  hipError_t e = hipMalloc(&d, 7 * sizeof *d);
  if (e == hipSuccess) e = hipMemset(d, 0, 7 * sizeof *d);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_check, (unsigned)((1ull << 32) / (256ull * PER)), 256, 0, nullptr, d, h, sq);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpy(out, d, 7 * sizeof *d, hipMemcpyDeviceToHost);
  if (d) (void)hipFree(d);
  return (int)e;
}
