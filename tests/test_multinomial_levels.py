"""The multinomial search's index arithmetic at every size that a filter may
have: on the CPU against 64-bit integers, with undefined behaviour trapped,
and on the GPU at the largest one."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1306_3277_amd", "csrc")
CXX = "/opt/rocm/llvm/bin/clang++"

SOURCE = r"""
#include <hip/hip_runtime_api.h>
#include "pf_internal.hpp"
#include <cstdio>
#include <cstdlib>
using namespace pfk;
static void check(int64_t N) {
  const MultiLevels m = multi_levels((int32_t)N);
  const int64_t n16 = (N + 15) / 16, n256 = (N + 255) / 256;
  const int64_t nt = N <= MULTI_NB ? N : n16 <= MULTI_NB ? n16 : n256;
  const int64_t per = (nt + MULTI_NB - 1) / MULTI_NB, ns = (nt + per - 1) / per;
  bool ok = m.n16 == n16 && m.nt == nt && m.per == per && m.ns == ns && ns <= MULTI_NB;
  // the samples' places, and the last particle of every lane near the end
  for (int64_t i = 0; i < MULTI_NB; ++i) {
    const int64_t at = ((i + 1) * per < nt ? (i + 1) * per : nt) - 1;
    ok = ok && at >= 0 && at < nt && (int64_t)(i + 1) * m.per <= INT32_MAX;
  }
  for (int64_t j0 = (N - 1) / K3_PER * K3_PER, k = 0; j0 >= 0 && k < 300; j0 -= K3_PER, ++k)
    ok = ok && lane_last((int32_t)j0, (int32_t)N) == (j0 + K3_PER < N ? j0 + K3_PER : N) - 1;
  if (!ok) {
    printf("N = %lld: n16 %d nt %d per %d ns %d\n", (long long)N, m.n16, m.nt, m.per, m.ns);
    exit(1);
  }
}
int main() {
  for (int64_t N = 1; N < 40000; ++N) check(N);
  for (int e = 15; e < 31; ++e)
    for (int64_t d = -600; d <= 600; ++d) check((1LL << e) + d);
  for (int64_t N = (1LL << 31) - 5000; N < (1LL << 31); ++N) check(N);
  printf("ok\n");
  return 0;
}
"""


def test_levels_match_64_bit_arithmetic(tmp_path):
    if not os.path.exists(CXX):
        pytest.skip("ROCm clang++ not found")
    (tmp_path / "levels.cpp").write_text(SOURCE)
    exe = str(tmp_path / "levels")
    r = subprocess.run([CXX, "-std=c++17", "-O1", "-ftrapv", "-D__HIP_PLATFORM_AMD__", "-w",
                        "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        "-o", exe, str(tmp_path / "levels.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.gpu
def test_largest_multinomial_filter():
    """2^31 - 1 particles of nearly equal weights (an observation sd of 1e12):
    output k's ancestor is floor(u_k N) up to the rounding of the cumulative
    weights, 2^31 of them to a few 2^-53 of their sum, so to one particle."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import dataclasses

    import oracle
    import paper_1306_3277_amd as pfm
    import workloads as W
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 110 << 30:
        pytest.skip("needs 110 GiB of free device memory")
    N = 2 ** 31 - 1
    pb = dataclasses.replace(W.windkessel(N=N, T=1, K=1, precision=1), obs_sd=1e12)
    f = pfm.Filter(pb.with_obs(np.full((1, 1), 90.0)))
    f.set_resampler(pfm.PF_RESAMPLE_MULTINOMIAL)
    f.advance(1)
    a = f.ancestors()
    f.close()
    del f
    torch.cuda.empty_cache()
    assert a.shape == (N,) and a.min() >= 0 and a.max() < N
    k = np.unique(np.concatenate([np.arange(64), N - 1 - np.arange(3000),
                                  np.random.default_rng(1).integers(0, N, 3000)]))
    u = np.array([oracle.multi_u(pb.seed, 1, 0, 0, int(i)) for i in k])
    assert np.max(np.abs(a[k].astype(np.int64) - np.floor(u * N).astype(np.int64))) <= 1
