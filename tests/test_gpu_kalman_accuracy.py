"""The windkessel Kalman filter's rounding over long series: against 80-bit
arithmetic, the likelihoods of parameter sets around the example's are no
further off, in the mean, than those of Alg. 1 stepped substep by substep in
64 bits (which the bound is, computed here on the same inputs)."""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

B = 200


def _chain(pb, real):
    """Alg. 1, every filter, in the arithmetic of `real`."""
    a, c, Z, sp, m, s0 = (pb.theta[:, i].astype(real) for i in range(6))
    V = s0 * s0
    R = real(pb.obs_sd) * real(pb.obs_sd)
    two_pi = 2 * real(np.arctan2(real(0), real(-1)))
    q, y = pb.q.astype(real), pb.obs[:, 0].astype(real)
    ll = np.zeros(B, dtype=real)
    for t in range(pb.T):
        for s in range(pb.K):
            m = a * m + c * q[t * pb.K + s]
            V = a * a * V + sp * sp
        v = y[t] - (m + Z * q[(t + 1) * pb.K])
        S = V + R
        ll = ll - (np.log(two_pi * S) + v * v / S) / 2
        gain = V / S
        m = m + gain * v
        V = (1 - gain) * V
    return ll


@pytest.mark.parametrize("T,K,obs_sd", [(5, 1, 1.0), (100, 1, 1.0), (100, 10, 2.0), (300, 20, 2.0),
                                        (400, 10, 1.0), (1000, 5, 2.0), (1000, 10, 2.0),
                                        (2000, 1, 0.2)])
def test_likelihoods_no_further_off_than_the_chain(T, K, obs_sd):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1306_3277_amd as pfm
    rng = np.random.default_rng([T, K])
    base = W.windkessel(N=1, T=T, K=K, B=B)
    scale = rng.uniform(0.8, 1.2, size=(B, 4))
    theta = np.stack([W.wk_theta(r, cc, z, r * (1 - np.exp(-base.h / (r * cc))) * np.sqrt(s2),
                                 90.0, 15.0, base.h)
                      for r, cc, z, s2 in np.array([1.0, 1.5, 0.03, 25.0]) * scale])
    pb = dataclasses.replace(base, obs_sd=1.0, theta=base.theta[:1], n_particles=np.ones(1, dtype=np.int64))
    y = pfm.simulate(pb)[1]
    pb = dataclasses.replace(base, obs_sd=obs_sd, theta=theta).with_obs(y)
    f = pfm.Filter(pb)
    ll, ell = f.kalman()
    f.close()
    exact = _chain(pb, np.longdouble)
    off = np.mean(np.abs((ll - exact) / exact))
    bound = np.mean(np.abs((_chain(pb, np.float64) - exact) / exact))
    assert off <= bound + 2.0 ** -54, (off, bound)  # (half of the likelihood's own rounding)
