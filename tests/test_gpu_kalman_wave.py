"""The windkessel Kalman filter's two forms (intervals spread over a wave's
lanes; one lane per filter) against the oracle, at the edges of the wave
form's passes (two intervals per lane, 128 per pass), with and without the
series in LDS, and with degenerate variances.  Both evaluate Alg. 1 in FP64:
increments within 1e-12 relative (a few ulps of the pressures over the
smallest increment), accept decisions equal."""
import dataclasses

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

REL = 1e-12


@pytest.fixture(scope="module")
def pfm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1306_3277_amd as pfm
    pfm.load()
    return pfm


def _problem(B, T, K, seed=3):
    base = W.windkessel(N=1, T=T, K=K, B=B)
    _, y = oracle.simulate(base)
    rng = np.random.default_rng(seed)
    th = np.stack([W.wk_theta(R, C, Z, sp, m0, s0, base.h) for R, C, Z, sp, m0, s0 in
                   zip(rng.uniform(0.6, 1.4, B), rng.uniform(1.0, 2.0, B),
                       rng.uniform(0.0, 0.05, B), rng.uniform(0.2, 2.0, B),
                       rng.uniform(80, 100, B), rng.uniform(1.0, 20.0, B))])
    return dataclasses.replace(base.with_obs(y), theta=th)


def _check(pb, ll, ell, sel):
    for b in sel:
        rl, rell = oracle.kf_wk(pb, pb.theta[b])
        assert abs(ll[b] - rl) <= REL * abs(rl)
        np.testing.assert_allclose(ell[b], rell, rtol=REL, atol=1e-300)


@pytest.mark.parametrize("T,K", [(1, 1), (2, 3), (63, 2), (64, 5), (127, 1), (128, 7), (129, 2),
                                 (255, 3), (256, 1), (257, 10)])
def test_pass_edges(pfm, T, K):
    pb = _problem(6, T, K)
    pb.theta[1, 3] = 0.0  # no pressure noise
    pb.theta[2, 5] = 0.0  # known initial pressure
    pb.theta[3, 3] = pb.theta[3, 5] = 0.0
    pb.theta[4, 0] = 1.02  # a growing pressure, held by the observations
    f = pfm.Filter(pb)
    ll, ell = f.kalman()
    f.close()
    _check(pb, ll, ell, range(6))


def test_many_short_filters_take_a_lane_each(pfm):
    pb = _problem(4000, 2, 2)
    f = pfm.Filter(pb)
    ll, ell = f.kalman()
    f.close()
    _check(pb, ll, ell, [0, 1, 63, 64, 255, 256, 3999])


@pytest.mark.parametrize("B,T,K,iters", [(3, 1, 1, 30), (2, 130, 2, 40), (2, 3000, 3, 8),
                                         (3000, 2, 1, 12)])
def test_chains_match_oracle(pfm, B, T, K, iters):
    """One pass and several, a series too long for LDS, and the lane form."""
    pb = W.windkessel_paper(N=1, T=T, K=K, B=B)
    _, y = oracle.simulate(pb)
    pb = pb.with_obs(y)
    spec = W.WkMh()
    rng = np.random.default_rng(B + T)
    th0 = np.array([1.0, 1.5, 0.03, 25.0]) * rng.uniform(0.9, 1.1, size=(B, 4))
    inp = W.wk_mh_inputs(spec, chains=B, iters=iters, seed=40, theta0=th0)
    f = pfm.Filter(pb)
    out = {k: v.cpu().numpy() for k, v in
           f.kalman_pmmh(spec, inp.theta0, inp.prop, inp.alpha).items()}
    f.close()
    sel = np.unique([0, 1, B // 2, B - 1])
    ref = oracle.kf_pmmh(dataclasses.replace(pb, theta=pb.theta[sel]), spec,
                         W.WkMhInputs(th0[sel], inp.prop[:, sel], inp.alpha[:, sel]))
    np.testing.assert_array_equal(out["accepts"][sel], ref["accepts"])
    atol = np.array(list(spec.step_sd) + [0.0]) * 1e-12
    assert np.all(np.abs(out["theta"][:, sel] - ref["theta"]) <= REL * np.abs(ref["theta"]) + atol)
    np.testing.assert_allclose(out["ll"][:, sel], ref["ll"], rtol=1e-11, atol=1e-12)
