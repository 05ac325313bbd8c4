"""GPU parity for the model instantiations the headline workloads do not
reach: the windkessel model in the batched layout (per-filter parameters),
Lorenz '96 at d = 4, 16 and 32, and the largest batched filter (8192
particles) on its own.  FP64 results are compared with the oracle (log-weights
bit for bit, ancestors outside the 1e-9 band, likelihood increments within
1e-10 relative); FP32 batched results with the FP32 plain layout, which runs
the same propagation arithmetic."""
import dataclasses

import numpy as np
import pytest

import oracle
from oracle_resync import resync
import workloads as W

pytestmark = pytest.mark.gpu

REL64 = 1e-10
BAND = 1e-9


@pytest.fixture(scope="module")
def pfm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1306_3277_amd as pfm
    pfm.load()
    return pfm


def _mismatches_in_band(lw, u, a_gpu, a_ref):
    mism = np.flatnonzero(a_gpu != a_ref)
    if mism.size:
        w = np.exp(lw - lw.max())
        cw = np.cumsum(w) / w.sum()
        for k in mism:
            assert np.min(np.abs(cw - (u + k) / lw.size)) < BAND
    return mism.size


def _check_batched_fp64(pfm, pb):
    """Every filter of a batched FP64 handle against its own oracle run."""
    n = pb.n_particles
    off = np.concatenate([[0], np.cumsum(n)])
    refs = [oracle.pf_run(pb, theta=pb.theta[b], N=int(n[b]), b=b, traces=True)
            for b in range(pb.B)]
    f = pfm.Filter(pb, precision=pfm.PF_FP64, layout=pfm.PF_LAYOUT_BATCHED)
    flips = 0
    for t in range(1, pb.T + 1):
        f.step()
        lw = f.logweights()
        for b in range(pb.B):
            np.testing.assert_array_equal(lw[off[b]:off[b + 1]], refs[b]["lw"][t - 1],
                                          err_msg=f"filter {b}, t = {t}")
        f.resample()
        a = f.ancestors()
        for b in range(pb.B):
            u = oracle.resample_u(pb.seed, t, b)
            flips += _mismatches_in_band(refs[b]["lw"][t - 1], u, a[off[b]:off[b + 1]],
                                         refs[b]["anc"][t - 1])
    ell, ess = f.trace()
    ll, _, _ = f.loglik()
    x = f.get_state()
    for b in range(pb.B):
        r = refs[b]
        np.testing.assert_array_less(np.abs(ell[b] - r["ell"]),
                                     REL64 * np.maximum(1.0, np.abs(r["ell"])))
        np.testing.assert_allclose(ess[b], r["ess"], rtol=1e-9)
        assert abs(ll[b] - r["loglik"]) <= REL64 * max(1.0, abs(r["loglik"]))
        if flips == 0:
            np.testing.assert_array_equal(x[:, off[b]:off[b + 1]], r["x"])
    f.close()
    return flips


def test_windkessel_batched_fp64_per_filter_parameters(pfm):
    """Five windkessel filters with their own (R, C, Z, sigma_p, m0, s0) and
    particle counts, one of them a single particle."""
    base = W.windkessel(N=1, T=12)
    _, y = oracle.simulate(base)
    th = np.stack([W.wk_theta(1.0, 1.5, 0.03, 0.5, 90.0, 15.0, base.h),
                   W.wk_theta(0.8, 1.2, 0.05, 0.8, 85.0, 10.0, base.h),
                   W.wk_theta(1.3, 2.0, 0.02, 0.3, 95.0, 20.0, base.h),
                   W.wk_theta(1.0, 1.0, 0.03, 1.0, 90.0, 5.0, base.h),
                   W.wk_theta(0.6, 1.7, 0.04, 0.4, 80.0, 12.0, base.h)])
    pb = dataclasses.replace(base.with_obs(y), theta=th,
                             n_particles=np.array([300, 1, 1024, 2100, 64], dtype=np.int64))
    _check_batched_fp64(pfm, pb)


def test_windkessel_fp32_batched_equals_fp32_plain(pfm):
    base = W.windkessel(N=1, T=15, precision=W.FP32_MIXED)
    _, y = oracle.simulate(base)
    th = np.stack([W.wk_theta(1.0, 1.5, 0.03, 0.5, 90.0, 15.0, base.h),
                   W.wk_theta(0.9, 1.3, 0.04, 0.6, 88.0, 14.0, base.h),
                   W.wk_theta(1.1, 1.6, 0.02, 0.4, 92.0, 16.0, base.h)])
    pb = dataclasses.replace(base.with_obs(y), theta=th,
                             n_particles=np.array([513, 2048, 77], dtype=np.int64))
    outs = []
    for layout in (pfm.PF_LAYOUT_PLAIN, pfm.PF_LAYOUT_BATCHED):
        f = pfm.Filter(pb, precision=pfm.PF_FP32_MIXED, layout=layout)
        f.advance(pb.T)
        outs.append((f.trace()[0], f.get_state(), f.loglik()[0]))
        f.close()
    np.testing.assert_allclose(outs[1][0], outs[0][0], rtol=1e-12, atol=1e-12)
    np.testing.assert_array_equal(outs[1][1], outs[0][1])
    np.testing.assert_allclose(outs[1][2], outs[0][2], rtol=1e-12)


@pytest.mark.parametrize("d,obs_every,N", [(4, 1, 300), (16, 2, 513), (32, 4, 1100)])
def test_lorenz96_other_dimensions_fp64_plain(pfm, d, obs_every, N):
    pb = W.lorenz96(d=d, N=N, T=5, obs_every=obs_every)
    _, y = oracle.simulate(pb)
    pb = pb.with_obs(y)
    ref = oracle.pf_run(pb, traces=True)
    f = pfm.Filter(pb, precision=pfm.PF_FP64)
    for t in range(1, pb.T + 1):
        f.step()
        np.testing.assert_array_equal(f.logweights(), ref["lw"][t - 1], err_msg=f"t = {t}")
        f.resample()
        if _mismatches_in_band(ref["lw"][t - 1], oracle.resample_u(pb.seed, t), f.ancestors(),
                               ref["anc"][t - 1]):
            resync(f, pb, [0], t)  # an in-band flip: carry on from the oracle's particles
    ell, _ = f.trace()
    np.testing.assert_array_less(np.abs(ell[0] - ref["ell"]),
                                 REL64 * np.maximum(1.0, np.abs(ref["ell"])))
    np.testing.assert_array_equal(f.get_state(), ref["x"])
    f.close()


def test_lorenz96_d16_batched_fp64(pfm):
    base = W.lorenz96(d=16, N=1, T=4, obs_every=2)
    _, y = oracle.simulate(base)
    pb = dataclasses.replace(base.with_obs(y),
                             theta=np.array([[8.0, 0.1], [7.0, 0.2], [9.5, 0.05]]),
                             n_particles=np.array([700, 256, 1500], dtype=np.int64))
    _check_batched_fp64(pfm, pb)


def test_largest_batched_filter_alone_fp64(pfm):
    """One filter of the largest batched size: 8192 particles, one workgroup."""
    base = W.lorenz96(d=8, N=1, T=5)
    _, y = oracle.simulate(base)
    pb = dataclasses.replace(base.with_obs(y), theta=np.array([[8.0, 0.1]]),
                             n_particles=np.array([pfm.PF_BATCHED_MAX_PARTICLES],
                                                  dtype=np.int64))
    _check_batched_fp64(pfm, pb)


def test_batched_rejects_more_than_the_largest_filter(pfm):
    base = W.lorenz96(d=8, N=1, T=2)
    pb = dataclasses.replace(base.with_obs(np.zeros((2, 8))), theta=np.array([[8.0, 0.1]]),
                             n_particles=np.array([pfm.PF_BATCHED_MAX_PARTICLES + 1],
                                                  dtype=np.int64))
    with pytest.raises(pfm.PfError):
        pfm.Filter(pb, precision=pfm.PF_FP64, layout=pfm.PF_LAYOUT_BATCHED)


def test_simulate_on_another_stream_waits_for_its_buffer(pfm):
    """The output buffer is cleared on torch's current stream: work queued there
    must not clear it under (or after) the simulation on the caller's."""
    import torch
    pb = W.windkessel(N=1, T=20)
    _, y = pfm.simulate(pb)
    a = torch.ones(4096, 4096, device="cuda")
    for _ in range(20):
        a @ a
    _, z = pfm.simulate(pb, stream=torch.cuda.Stream())
    np.testing.assert_array_equal(y, z)
