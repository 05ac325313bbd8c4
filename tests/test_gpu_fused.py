"""Fused intervals of the batched layout (a run's collectives each in one
launch with the next propagation) against the eager steps' two kernels: the
same code in another order of launches, so the same bits, whatever the run's
length (odd, even: the log-weights alternate between two buffers), the filters'
sizes around whole workgroups, the form, the trigger and a history."""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pfm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1306_3277_amd as pfm
    pfm.load()
    return pfm


def _problem(pfm, model, d, n, T):
    B = len(n)
    if model == 1:
        base = W.windkessel(N=1, T=T, K=4, B=B)
    else:
        base = W.lorenz96(d=d, N=1, T=T, K=2, B=B, stage_noise=model == 3)
        th, _ = W.batched_thetas(B, 3)
        base = dataclasses.replace(base, theta=th)
    base = dataclasses.replace(base, n_particles=np.asarray(n, dtype=np.int64))
    return base.with_obs(pfm.simulate(base)[1])


def _outputs(f):
    ll, ess, t = f.loglik(allow_numeric=True)
    return [f.logweights(), f.ancestors(), f.get_state(), ll, ess, np.array([t]), *f.trace()]


CASES = [  # model, d, threads, groups, particle counts
    (2, 8, 256, 1, [2048, 1, 255, 256, 257, 511, 513, 2047]),
    (2, 4, 256, 2, [700, 64, 65, 1024, 1025]),
    (3, 16, 256, 1, [300, 1800]),
    (3, 8, 512, 2, [4096, 2049, 4095, 512, 513]),
    (2, 16, 512, 2, [2100, 3000]),
    (1, 1, 256, 1, [1000, 2048, 3]),
    (1, 1, 512, 2, [3333, 2500]),
]


@pytest.mark.parametrize("model,d,threads,groups,n", CASES)
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_fused_runs_equal_eager_steps(pfm, model, d, threads, groups, n, precision):
    T = 12
    pb = _problem(pfm, model, d, n, T)
    for frac in (float("inf"), 0.6):
        f, g = (pfm.Filter(pb, precision=precision, layout=1) for _ in range(2))
        for h in (f, g):
            h.set_tuning(threads, groups)
            if frac < 1.0:
                h.set_resampler(0, 0, frac)
        hist = precision == 2 and frac > 1.0
        if hist:
            f.attach_history()
            g.attach_history()
        f.advance(T)
        g.graph_run(7)  # 4 + 2 + 1 intervals
        g.advance(1)
        g.set_replay(True)
        g.graph_run(4)  # eager launches
        for a, b in zip(_outputs(f), _outputs(g)):
            np.testing.assert_array_equal(a, b)
        if hist:
            for a, b in zip(f.backtrace(), g.backtrace()):
                np.testing.assert_array_equal(a, b)
        f.close()
        g.close()


def test_fused_run_with_lost_weights(pfm):
    pb = _problem(pfm, 2, 8, [300, 1000], 8)
    obs = pb.obs.copy()
    obs[3] = 1e200  # no particle explains it: every weight 0, every filter flagged
    pb = pb.with_obs(obs)
    f, g = (pfm.Filter(pb, precision=0, layout=1) for _ in range(2))
    f.advance(8)
    g.graph_run(8)
    for a, b in zip(_outputs(f), _outputs(g)):
        np.testing.assert_array_equal(a, b)
    assert np.all(np.isneginf(g.loglik(allow_numeric=True)[0]))
    f.close()
    g.close()


@pytest.mark.parametrize("threads,groups,n,precision", [
    (512, 2, [2049] * 52, 1), (512, 2, [2049] * 52, 2),      # 20 rows of workgroups
    (512, 2, [4096] * 16, 1), (512, 2, [4096] * 16, 2),      # 8: the fast form alone
    (512, 2, [4096] * 64, 2), (512, 2, [4096] * 66, 2),      # 32 and 40
    (512, 2, [4096] * 34, 0), (512, 4, [4096] * 80, 1),      # neither
    (256, 1, [7] * 768, 1), (256, 1, [7] * 769, 1),          # workgroups nearly empty
    (256, 1, [128] * 1280, 0), (256, 1, [129] * 1281, 0), (256, 2, [2048] * 73, 2)])
def test_both_sides_of_the_rule(pfm, threads, groups, n, precision):
    T = 6
    pb = _problem(pfm, 2, 4, n, T)
    f, g = (pfm.Filter(pb, precision=precision, layout=1) for _ in range(2))
    for h in (f, g):
        h.set_tuning(threads, groups)
    f.advance(T)
    g.graph_run(5)
    g.graph_run(1)
    for a, b in zip(_outputs(f), _outputs(g)):
        np.testing.assert_array_equal(a, b)
    f.close()
    g.close()
