"""Small sets of weights, resampled by one workgroup (up to 4,096 of them):
sizes around the rows, blocks and spans of its three widths, against the
oracle's collective under the same criteria as the large sets."""
import numpy as np
import pytest

from test_gpu_systematic import check, env, run, weights  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 769, 1023, 1024, 1025, 2047, 2048,
                               2049, 3073, 4095, 4096, 4097])
def test_systematic_small_sizes(env, n):  # noqa: F811
    rng = np.random.default_rng(n)
    for kind in ("spread", "wide", "concentrated", "holes", "last_only"):
        if kind in ("concentrated", "holes") and n < 4:
            continue
        lw = weights(kind, n, rng)
        for u in (0.0, float(rng.random()), 1.0 - 2.0 ** -40):
            a, stats = run(env, lw, u)
            check(lw, u, a, stats)


SCHEMES = {"systematic": (0, 0, float("inf")), "stratified": (1, 0, float("inf")),
           "multinomial": (3, 0, float("inf")), "metropolis": (2, 5, float("inf")),
           "ess": (0, 0, 0.5)}


def _outputs(f):
    ll, ess, t = f.loglik(allow_numeric=True)
    return [f.logweights(), f.ancestors(), f.get_state(), ll, ess, np.array([t]), *f.trace()]


@pytest.mark.parametrize("n,K", [(1, 1), (64, 3), (65, 2), (256, 12), (257, 13), (1000, 10), (1024, 1),
                                 (1025, 5), (2048, 14), (2049, 2), (4095, 3), (4096, 17)])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_small_run_equals_eager_steps(env, n, K, precision):  # noqa: F811
    """A windkessel filter's run in one launch has the bits of the eager
    steps' kernels, whatever comes before and after it."""
    _, pfm = env
    import workloads as W
    T = 9
    pb = W.windkessel(N=n, T=T, K=K, seed=n + K)
    pb = pb.with_obs(90.0 + 5.0 * np.random.default_rng(n).standard_normal((T, 1)))
    for name, (scheme, steps, frac) in SCHEMES.items():
        f, g = (pfm.Filter(pb, precision=precision) for _ in range(2))
        for h in (f, g):
            h.set_resampler(scheme, steps, frac)
        f.advance(T)
        g.graph_run(4)
        g.advance(2)
        g.graph_run(3)
        for a, b in zip(_outputs(f), _outputs(g)):
            np.testing.assert_array_equal(a, b, err_msg=name)
        f.close()
        g.close()


@pytest.mark.parametrize("sizes,K", [((2049, 1), 2), ((4095, 4096), 17), ((4096, 3000, 40), 5)])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_small_run_of_several_large_filters(env, sizes, K, precision):  # noqa: F811
    """Past 2,048 particles only several filters take one launch."""
    _, pfm = env
    import dataclasses

    import workloads as W
    T = 6
    base = W.windkessel(N=1, T=T, K=K, B=len(sizes), seed=K)
    pb = dataclasses.replace(
        base.with_obs(90.0 + 5.0 * np.random.default_rng(K).standard_normal((T, 1))),
        n_particles=np.array(sizes, dtype=np.int64))
    for name, (scheme, steps, frac) in SCHEMES.items():
        f, g = (pfm.Filter(pb, precision=precision) for _ in range(2))
        for h in (f, g):
            h.set_resampler(scheme, steps, frac)
        f.advance(T)
        g.graph_run(T)
        for a, b in zip(_outputs(f), _outputs(g)):
            np.testing.assert_array_equal(a, b, err_msg=name)
        f.close()
        g.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
def test_small_run_of_uneven_filters_and_lost_weights(env, precision):  # noqa: F811
    _, pfm = env
    import dataclasses

    import workloads as W
    T = 70  # more than the 64 intervals whose likelihoods are formed at once
    base = W.windkessel(N=1, T=T, K=2, B=4)
    obs = 90.0 + 4.0 * np.random.default_rng(2).standard_normal((T, 1))
    obs[66] = 1e200  # no particle explains it: every weight 0
    pb = dataclasses.replace(base.with_obs(obs),
                             n_particles=np.array([5, 1500, 256, 3000], dtype=np.int64))
    f, g = (pfm.Filter(pb, precision=precision) for _ in range(2))
    f.advance(T)
    g.graph_run(T)
    for a, b in zip(_outputs(f), _outputs(g)):
        np.testing.assert_array_equal(a, b)
    assert np.all(np.isneginf(g.loglik(allow_numeric=True)[0]))
    f.close()
    g.close()


def test_small_run_refused_on_a_capturing_stream(env):  # noqa: F811
    """pf_graph_run inside a caller's capture is refused with nothing recorded;
    the resampling that was pending is not lost."""
    torch, pfm = env
    import workloads as W
    T = 6
    pb = W.windkessel(N=700, T=T, K=3)
    pb = pb.with_obs(90.0 + 5.0 * np.random.default_rng(1).standard_normal((T, 1)))
    s = torch.cuda.Stream()
    f, g = (pfm.Filter(pb, stream=s) for _ in range(2))
    for h in (f, g):
        h.advance(2)
    x = torch.zeros(4, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        graph.capture_begin(capture_error_mode="thread_local")
        with pytest.raises(pfm.PfError):
            g.graph_run(2)
        x.add_(1.0)
        graph.capture_end()
        graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(x.cpu(), torch.ones(4))
    f.advance(T - 2)
    g.graph_run(T - 2)
    for a, b in zip(_outputs(f), _outputs(g)):
        np.testing.assert_array_equal(a, b)
    f.close()
    g.close()


@pytest.mark.parametrize("sizes,scheme,steps,frac", [
    ((64,), 4, 0, float("inf")), ((64,), 4, 0, 0.5), ((700,), 4, 0, float("inf")),
    ((300, 200, 257), 4, 0, float("inf")), ((300, 200, 257), 4, 0, 0.5),
    ((4096, 1, 3000, 2049, 65), 4, 0, float("inf")), ((193, 65), 4, 0, 0.5),
    ((1024,), 2, 21, float("inf")), ((1024,), 2, 22, float("inf")), ((193,), 2, 40, 0.5),
    ((64,), 2, 508, float("inf")), ((2048, 1500), 2, 33, float("inf")),
    ((4096, 4096), 2, 0, float("inf"))])
@pytest.mark.parametrize("precision", [0, 1])
def test_rejection_and_many_moves_equal_eager_steps(env, sizes, scheme, steps, frac,  # noqa: F811
                                                    precision):
    """Rejection and long Metropolis runs go one workgroup per filter or the
    multi-kernel path's graphs by sizes, filters and moves: the eager steps'
    bits either way, over more intervals than a launch of rejection takes and
    with eager steps between."""
    _, pfm = env
    import dataclasses

    import workloads as W
    T = 24
    base = dataclasses.replace(W.windkessel(N=1, T=T, K=3, B=len(sizes), seed=steps), obs_sd=8.0)
    pb = dataclasses.replace(
        base.with_obs(90.0 + 5.0 * np.random.default_rng(steps).standard_normal((T, 1))),
        n_particles=np.array(sizes, dtype=np.int64))
    f, g = (pfm.Filter(pb, precision=precision) for _ in range(2))
    for h in (f, g):
        h.set_resampler(scheme, steps, frac)
    f.advance(T)
    g.graph_run(18)
    g.advance(2)
    g.graph_run(4)
    for a, b in zip(_outputs(f), _outputs(g)):
        np.testing.assert_array_equal(a, b)
    f.close()
    g.close()


@pytest.mark.parametrize("sizes", [(1,), (3,), (63,), (64, 1, 33), (65, 64, 2), (17,) * 40])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_small_run_of_single_row_filters(env, sizes, precision):  # noqa: F811
    """Filters of up to 64 particles keep numbers for those alone."""
    _, pfm = env
    import dataclasses

    import workloads as W
    T = 7
    base = W.windkessel(N=1, T=T, K=14, B=len(sizes))
    pb = dataclasses.replace(
        base.with_obs(90.0 + 5.0 * np.random.default_rng(3).standard_normal((T, 1))),
        n_particles=np.array(sizes, dtype=np.int64))
    for name, (scheme, steps, frac) in SCHEMES.items():
        f, g = (pfm.Filter(pb, precision=precision) for _ in range(2))
        for h in (f, g):
            h.set_resampler(scheme, steps, frac)
        f.advance(T)
        g.graph_run(5)
        g.graph_run(2)
        for a, b in zip(_outputs(f), _outputs(g)):
            np.testing.assert_array_equal(a, b, err_msg=name)
        f.close()
        g.close()
