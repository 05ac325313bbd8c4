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
