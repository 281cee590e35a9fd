"""The two groupings of the clustering (runs in LDS, and the radix sort for large clusters) at
the sizes where the choice and the scans turn: bit-exact against the oracle on either side of
the mean cluster size, at the single-workgroup scan's largest size and one above, with one
cluster larger than a run (the whole call is taken again by the radix sort), and a run filled
to its last place."""

import numpy as np
import pytest

import oracle as O
from test_gpu_cluster import compare, compare_minibatch, landau_markers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k,iters", [(96 * 40, 40, 3), (96 * 40 + 1, 40, 3),   # mean 96, above
                                       (16384, 16384, 1), (17000, 16385, 2),     # scans
                                       (257, 256, 2), (300, 257, 2), (65, 1, 2)])
def test_runs_and_radix_match_oracle(vp, m, k, iters):
    q, p, w, L = landau_markers(m, seed=3 * m + k)
    init = np.random.default_rng(m).choice(m, k, replace=False)
    compare(vp, q, p, w, k, L, iters, init)


@pytest.mark.parametrize("bunch", [1023, 1024, 1025, 4000])
def test_one_large_cluster(vp, bunch):
    """`bunch` markers at one place, with one starting centre there: their cluster fills a run
    exactly, or does not fit one.  The other clusters are small (mean below 96)."""
    m, k = 12000, 400
    q, p, w, L = landau_markers(m, seed=bunch)
    at = np.random.default_rng(bunch).choice(m, bunch, replace=False)
    q[at], p[at] = 3.0, 7.5          # far from the others: exactly these markers
    others = np.setdiff1d(np.arange(m), at)
    init = np.concatenate([at[:1], np.random.default_rng(2).choice(others, k - 1, replace=False)])
    got, ref = compare(vp, q, p, w, k, L, 2, init)
    assert np.bincount(got["assign"].cpu().numpy(), minlength=k)[0] == bunch
    batches = np.stack([np.concatenate([at[:1025], others[:1000]]), others[1000:1000 + 1025 + 1000]]) \
        if bunch >= 1025 else others[:2000].reshape(2, 1000)
    compare_minibatch(vp, q, p, w, k, L, init, batches)


def test_empty_clusters_and_repeated_centres(vp):
    """Repeated starting markers (the higher-numbered centre stays empty) among small runs."""
    q, p, w, L = landau_markers(3000, seed=8)
    init = np.concatenate([np.arange(150), np.arange(150)])
    got, ref = compare(vp, q, p, w, 300, L, 0, init)
    assert got["Q"].shape[0] == 150
