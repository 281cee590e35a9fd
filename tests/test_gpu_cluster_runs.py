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


@pytest.mark.parametrize("bunch", [511, 512, 513, 1023, 1025, 4000])
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


@pytest.mark.parametrize("m,k", [(20000, 8192), (20000, 8193), (60000, 7000)])
def test_scans_fused_with_their_fills(vp, m, k):
    """At the largest number of counters whose scan runs inside the fills, and one above; the
    mini-batch form at the same sizes (a batch counts, and clears, the same counters)."""
    q, p, w, L = landau_markers(m, seed=m + k)
    rng = np.random.default_rng(k)
    init = rng.choice(m, k, replace=False)
    compare(vp, q, p, w, k, L, 2, init)
    compare_minibatch(vp, q, p, w, k, L, init, rng.integers(0, m, (3, k + 100)))


def test_markers_far_from_every_centre(vp):
    """Markers in empty corners of the grid (the search starts from the neighbours in cell
    order), some at the very edge, all centres in one thin row."""
    rng = np.random.default_rng(7)
    L = 10.0
    q = np.concatenate([rng.uniform(0, L, 900), [0.0, np.nextafter(L, 0), 0.0, np.nextafter(L, 0), 5.0]])
    p = np.concatenate([rng.normal(0, 0.01, 900), [-40.0, -40.0, 40.0, 40.0, 39.0]])
    w = rng.uniform(0.5, 1.5, q.size)
    init = rng.choice(900, 200, replace=False)
    for iters in (0, 3):
        compare(vp, q, p, w, 200, L, iters, init)


@pytest.mark.parametrize("m,k,batch,nbatch", [
    (6000, 500, 900, 8),      # six batches ordered at once, then two
    (6000, 500, 6000, 2),     # a batch of every marker: one at a time
    (6000, 500, 3000, 2),     # two exactly
    (3000, 2900, 700, 4),     # about as many cells as markers: no room for two
    (20000, 1500, 1700, 11),  # eleven at once
    (2000, 150, 1, 40),       # batches of one marker
    (4100, 40, 600, 5)])      # above the runs' mean size: one at a time, by the radix sort
def test_batches_ordered_together(vp, m, k, batch, nbatch):
    """Several mini-batches are put in cell order at once where their records fit."""
    q, p, w, L = landau_markers(m, seed=m + batch)
    rng = np.random.default_rng(batch + nbatch)
    init = rng.choice(m, k, replace=False)
    compare_minibatch(vp, q, p, w, k, L, init, rng.integers(0, m, (nbatch, batch)))
