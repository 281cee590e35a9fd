"""The per-pass sums (K, momentum, charge, U) and the field summary (W, E1) of every stepping
kernel against the oracle, each by itself: all of a wavefront's sums share one tree, so a sum
that took another's lanes shows here.  Sums of 3000 float64 terms in a tree and six steps of a
trajectory that follows the oracle's to rounding: 1e-12 of the sum of magnitudes."""

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("Q", "P", "qs", "ps", "psi")


@pytest.mark.parametrize("ext", [None, {"amp": 0.3, "mode": 2}])
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("tuning", [None, dict(persistent=0), dict(persistent=1)])
def test_every_sum_matches_oracle(vp, tuning, order, ext):
    w = W.landau_linear(seed=5, nx=60, nv=50, ng=64)
    w.params["alpha"] = 0.3
    st = w.state()
    st["P"] = st["P"] + 0.7     # a mean momentum
    opts = {} if ext is None else {"external": ext}
    sim = vp.Simulation(st, w.L, w.ng, w.dt, "fp64", hist_cap=16, element_order=order, **opts)
    if tuning is not None:
        sim.set_tuning(threads=512, ppt=2, acc_copies=2, **tuning)
    sim.step(6)
    got = sim.history(0, 0, 6)
    run = O.run if order == 1 else O.run_p2
    ref = run(*(np.asarray(st[k], dtype=np.float64) for k in FIELDS), w.L, w.ng, w.dt, 6,
              ext=ext)[2]
    psi, P = np.asarray(st["psi"]), np.asarray(st["P"])
    # (P of the trajectory stays within a few percent of the start's)
    scale = {"K": 2.0 * np.sum(psi * P * P), "momentum": 2.0 * np.sum(psi * np.abs(P)),
             "charge": np.sum(psi), "U": np.sum(psi), "W": max(r["W"] for r in ref),
             "e1_re": 1.0, "e1_im": 1.0}
    for key, s in scale.items():
        g = np.array([h[key] for h in got])
        r = np.array([h[key] for h in ref[:6]])
        assert np.max(np.abs(g - r)) <= 1e-12 * s, key
    sim.close()
