"""The tuner tries the shapes that the library chooses by size as well, so that tuning does not take
an engine of small instances off its resident steps (3.7 us a step at 4096 float64 particles,
against 4.8 for the fastest uniform shape), and leaves the state as it found it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 4 * np.pi
FIELDS = ("Q", "P", "qs", "ps", "psi")


def state(n):
    r = np.random.default_rng(n)
    return {"Q": r.uniform(0, L * 0.999, n), "P": r.normal(0, 1, n), "qs": 0.01 * r.normal(0, 1, n) / n,
            "ps": 0.01 * r.normal(0, 1, n) / n, "psi": np.full(n, L / n)}


@pytest.mark.parametrize("sizes", [(4096,), (1000, 300, 2048)])
@pytest.mark.parametrize("before", [{}, {"threads": 512, "ppt": 2}, {"acc_copies": 1}])
def test_small_instances_stay_resident(vp, sizes, before):
    import torch
    eng = vp.Engine("fp64", max_slots=len(sizes), stream=torch.cuda.Stream())
    ref = vp.Engine("fp64", max_slots=len(sizes))
    for s, n in enumerate(sizes):
        eng.admit(s, state(n), L, 64, 1e-3, hist_cap=64)
        ref.admit(s, state(n), L, 64, 1e-3, hist_cap=64)
    if before:
        eng.set_tuning(**before)
    eng.step(3)
    best, us = eng.tune(steps_per_trial=60)
    assert (best["threads"], best["ppt"], best["persistent"]) == (0, 0, 0) and 0 < us < 100
    assert eng.get_tuning() == best
    shape = eng.step_launch(60)
    assert shape["threads"] == 1024 and shape["steps_per_launch"] == 60
    eng.step(7)
    ref.step(10)
    assert all(v == (10, True) for v in eng.slot_status().values())
    for s in range(len(sizes)):
        got, want = eng.retire(s), ref.retire(s)
        for f in FIELDS:
            a, b = got[f].cpu().numpy(), want[f].cpu().numpy()
            assert np.linalg.norm(a - b) <= 1e-12 * np.linalg.norm(b), (s, f)
    eng.close()
    ref.close()
