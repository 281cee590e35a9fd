"""Sums that overflow while the state is finite: the resident steps freeze the instance at the
step where one launch per step freezes it, also where that is the last step of a call, with the
same records and state (1e-12 in float64, as the two differ in the order of their sums)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FIELDS = ("Q", "P", "qs", "ps")


def both(vp, st, L, ng, dt, first, **opt):
    """(statuses after `first` and eight more steps, records, state as stepped, diagnostics) of
    either.  The record of the step an instance froze at is left out: reading it solves the field
    of a ring entry the frozen instance did not reach."""
    runs = []
    for tuned in (False, True):
        sim = vp.Simulation(st, L, ng, dt, "fp64", hist_cap=32, **opt)
        if tuned:
            sim.set_tuning(threads=512, ppt=2, acc_copies=1)
        steps = []
        for k in (first, 8):
            sim.step(k)
            steps.append(sim.slot_status()[0])
        n = steps[-1][0]
        state = {f: sim.state(0)[f].cpu().numpy() for f in FIELDS}
        rec = sim.history_array(0, 0, n - 1, allow_nonfinite=True)
        diag = []
        for k in (0, 1, 1):       # the engine's phase goes on: each entry of the ring in turn
            sim.step(k)
            diag.append(sim.diagnostics(0, grid=True, allow_nonfinite=True))
        runs.append((steps, rec, state, diag))
        sim.close()
    return runs


def agree(runs, momentum):
    """`momentum`: the sum of the particles' |psi P|, the scale of the momentum's sum (which may
    cancel)."""
    (sa, ra, ga, da), (sb, rb, gb, db) = runs
    assert sa == sb
    for f in ("K", "W", "U", "charge", "momentum"):
        fin = np.isfinite(rb[f])
        assert np.array_equal(fin, np.isfinite(ra[f])), f
        scale = momentum if f == "momentum" else np.max(np.abs(rb[f][fin]), initial=0.0)
        assert np.all(np.abs(ra[f][fin] - rb[f][fin]) <= 1e-12 * scale), f
    for f in FIELDS:
        assert np.max(np.abs(ga[f] - gb[f])) <= 1e-12 * np.max(np.abs(gb[f])), f
    for k, (x, y) in enumerate(zip(da, db)):
        assert x["step"] == y["step"], k
        for f in ("W", "K"):          # K counts the half-kick pending at that entry
            assert np.isfinite(x[f]) == np.isfinite(y[f]), (k, f)
            assert not np.isfinite(y[f]) or abs(x[f] - y[f]) <= 1e-10 * abs(y[f]), (k, f)
        for f in ("bt", "E"):
            scale = max(np.max(np.abs(y[f])), 1e-300)
            assert np.max(np.abs(x[f] - y[f])) <= 1e-10 * scale, (k, f)


@pytest.mark.parametrize("opt,ng", [({}, 32), ({}, 512), ({"solver": "fft"}, 64),
                                    ({"element_order": 2}, 32),
                                    ({"element_order": 2, "solver": "fft"}, 1024),
                                    ({"projection": "consistent"}, 128)])
@pytest.mark.parametrize("first", [3, 5, 6, 12])
def test_overflowing_field_energy(vp, opt, ng, first):
    """A uniform charge of C bunches by a fiftieth per step: |E| is C / (100 pi) times the steps,
    and the sum of E^2 over the mesh, Ng / 2 of the square of that, overflows in the sixth; K
    (about 1e303) does not."""
    n, L, dt = 2048, np.pi * 1e-6, 1e-82
    charge = 1e155 * np.sqrt(128 / ng)
    q = (np.arange(n) + 0.5) * (L / n)
    st = {"Q": q, "P": 1e74 * np.sin(2 * np.pi * q / L), "qs": np.zeros(n), "ps": np.zeros(n),
          "psi": np.full(n, charge / n)}
    runs = both(vp, st, L, ng, dt, first, **opt)
    steps, rec = runs[1][:2]
    assert 3 < steps[-1][0] < 10 and not steps[-1][1]    # the fused steps froze on the way
    assert np.all(np.isfinite(rec["K"])) and np.all(np.isfinite(rec["W"]))
    agree(runs, charge * 1e74)


@pytest.mark.parametrize("first", range(2, 9))
def test_overflowing_kinetic_energy(vp, first):
    """Particles at one place cross the box once a step, pushed on by a prescribed potential: K
    starts at 0.9 of the largest double, 0.97 two steps later, and overflows in the fourth pass, in
    the middle or at the end of a call."""
    n, L, dt = 700, 4 * np.pi, 1e-100
    P = L / dt
    st = {"Q": np.full(n, 0.75 * L), "P": np.full(n, P), "qs": np.zeros(n), "ps": np.zeros(n),
          "psi": np.full(n, 2 * 0.9 * (1.797e308 / P / P) / n)}
    amp = 0.02 * P / dt / (2 * np.pi / L)
    runs = both(vp, st, L, 64, dt, first, external={"amp": amp, "mode": 1})
    steps, rec = runs[1][:2]
    assert np.isfinite(rec["K"][0]) and not np.isfinite(rec["K"][-1]) and np.all(np.isfinite(rec["W"]))
    assert steps[-1] == (5, False)     # found in the fifth pass, which still ran
    agree(runs, 2 * 1.8e308 / P)
