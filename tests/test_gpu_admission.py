"""Admissions, retirements and read-backs that share one upload or one read-back launch: slots
admitted and retired in mixed orders (only the changed tail of the tile table is sent), a
history longer than the pinned read-back memory, and steps before and after graphs are
captured.  Float64 runs of the same input differ in the order of their sums only (1e-12
relative over these horizons, as two runs of one input do)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("Q", "P", "qs", "ps", "psi")


def rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def alone(vp, w, st, steps, **kw):
    sim = vp.Simulation(st, w.L, w.ng, w.dt, "fp64", hist_cap=steps + 1, **kw)
    sim.step(steps)
    out = sim.state_numpy(0)
    sim.close()
    return out


@pytest.mark.parametrize("own_stream", [False, True])
def test_mixed_admissions_match_runs_alone(vp, own_stream):
    import torch
    ws = [W.landau_linear(seed=s, nx=64, nv=40 + 61 * s, ng=64) for s in range(5)]
    sts = [w.state() for w in ws]
    kw = [dict(), dict(element_order=2), dict(solver="fft"), dict(monopole_only=True), dict()]
    for s in (3,):
        sts[s] = {k: v for k, v in sts[s].items() if k not in ("qs", "ps")}
    eng = vp.Engine("fp64", max_slots=6, stream=torch.cuda.Stream() if own_stream else None)
    took = {}
    # the second column: steps taken with those slots resident
    for admits, retires, steps in (((0, 3), (), 3), ((1,), (0,), 2), ((2, 4), (3,), 40),
                                   ((), (1, 4), 5), ((), (2,), 0)):
        for s in admits:
            eng.admit(s, sts[s], ws[s].L, ws[s].ng, ws[s].dt, hist_cap=64, **kw[s])
            took[s] = 0
        eng.step(steps)
        for s in took:
            took[s] += steps
        for s in retires:
            assert eng.slot_status()[s] == (took[s], True)
            got = {k: v.cpu().numpy() for k, v in eng.retire(s).items()}
            ref = alone(vp, ws[s], sts[s], took.pop(s), **kw[s])
            for f in FIELDS:
                assert rel(got[f], ref[f]) < 1e-12, (s, f)
    assert not took
    eng.close()


def test_history_longer_than_the_readback_memory(vp):
    w = W.landau_linear(nx=16, nv=16, ng=16)
    sim = vp.Simulation(w.state(), w.L, w.ng, 1e-4, "fp64", hist_cap=3000)
    sim.step(4000)                     # 3000 records kept, 288 KB; the ring has wrapped
    whole = sim.history_array(0, 1000, 3000)
    parts = np.concatenate([sim.history_array(0, a, 1000) for a in (1000, 2000, 3000)])
    assert np.array_equal(whole["step"], np.arange(1000, 4000))
    for f in ("K", "W", "charge"):
        assert np.array_equal(whole[f], parts[f]), f
    for first, count in ((999, 2), (3999, 2), (-1, 1), (1000, 3001)):
        with pytest.raises(vp.VPError):
            sim.history_array(0, first, count)
    sim.close()


@pytest.mark.parametrize("prepared", [False, True])
def test_steps_before_and_after_capture(vp, prepared):
    """On a stream of its own an engine launches its steps directly until the tables have stood
    for eight graph lengths (here 48 steps), or replays at once when prepared."""
    import torch
    w = W.landau_linear(nx=64, nv=16, ng=64)
    st = w.state()
    sim = vp.Simulation(st, w.L, w.ng, w.dt, "fp64", hist_cap=128, stream=torch.cuda.Stream())
    sim.set_tuning(graph_steps=6)
    if prepared:
        sim.prepare_step(7)
    for k in (7, 40, 13, 1, 20):       # the third call captures
        sim.step(k)
        torch.zeros(8, device="cuda")  # the program's own work between replays
    got = sim.state_numpy(0)
    ref = alone(vp, w, st, 81)
    for f in FIELDS:
        assert rel(got[f], ref[f]) < 1e-12, f
    sim.close()
