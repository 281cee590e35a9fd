"""Small instances run many steps per launch, one workgroup each (the default tuning): against
the oracle at the sizes where the register layout changes, and against one launch per step
(an explicit tuning) for every option, across switches between the two, the history ring, and
the freezing of non-finite instances.

Bars: float64 runs against the oracle 1e-10 (as the persistent steps, whose launches change the
order of sums only); against the fused steps of the same build 1e-12 in float64 over 20 steps,
and 1e-5 in the float32 modes, the stated float32 bar."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("Q", "P", "qs", "ps", "psi")
L = 4 * np.pi


def state(n, seed, dtype=np.float64):
    r = np.random.default_rng(seed)
    st = {"Q": r.uniform(0, L, n), "P": r.normal(0, 1, n), "qs": 0.02 * r.normal(0, 1, n) / n,
          "ps": 0.02 * r.normal(0, 1, n) / n, "psi": r.uniform(0.5, 1.5, n) * (L / n)}
    st = {k: v.astype(dtype) for k, v in st.items()}
    st["Q"] = np.where(st["Q"] >= L, 0, st["Q"]).astype(dtype)
    return st


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("n,ng", [(1, 8), (2, 16), (1023, 64), (1024, 64), (1025, 32), (3000, 1024),
                                  (4096, 512), (4095, 8)])
def test_matches_oracle(vp, n, ng):
    st = state(n, n + ng)
    sim = vp.Simulation(st, L, ng, 0.05, "fp64", hist_cap=32)
    sim.step(20)
    hist = sim.history_array(0, 0, 20)
    got = sim.state_numpy(0)
    ref, _, ref_hist = O.run(st["Q"], st["P"], st["qs"], st["ps"], st["psi"], L, ng, 0.05, 20)
    for f, r in zip(FIELDS, ref):
        assert rel(got[f], r) < 1e-10, f
    for f in ("W", "K", "charge", "momentum"):
        want = np.array([h[f] for h in ref_hist[:20]])
        assert np.max(np.abs(hist[f] - want)) < 1e-10 * max(1.0, np.max(np.abs(want))), f
    assert np.array_equal(hist["step"], np.arange(20))
    sim.close()


OPTIONS = [("fp64", {}, 4096), ("fp64", {"solver": "fft"}, 2500),
           ("fp64", {"projection": "consistent"}, 4000), ("fp64", {"element_order": 2}, 4096),
           ("fp64", {"element_order": 2, "solver": "fft"}, 700),
           ("fp64", {"external": {"amp": 0.3, "mode": 1}}, 2000),
           ("fp64", {"self_field": False, "external": {"amp": 1.0, "mode": 2}}, 4096),
           ("fp64", {"monopole_only": True}, 3001), ("fp32c", {}, 4097), ("fp32c", {}, 8192),
           ("fp32c", {"element_order": 2}, 4000), ("fp32c", {"projection": "nodal"}, 4096),
           ("fp32c", {"projection": "nodal"}, 4097), ("fp32ts", {}, 2048), ("fp32ts", {}, 2049),
           ("fp32ts", {"element_order": 2, "solver": "fft"}, 1025),
           ("fp32", {}, 1024), ("fp32", {}, 1025), ("fp32", {"solver": "fft"}, 900)]


@pytest.mark.parametrize("prec,opt,n", OPTIONS)
def test_matches_fused_steps(vp, prec, opt, n):
    st = state(n, n, np.float64 if prec == "fp64" else np.float32)
    ng, dt = 128, 0.02
    a = vp.Simulation(st, L, ng, dt, prec, hist_cap=16, **opt)
    b = vp.Simulation(st, L, ng, dt, prec, hist_cap=16, **opt)
    b.set_tuning(threads=512, ppt=2, acc_copies=3, graph_steps=3)
    for k in (5, 1, 2, 9, 3):               # single steps are fused launches in both
        a.step(k)
        b.step(k)
    bar = 1e-12 if prec == "fp64" else 1e-5
    ha, hb = a.history_array(0, 4, 16), b.history_array(0, 4, 16)
    for f in ("K", "W", "U", "charge", "momentum"):
        scale = max(np.max(np.abs(hb[f])), np.max(np.abs(hb["K"])))
        assert np.max(np.abs(ha[f] - hb[f])) <= bar * scale, f
    assert np.array_equal(ha["step"], hb["step"])
    a.set_tuning(threads=512, ppt=2, acc_copies=3, graph_steps=3)    # go on from a's ring
    a.step(3)
    b.step(3)
    ga, gb = a.state_numpy(0), b.state_numpy(0)
    for f in FIELDS:
        assert rel(ga[f], gb[f]) <= bar, f
    assert abs(a.diagnostics(0)["W"] - b.diagnostics(0)["W"]) <= bar * abs(b.diagnostics(0)["K"])
    a.close()
    b.close()


def test_batch_and_long_calls(vp):
    """Uneven small instances in one launch, over more steps than a launch takes; admission and
    retirement in between; an instance too large for a workgroup sends all to fused launches."""
    ns = (1, 700, 4096, 2048)
    sts = [state(n, n) for n in ns]
    eng = vp.Engine("fp64", max_slots=5)
    for s, st in enumerate(sts):
        eng.admit(s, st, L, (8, 64, 256, 32)[s], 1e-3, hist_cap=8)
    eng.step(1030)
    eng.admit(4, state(5000, 9), L, 64, 1e-3, hist_cap=8)
    eng.step(4)
    eng.retire(4)
    eng.step(6)
    for s, st in enumerate(sts):
        ref = vp.Simulation(st, L, (8, 64, 256, 32)[s], 1e-3, "fp64", hist_cap=8)
        ref.set_tuning(threads=1024, ppt=2, acc_copies=2)
        ref.step(1040)
        assert eng.slot_status()[s] == (1040, True)
        h, hr = eng.history_array(s, 1032, 8), ref.history_array(0, 1032, 8)
        assert np.max(np.abs(h["W"] - hr["W"])) <= 1e-9 * np.max(np.abs(hr["K"]))
        got, want = eng.retire(s), ref.state_numpy(0)
        for f in FIELDS:
            assert rel(got[f].cpu().numpy(), want[f]) < 1e-9, (s, f)
        ref.close()
    eng.close()


@pytest.mark.parametrize("field,at", [("P", 3), ("psi", 700)])
def test_non_finite_instances_stop_where_fused_steps_freeze_them(vp, field, at):
    st = state(1000, 5)
    st[field][at] = np.nan
    steps = []
    for tuned in (False, True):
        sim = vp.Simulation(st, L, 64, 0.05, "fp64", hist_cap=32)
        if tuned:
            sim.set_tuning(threads=1024, ppt=1, acc_copies=1)
        for k in (2, 2, 4):
            sim.step(k)
        steps.append(sim.slot_status()[0])
        sim.close()
    assert steps[0] == steps[1] and not steps[0][1]
