"""Captured steps of every kind of instance: the whole graph and the one-step graphs, replayed
several times with the program's own work between them, against direct launches of the same build
after each call.  The two differ in the order of their sums only: 1e-12 in float64, one rounding
of the state (1e-6) in the float32 modes with float64 sums, 1e-5 in the naive mode."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 4 * np.pi
FIELDS = ("Q", "P", "qs", "ps")
BAR = {"fp64": 1e-12, "fp32c": 1e-6, "fp32ts": 1e-6, "fp32": 1e-5}
P2, K3 = {"element_order": 2}, {"element_order": 2, "moment_order": 3}
EXT = {"external": {"amp": 0.1, "mode": 1}}


def state(n, prec, kw):
    r = np.random.default_rng(n)
    st = {"Q": r.uniform(0, L * 0.999, n), "P": r.normal(0, 1, n), "qs": 0.01 * r.normal(0, 1, n) / n,
          "ps": 0.01 * r.normal(0, 1, n) / n, "psi": r.uniform(0.5, 1.5, n) * (L / n)}
    if kw.get("moment_order") == 3:
        st.update(Mqq=r.uniform(1, 2, n) * 1e-4 / n, Mqp=np.zeros(n), Mpp=r.uniform(1, 2, n) * 1e-4 / n)
    dt = np.float64 if prec == "fp64" else np.float32
    return {k: v.astype(dt) for k, v in st.items()}


def engine(vp, stream, prec, kinds, tuning, sizes):
    eng = vp.Engine(prec, max_slots=len(kinds), stream=stream)
    for s, (kw, n) in enumerate(zip(kinds, sizes)):
        eng.admit(s, state(n, prec, kw), L, 64 << (s % 2), 1e-3, hist_cap=512, **kw)
    if tuning:
        eng.set_tuning(**tuning)
    return eng


def replay(vp, prec, kinds, tuning, calls, sizes, prepare=None):
    import torch
    stream = torch.cuda.Stream()
    a = engine(vp, stream, prec, kinds, tuning, sizes)
    b = engine(vp, None, prec, kinds, {**(tuning or {}), "use_graph": 0}, sizes)
    assert a.get_tuning()["use_graph"] == 1 and b.get_tuning()["use_graph"] == 0
    if prepare:
        a.prepare_step(prepare)
    for k in calls:
        a.step(k)
        b.step(k)
        torch.zeros(64, device="cuda").add_(1.0)     # the program's own work between replays
        torch.cuda.synchronize()
        for s in range(len(kinds)):
            names = FIELDS + (("Mqq", "Mpp") if "Mqq" in a.state(s) else ())
            for f in names:
                x, y = a.state(s)[f].double(), b.state(s)[f].double()
                assert float((x - y).norm()) <= BAR[prec] * max(float(y.norm()), 1e-300), (k, s, f)
    n = sum(calls)
    assert all(v == (n, True) for v in a.slot_status().values())
    for s in range(len(kinds)):
        ha, hb = a.history_array(s, 0, n), b.history_array(s, 0, n)
        assert np.array_equal(ha["step"], np.arange(n))
        for f in ("K", "W", "U", "charge"):
            scale = max(np.max(np.abs(hb[f])), np.max(np.abs(hb["K"])))
            assert np.max(np.abs(ha[f] - hb[f])) <= BAR[prec] * scale, (s, f)
    a.close()
    b.close()


@pytest.mark.parametrize("prec,kinds", [
    ("fp64", [{}]), ("fp64", [P2]), ("fp64", [K3]), ("fp64", [{"monopole_only": True}]),
    ("fp64", [{"solver": "fft"}]), ("fp64", [EXT]), ("fp64", [{**P2, "solver": "fft"}]),
    ("fp32c", [{}]), ("fp32c", [K3]), ("fp32ts", [P2]), ("fp32", [{}]),
    ("fp64", [{}, P2, K3, {"monopole_only": True}, {"solver": "fft"}, EXT, {**K3, **EXT},
              {**P2, "monopole_only": True}]),
    ("fp32c", [{}, P2, K3, {"monopole_only": True}])])
def test_prepared_replays_match_direct_launches(vp, prec, kinds):
    # graphs of six steps: calls of several graphs, of none, with a lead, and with a rest
    replay(vp, prec, kinds, {"threads": 512, "ppt": 2, "acc_copies": 2, "graph_steps": 6},
           (13, 2, 12, 1, 20), [2500 + 700 * s for s in range(len(kinds))], prepare=20)


@pytest.mark.parametrize("prec", ["fp64", "fp32c"])
def test_default_shapes_are_captured_after_a_while(vp, prec):
    """Untuned: direct launches until the tables have stood for eight graphs of 33 steps."""
    replay(vp, prec, [{}, {"monopole_only": True}], None, (33, 200, 40, 70, 5), [9000, 20000])
