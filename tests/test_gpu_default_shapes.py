"""The default launch shapes: tiles chosen per instance by size, so that one launch holds tiles
of different depth.  Instances at the sizes where the rule turns run together in one engine and
agree with runs of an explicit uniform shape to the order of sums (float64 1e-12 relative over
three steps; float32 states 1e-6: one rounding of the state where a sum's last bit differs),
with a kind of its own (second moments) admitted and retired between the steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 10 * np.pi
FIELDS = ("Q", "P", "qs", "ps")


def state(n, seed, dtype, moments=False):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def r(lo, hi):
        return lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    st = {"Q": r(0, L * (1 - 1e-6)), "P": r(-3, 3), "qs": r(-1, 1) * 1e-2 / n,
          "ps": r(-1, 1) * 1e-2 / n, "psi": r(0.5, 1.5) * (L / n)}
    if moments:
        st.update(Mqq=r(1, 2) * 1e-4 / n, Mqp=r(-1, 1) * 1e-5 / n, Mpp=r(1, 2) * 1e-4 / n)
    return {k: v.to(dtype) for k, v in st.items()}


def rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.mark.parametrize("prec,sizes", [
    ("fp64", (1 << 20, (1 << 20) + 1, 9000, 70000)),
    ("fp32c", ((7 << 19) - 1, 7 << 19, (3 << 19) + 5, 5000)),
    ("fp32c", ((3 << 19), 3000)), ("fp32c", ((7 << 19) - 2,))])   # streamed; plain accesses
def test_tiles_of_several_depths_in_one_launch(vp, prec, sizes):
    import torch
    dt = torch.float64 if prec == "fp64" else torch.float32
    eng = vp.Engine(prec, max_slots=len(sizes) + 1)
    sts = [state(n, n, dt) for n in sizes]
    for s, st in enumerate(sts):
        eng.admit(s, st, L, 64 << (s % 3), 0.02, hist_cap=8)
    eng.step(2)
    k3 = state(600000, 1, dt, True)
    eng.admit(len(sizes), k3, L, 64, 0.02, element_order=2, hist_cap=8)
    eng.step(1)
    eng.retire(len(sizes))
    eng.step(1)
    bar = 1e-12 if prec == "fp64" else 1e-6
    for s, st in enumerate(sts):
        ref = vp.Simulation(st, L, 64 << (s % 3), 0.02, prec, hist_cap=8)
        ref.set_tuning(threads=1024, ppt=4, acc_copies=4)
        ref.step(4)
        h, hr = eng.history_array(s, 0, 4), ref.history_array(0, 0, 4)
        for f in ("K", "W", "charge"):
            assert np.max(np.abs(h[f] - hr[f])) <= 1e-9 * np.max(np.abs(hr["K"])), (s, f)
        got, want = eng.retire(s), ref.retire(0)
        for f in FIELDS:
            assert rel(got[f], want[f]) <= bar, (s, f)
        ref.close()
    eng.close()


def test_get_tuning_keeps_its_defaults(vp):
    sim = vp.Simulation(state(2000, 3, __import__("torch").float64), L, 64, 0.02, "fp64")
    t = sim.get_tuning()
    assert (t["threads"], t["ppt"], t["acc_copies"], t["persistent"]) == (1024, 4, 4, 0)
    sim.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32c", "fp32ts"])
@pytest.mark.parametrize("opt", [{}, {"external": {"amp": 0.2, "mode": 1}}, {"self_field": False},
                                 {"solver": "fft"}])
@pytest.mark.parametrize("n", [1, 1023, 2500])
def test_second_moments_with_and_without_general_options(vp, prec, opt, n):
    """The kernel of k = 3 instances without general options (no field but the mesh's) and the
    general one, through a ragged tile, against the primitive steps of the same build."""
    import torch
    dt = torch.float64 if prec == "fp64" else torch.float32
    st = state(n, n, dt, True)
    a = vp.Simulation(st, L, 64, 0.02, prec, element_order=2, **opt)
    b = vp.Simulation(st, L, 64, 0.02, prec, element_order=2, **opt)
    a.step(1)
    a.sync_state()
    b.gather_push(0.01, 0.02)
    b.deposit()
    b.poisson()
    b.gather_push(0.01, 0.0)
    bar = 1e-12 if prec == "fp64" else 1e-6
    for f in FIELDS + ("Mqq", "Mqp", "Mpp"):
        assert rel(a.state(0)[f], b.state(0)[f]) <= bar, f
    a.close()
    b.close()
