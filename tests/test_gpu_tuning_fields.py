"""Launch shapes chosen by size, and changes of the tuning's other fields: those keep the shapes,
an explicit shape is taken as it is, and threads = ppt = 0 goes back to shapes by size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 4 * np.pi


def sim(vp, n, prec, **kw):
    r = np.random.default_rng(n)
    dt = np.float64 if prec == "fp64" else np.float32
    st = {"Q": r.uniform(0, L * 0.999, n), "P": r.normal(0, 1, n), "qs": np.zeros(n),
          "ps": np.zeros(n), "psi": np.full(n, L / n)}
    if "element_order" in kw:
        st.update(Mqq=np.full(n, 1e-8), Mqp=np.zeros(n), Mpp=np.full(n, 1e-8))
    return vp.Simulation({k: v.astype(dt) for k, v in st.items()}, L, 64, 0.01, prec, hist_cap=64, **kw)


def shape(s, k=20):
    v = s.step_launch(k)
    return v["threads"], v["ppt"], v["steps_per_launch"]


@pytest.mark.parametrize("prec,n,kw,want", [
    ("fp64", 4096, {}, (1024, 4, 20)), ("fp64", 700, {}, (1024, 1, 20)),
    ("fp64", 4097, {}, (512, 4, 1)), ("fp32c", 8192, {}, (1024, 8, 20)),
    ("fp32c", 8192, {"solver": "fft"}, (512, 4, 1)), ("fp64", (1 << 20) + 1, {}, (512, 8, 1)),
    ("fp64", 1000, {"element_order": 2}, (512, 2, 1)), ("fp32c", 7 << 19, {}, (512, 16, 1)),
    ("fp64", 1000, {"sort_every": 4}, (1024, 1, 4)), ("fp64", 1000, {"sort_every": 1}, (512, 4, 1))])
def test_other_fields_keep_the_shapes(vp, prec, n, kw, want):
    s = sim(vp, n, prec, **kw)
    assert shape(s) == want and shape(s, 1) == (512, s.step_launch(1)["ppt"], 1)
    single = shape(s, 1)
    for field in ({"graph_steps": 6}, {"acc_copies": 2}, {"use_graph": 0}, {"persistent": 0}):
        s.set_tuning(**field)
        assert shape(s) == want and shape(s, 1) == single, field
        assert all(s.get_tuning()[f] == v for f, v in field.items())
    s.step(3)
    s.set_tuning(**s.get_tuning())                 # what is reported now is taken as it was
    assert shape(s) == want
    s.set_tuning(threads=512, ppt=2)
    assert shape(s) == (512, 2, 1)
    s.set_tuning(graph_steps=9)                    # an explicit shape stays as well
    assert shape(s) == (512, 2, 1)
    s.step(3)
    s.set_tuning(threads=0, ppt=0)
    assert shape(s) == want
    s.step(3)
    assert s.slot_status()[0] == (9, True)
    s.close()


def test_shape_fields_are_validated(vp):
    s = sim(vp, 1000, "fp64")
    for bad in ({"threads": 0}, {"threads": 0, "ppt": 4}, {"threads": 512, "ppt": 0},
                {"threads": 0, "ppt": 0, "persistent": 1}, {"graph_steps": 0}):
        with pytest.raises(vp.VPError):
            s.set_tuning(**bad)
        assert shape(s) == (1024, 1, 20)
    s.set_tuning(persistent=1)                     # a shape of its own: 1024 x 4, as before
    assert shape(s) == (1024, 4, 20) and s.get_tuning()["ppt"] == 4
    s.set_tuning(ppt=2)
    assert shape(s) == (1024, 2, 20)
    with pytest.raises(vp.VPError):
        s.step_launch(0)
    with pytest.raises(vp.VPError):
        s.step_launch(1, slot=1)
    s.close()
