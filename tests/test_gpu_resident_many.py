"""Engines of many more small instances than the card has CUs: the resident launch takes them in
rounds.  Instances throughout the engine agree with runs alone to the order of sums (1e-12), and
the (hi, lo) pairs leave the resident steps where the line beside resident_capacity says."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 4 * np.pi
FIELDS = ("Q", "P", "qs", "ps")


def state(n, seed, dtype=np.float64):
    r = np.random.default_rng(seed)
    st = {"Q": r.uniform(0, L * 0.999, n), "P": r.normal(0, 1, n), "qs": 0.01 * r.normal(0, 1, n) / n,
          "ps": 0.01 * r.normal(0, 1, n) / n, "psi": r.uniform(0.5, 1.5, n) * (L / n)}
    return {k: v.astype(dtype) for k, v in st.items()}


def test_many_hundreds_of_instances(vp):
    S = 700
    sizes = [1 + (97 * s) % 1500 for s in range(S)]
    sizes[3] = 4096
    eng = vp.Engine("fp64", max_slots=S)
    for s, n in enumerate(sizes):
        eng.admit(s, state(n, s), L, 16 << (s % 4), 1e-3, hist_cap=32)
    shape = eng.step_launch(20)
    assert shape == {"threads": 1024, "ppt": 4, "steps_per_launch": 20}
    eng.step(20)
    eng.step(2)
    assert all(v == (22, True) for v in eng.slot_status().values())
    for s in (0, 1, 3, 255, 256, 257, 511, 512, 600, S - 1):
        ref = vp.Simulation(state(sizes[s], s), L, 16 << (s % 4), 1e-3, "fp64", hist_cap=32)
        ref.set_tuning(threads=512, ppt=2, acc_copies=1)
        ref.step(22)
        h, hr = eng.history_array(s, 0, 22), ref.history_array(0, 0, 22)
        for f in ("K", "W", "charge"):
            assert np.max(np.abs(h[f] - hr[f])) <= 1e-12 * np.max(np.abs(hr["K"])), (s, f)
        got, want = eng.retire(s), ref.retire(0)
        for f in FIELDS:
            a, b = got[f].cpu().numpy(), want[f].cpu().numpy()
            assert np.linalg.norm(a - b) <= 1e-12 * np.linalg.norm(b), (s, f)
        ref.close()
    eng.close()


@pytest.mark.parametrize("slots,n,threads", [(256, 2048, 1024), (257, 2048, 512), (257, 1024, 1024),
                                             (257, 1025, 512)])
def test_pairs_leave_the_resident_steps(vp, slots, n, threads):
    eng = vp.Engine("fp32ts", max_slots=slots)
    st = state(n, 1, np.float32)
    for s in range(slots):
        eng.admit(s, st, L, 64, 1e-3, hist_cap=8)
    assert eng.step_launch(10)["threads"] == threads
    eng.step(10)
    assert all(v == (10, True) for v in eng.slot_status().values())
    eng.close()
