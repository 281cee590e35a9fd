"""Calls in which one cluster is too large for a run of members and everything is taken again by
the radix sort: the passes before write nothing to the caller's arrays, so outputs that lie over
the inputs, and what follows the last particle, are as in a call that needs no second take."""
from ctypes import byref, c_int32, c_size_t, c_void_p

import numpy as np
import pytest

import oracle as O
from test_gpu_cluster import landau_markers

pytestmark = pytest.mark.gpu

FIELDS = ("Q", "P", "qs", "ps", "psi")


def uneven(m, k, bunch, seed):
    """`bunch` markers at one place, with one starting centre there."""
    q, p, w, L = landau_markers(m, seed=seed)
    rng = np.random.default_rng(seed)
    at = rng.choice(m, bunch, replace=False)
    q[at], p[at] = 3.0, 7.5
    others = np.setdiff1d(np.arange(m), at)
    init = np.concatenate([at[:1], rng.choice(others, k - 1, replace=False)]).astype(np.int32)
    return q, p, w, L, init


def device(torch, *arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).to("cuda") for a in arrays]


@pytest.mark.parametrize("m,k,bunch", [(12000, 400, 700), (30000, 9000, 700), (12000, 400, 512)])
@pytest.mark.parametrize("iters", [0, 3])
def test_outputs_over_the_inputs(vp, m, k, bunch, iters):
    """Q, P and psi are written over Qm, Pm and wm, and the assignment over the (long enough)
    array of starting indices."""
    import torch
    lib = vp.load_library()
    q, p, w, L, init = uneven(m, k, bunch, m + bunch)
    ref, a = O.cluster_markers(q, p, w, init, iters, L)
    n = ref["Q"].shape[0]
    qd, pd, wd = device(torch, q, p, w)
    idx = torch.zeros(m, dtype=torch.int32, device="cuda")
    idx[:k] = torch.from_numpy(init).to("cuda")
    qs = torch.full((k,), -7.0, dtype=torch.float64, device="cuda")
    ps = torch.full((k,), -7.0, dtype=torch.float64, device="cuda")
    b, got_n = c_size_t(), c_int32(-1)
    assert lib.vp_cluster_workspace_bytes(m, k, byref(b)) == 0
    ws = torch.empty(b.value, dtype=torch.uint8, device="cuda")
    ptr = lambda t: c_void_p(t.data_ptr())  # noqa: E731
    st = lib.vp_cluster_markers(ptr(qd), ptr(pd), ptr(wd), m, k, ptr(idx), iters, L, ptr(ws),
                                c_void_p(torch.cuda.current_stream().cuda_stream), ptr(qd), ptr(pd),
                                ptr(qs), ptr(ps), ptr(wd), ptr(idx), byref(got_n))
    assert st == 0 and got_n.value == n
    assert np.array_equal(idx.cpu().numpy(), a.astype(np.int32))
    for name, t, before in (("Q", qd, q), ("P", pd, p), ("psi", wd, w)):
        t = t.cpu().numpy()
        assert np.array_equal(t[:n], ref[name]), name
        assert np.array_equal(t[n:], before[n:]), name      # nothing behind the last particle
    assert np.array_equal(qs.cpu().numpy()[:n], ref["qs"])
    assert np.all(qs.cpu().numpy()[n:] == -7.0) and np.all(ps.cpu().numpy()[n:] == -7.0)


def test_minibatch_absorbed_weights_over_the_weights(vp):
    """The absorbed weights over the marker weights, which the final passes read, in a call whose
    first batch already has a cluster too large for a run."""
    import torch
    lib = vp.load_library()
    m, k = 12000, 400
    q, p, w, L, init = uneven(m, k, 1100, 5)
    bunch = np.flatnonzero((q == 3.0) & (p == 7.5))
    others = np.setdiff1d(np.arange(m), bunch)
    batches = np.stack([np.concatenate([bunch[:900], others[:1100]]), others[2000:4000]]).astype(np.int32)
    out = {f: torch.empty(k, dtype=torch.float64, device="cuda") for f in FIELDS}
    results = []
    for over in (False, True):
        qd, pd, wd = device(torch, q, p, w)
        idx, bidx = device(torch, init, batches)
        absorbed = wd if over else torch.empty(k, dtype=torch.float64, device="cuda")
        b, n = c_size_t(), c_int32(-1)
        assert lib.vp_cluster_minibatch_workspace_bytes(m, k, 2000, byref(b)) == 0
        ws = torch.empty(b.value, dtype=torch.uint8, device="cuda")
        ptr = lambda t: c_void_p(t.data_ptr())  # noqa: E731
        st = lib.vp_cluster_markers_minibatch(
            ptr(qd), ptr(pd), ptr(wd), m, k, ptr(idx), ptr(bidx), 2000, 2, L, ptr(ws),
            c_void_p(torch.cuda.current_stream().cuda_stream), *[ptr(out[f]) for f in FIELDS], None,
            ptr(absorbed), byref(n))
        assert st == 0
        results.append((n.value, absorbed[:k].cpu().numpy(),
                        {f: out[f][:n.value].cpu().numpy().copy() for f in FIELDS}))
    ref, _, v = O.cluster_markers_minibatch(q, p, w, init, batches, L)
    for n, absorbed, got in results:
        assert n == ref["Q"].shape[0]
        assert np.array_equal(absorbed, v)
        for f in ("Q", "P", "psi", "qs"):
            assert np.array_equal(got[f], ref[f]), f
