"""One workspace, of the largest call, for calls on either side of the line where the grouping
changes: every call stays inside it (what lies behind is untouched) and gives the oracle's
clusters bit for bit, whatever an earlier call left in it."""
from ctypes import byref, c_int32, c_size_t, c_void_p

import numpy as np
import pytest

import oracle as O
from test_gpu_cluster import landau_markers

pytestmark = pytest.mark.gpu

FIELDS = ("Q", "P", "qs", "ps", "psi")


def test_one_workspace_for_smaller_calls(vp):
    import torch
    lib = vp.load_library()
    largest = (97 * 300, 300, 7000)          # mean 97: the radix sort
    b = c_size_t()
    assert lib.vp_cluster_minibatch_workspace_bytes(*largest, byref(b)) == 0
    guard = 1 << 20
    ws = torch.full((b.value + guard,), 0xa5, dtype=torch.uint8, device="cuda")
    ptr = lambda t: c_void_p(t.data_ptr())  # noqa: E731
    stream = c_void_p(torch.cuda.current_stream().cuda_stream)
    # (m, k, batches of): runs at the line, one batch and several at once, the sort, small calls
    for m, k, batch in ((96 * 300, 300, 0), largest, (96 * 300, 300, 7000), (96 * 300, 300, 1000),
                        (96 * 300 + 1, 300, 0), (5000, 300, 5000), (300, 300, 0), (300, 300, 2)):
        q, p, w, L = landau_markers(m, seed=m + batch)
        rng = np.random.default_rng(m + k)
        init = rng.choice(m, k, replace=False).astype(np.int32)
        dev = [torch.from_numpy(np.ascontiguousarray(x)).to("cuda") for x in (q, p, w, init)]
        out = {f: torch.empty(k, dtype=torch.float64, device="cuda") for f in FIELDS}
        outs, n = [ptr(out[f]) for f in FIELDS], c_int32(-1)
        if batch:
            batches = rng.integers(0, m, (6, batch)).astype(np.int32)
            bd = torch.from_numpy(batches).to("cuda")
            st = lib.vp_cluster_markers_minibatch(*map(ptr, dev[:3]), m, k, ptr(dev[3]), ptr(bd),
                                                  batch, 6, L, ptr(ws), stream, *outs, None, None,
                                                  byref(n))
            ref = O.cluster_markers_minibatch(q, p, w, init, batches, L)[0]
        else:
            st = lib.vp_cluster_markers(*map(ptr, dev[:3]), m, k, ptr(dev[3]), 2, L, ptr(ws), stream,
                                        *outs, None, byref(n))
            ref = O.cluster_markers(q, p, w, init, 2, L)[0]
        assert st == 0 and n.value == ref["Q"].shape[0]
        for f in ("Q", "P", "psi", "qs"):
            assert np.array_equal(out[f][:n.value].cpu().numpy(), ref[f]), (m, k, batch, f)
        assert bool((ws[b.value:] == 0xa5).all()), (m, k, batch)
