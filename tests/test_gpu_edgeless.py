"""Graphs with vertices and no entries, weighted (a weight array of length zero)
and not, over every route a solve can take: nothing is matched, no phase."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tail_entries", [0, 3000, 1 << 20])
@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("n", [1, 64, 70000])
def test_no_entries(n, weighted, tail_entries):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    from paper_1302_4587_amd import _lib as L
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    some = torch.zeros(4, device="cuda")  # a pointer that is not null makes the graph weighted
    mate = torch.empty(n, dtype=torch.int32, device="cuda")
    with lm.Context(0) as ctx:
        ctx.set_tuning(tail_entries=tail_entries)
        g = L.Csr(n, 0, rp.data_ptr(), some.data_ptr(), some.data_ptr() if weighted else None)
        dev = L.LM_IN_DEVICE | L.LM_OUT_DEVICE
        for flags in (dev, dev | L.LM_GRAPH, dev | L.LM_ASYNC, dev | L.LM_CHECK_GRAPH, dev | L.LM_RENEW_KEYS, dev | L.LM_PROFILE):
            print(f"case: edgeless n={n} weighted={weighted} tail={tail_entries} flags={flags:#x}", flush=True)
            mate.fill_(-7)
            st = L.Stats()
            ref = None if flags & L.LM_ASYNC else ctypes.byref(st)
            assert ctx._lib.lm_match(ctx.handle, ctypes.byref(g), 1, mate.data_ptr(), flags, None, ref) == L.LM_OK
            torch.cuda.synchronize()
            assert bool((mate == -1).all()) and st.phases == 0 and st.matched_edges == 0
        mate.fill_(-7)
        assert ctx._lib.lm_match_noalloc(ctx.handle, ctypes.byref(g), 1, mate.data_ptr(), dev, None, None) == L.LM_OK
        torch.cuda.synchronize()
        assert bool((mate == -1).all())
        host = np.full(n, -7, np.int32)
        mate_h, st = ctx.match(np.zeros(n + 1, np.int64), np.empty(0, np.int32), np.empty(0, np.float32) if weighted else None,
                               mate=host)
        assert np.all(mate_h == -1) and st.phases == 0
        off = np.array([0, n // 2, n])
        mate_b, st, gp = ctx.match_batch(off, rp, torch.empty(0, dtype=torch.int32, device="cuda"), None)
        assert bool((mate_b == -1).all()) and st.phases == 0 and not gp.any()
