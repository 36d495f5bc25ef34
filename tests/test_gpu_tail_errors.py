"""Bad input found by the tail kernel itself, while some of its workgroups have
not started: all of them leave together, and the call ends at once (a workgroup
that left alone would have the others wait out their limit of two seconds)."""
import time

import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["plain", "hip_graph", "noalloc", "noalloc_checked"])
@pytest.mark.parametrize("weighted", [True, False])
def test_bad_offset_ends_at_once(weighted, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    from paper_1302_4587_amd import _lib as L
    g = lmgen.er(70001, 250000, 5)
    good = torch.from_numpy(g.row_ptr).cuda()
    rp = g.row_ptr.copy()
    rp[777] = rp[776] - 1  # among the first rows a workgroup looks at
    bad = torch.from_numpy(rp).cuda()
    col, w = torch.from_numpy(g.col).cuda(), torch.from_numpy(g.w).cuda() if weighted else None
    ones = np.ones_like(g.w)
    want = oracle.local_max(g.n, g.row_ptr, g.col, g.w if weighted else ones, 1)[0]
    with lm.Context(0) as ctx:
        solve, kw = {"plain": (ctx.match, {}), "hip_graph": (ctx.match, {"hip_graph": True}), "noalloc": (ctx.match_noalloc, {}),
                     "noalloc_checked": (ctx.match_noalloc, {"check_graph": True})}[mode]
        assert np.array_equal(solve(good, col, w, seed=1, **kw)[0].cpu().numpy(), want)
        for _ in range(20):
            print(f"case: bad offset {mode} weighted={weighted}", flush=True)
            t = time.perf_counter()
            with pytest.raises(lm.LMError) as e:
                solve(bad, col, w, seed=1, **kw)
            assert e.value.status == L.LM_EGRAPH and time.perf_counter() - t < 0.5
        assert np.array_equal(solve(good, col, w, seed=1, **kw)[0].cpu().numpy(), want)
