"""The first phase of one weighted graph by whole rows with phases left to the phase
kernels in every mode: a small hand-over size keeps captured, stream-ordered and
allocation-free solves from starting in the tail kernel, and the profile says which
kernels ran. mate[] and the phase log equal the oracle's, tolerance 0."""
import numpy as np
import pytest

import oracle
from tests import test_gpu_compact_rows, test_gpu_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        c.set_tuning(tail_entries=3000)
        yield c


def _check(ctx, g, name):
    import torch
    rp, w = torch.from_numpy(g.row_ptr).cuda(), torch.from_numpy(g.w).cuda()
    col = torch.from_numpy(np.concatenate([[0], g.col]).astype(np.int32)).cuda()[1:]  # 4-byte aligned only
    for renew in (False, True):
        want, log = oracle.local_max_graph(g, 7, renew=renew)
        for kw in ({}, {"hip_graph": True}, {"asynchronous": True}, {"profile": True}, None):
            print(f"case: {name} renew={renew} {kw}", flush=True)
            if kw is None:
                if renew:
                    continue
                mate, st = ctx.match_noalloc(rp, col, w, seed=7)
            else:
                mate, st = ctx.match(rp, col, w, seed=7, renew_keys=renew, **kw)
            torch.cuda.synchronize()
            assert np.array_equal(mate.cpu().numpy(), want)
            assert st is None or np.array_equal(st.log[:, :3], log * [2, 1, 1])
            if kw and kw.get("profile"):
                ran = st.kernel_launches
                # the first compaction by rows and, for graphs that it leaves, by windows
                assert ran["argmax"] == 1 and ran["compact"] >= 3 and ran["mutual"] >= 2 and ran["tail"] == 1
                assert st.kernel_ms["argmax"] > 0


@pytest.mark.parametrize("weights", ["uniform", "tied", "signed"])
@pytest.mark.parametrize("avg", [4, 10, 30, 60])
def test_rows_in_every_mode(ctx, avg, weights):
    _check(ctx, test_gpu_rows._graph(avg, weights, avg), f"rows avg={avg} {weights}")


@pytest.mark.parametrize("weights", ["uniform", "tied", "signed"])
@pytest.mark.parametrize("avg,copies", [(3, 1), (10, 90), (30, 4)])
def test_compaction_in_every_mode(ctx, avg, copies, weights):
    _check(ctx, test_gpu_compact_rows._graph(avg, copies, weights, avg + copies), f"compact avg={avg} copies={copies} {weights}")


def test_profile_counts_the_listed_rows(ctx):
    """The first argmax's time has the rows left to whole workgroups in it: a star of 3 M leaves keeps them busy for
    several times as long as its leaves' own rows take."""
    import torch
    import lmgen
    u = 3000000
    g = lmgen.from_edges(u + 1, np.stack([np.zeros(u, int), np.arange(1, u + 1)], 1), np.random.default_rng(1).random(u).astype(np.float32))
    n = 3000001
    flat = lmgen.from_edges(n, np.arange(n - 1).reshape(-1, 2), np.ones(n // 2, np.float32))  # as many short rows, no long one
    ms = []
    for x in (g, flat):
        dev = [torch.from_numpy(a).cuda() for a in (x.row_ptr, x.col, x.w)]
        print(f"case: profile of the first argmax nnz={x.nnz}", flush=True)
        ctx.match(*dev, seed=1, profile=True)
        st = [ctx.match(*dev, seed=1, profile=True)[1] for _ in range(5)]
        assert all(s.kernel_launches["argmax"] == 1 for s in st)
        ms.append(min(s.kernel_ms["argmax"] for s in st))
    print(f"first argmax with and without a listed row: {ms}", flush=True)
    assert ms[0] > 1.2 * ms[1]
