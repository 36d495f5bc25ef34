"""A stream-ordered solve on the default stream is in order there, also where a
captured graph is asked for beside it (which is then ignored): what is queued
behind the call sees the whole result."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hip_graph", [False, True])
@pytest.mark.parametrize("batch", [False, True])
def test_default_stream_order(batch, hip_graph):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    g = lmgen.er(300000, 1500000, 3)
    e = lmgen.er(500, 900, 4)
    dev = [torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)]
    if batch:  # one graph has too many vertices for one workgroup: the union's phases
        rp = np.concatenate([g.row_ptr, g.nnz + e.row_ptr[1:]]).astype(np.int64)
        col, w = np.concatenate([g.col, e.col]), np.concatenate([g.w, e.w])
        want = oracle.local_max_batch(np.array([0, g.n, g.n + e.n]), rp, col, w, seed0=5)[0]
        dev = [torch.from_numpy(x).cuda() for x in (rp, col, w)]
    else:
        want = oracle.local_max_graph(g, 5)[0]
    want = torch.from_numpy(want.astype(np.int32)).cuda()
    mate = torch.empty_like(want)
    with lm.Context(0) as ctx:
        for k in range(8):
            print(f"case: default stream batch={batch} hip_graph={hip_graph} {k}", flush=True)
            mate.fill_(-7)
            if batch:
                ctx.match_batch([0, g.n, g.n + e.n], *dev, seed0=5, mate=mate, asynchronous=True, hip_graph=hip_graph)
            else:
                ctx.match(*dev, seed=5, mate=mate, asynchronous=True, hip_graph=hip_graph)
            wrong = (mate != want).sum()
            mate.fill_(-9)
            assert int(wrong) == 0
