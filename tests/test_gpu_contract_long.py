"""Coarse rows of half a million entries and more: merged through tables in device
memory from 2^19 entries on, in parts where the budget has no room for the
tables. Results equal the oracle's, weights bit for bit."""
import numpy as np
import pytest

import lmgen
from tests.test_gpu_contract import _case

pytestmark = pytest.mark.gpu

LIMIT = 1 << 19


def _hubs(bounds, merged, seed):
    """One free hub per bound, its leaves its own; merged: they are paired among themselves, so that two of a hub's
    entries make one; numbered at random, rows in random order."""
    rng = np.random.default_rng(seed)
    edges, mate, at = [], [], 0
    for u in bounds:
        leaf = np.arange(at + 1, at + 1 + u)
        edges.append(np.stack([np.full(u, at), leaf], 1))
        m = np.full(u + 1, -1)
        if merged:
            k = u // 2 * 2
            m[1:k + 1] = leaf[:k].reshape(-1, 2)[:, ::-1].ravel()
        mate.append(m)
        at += u + 1
    mate, e = np.concatenate(mate), np.concatenate(edges)
    relabel = rng.permutation(at)
    g = lmgen.from_edges(at, relabel[e], rng.random(len(e)).astype(np.float32))
    out = np.full(at, -1, np.int32)
    out[relabel[mate >= 0]] = relabel[mate[mate >= 0]]
    hub_rows = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    order = np.lexsort([rng.random(g.nnz), hub_rows])
    return lmgen.Graph(g.n, g.row_ptr, g.col[order], g.w[order]), out


@pytest.mark.parametrize("unweighted", [False, True])
@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("bounds", [(LIMIT - 1, LIMIT, LIMIT + 1, 20001, 700, 40), (3 * LIMIT + 5, 600), (600, 9000, LIMIT + 8191, 4097, LIMIT + 1, 30)])
def test_very_long_rows_equal_oracle(bounds, merged, unweighted):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    g, mate = _hubs(bounds, merged, len(bounds))
    tables = sum(u > LIMIT for u in bounds)
    need = 8 * g.nnz + 8 * g.n + 4 * (g.n + 1)  # what a contraction holds in any case, and more
    for budget in (0, need + (8 << 20)):
        with lm.Context(0, budget) as ctx:
            for call in range(2):  # the second on the buffers the first left behind
                st = _case(ctx, torch.device("cuda:0"), g, mate, f"long rows {bounds[:3]} merged {merged} budget {budget}", unweighted=unweighted)
                assert st.long_rows == sum(u > 512 for u in bounds) and st.long_entries == sum(u for u in bounds if u > 512)
                assert st.table_rows == (0 if budget else tables)


def test_row_listed_twice_is_refused():
    """A neighbour listed five times in a row with a table, and twice where the input check looks."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    u = LIMIT + 100
    star = lmgen.from_edges(u + 1, np.stack([np.zeros(u, int), np.arange(1, u + 1)], 1), np.ones(u, np.float32))
    col = star.col.copy()
    col[10:14] = col[3]
    dev = [torch.from_numpy(x).cuda() for x in (star.row_ptr, col, star.w)]
    with lm.Context(0) as ctx:
        for f in (lambda: ctx.contract(*dev, torch.full((u + 1,), -1, dtype=torch.int32, device="cuda")), lambda: ctx.match(*dev, check_graph=True)):
            with pytest.raises(lm.LMError) as e:
                f()
            assert e.value.status == lm._lib.LM_EGRAPH
