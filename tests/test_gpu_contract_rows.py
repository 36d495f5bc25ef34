"""Coarse rows at the sizes where the contraction changes its ways: a tile of
rows, a wave a row, one workgroup, a wide one, several parts, several chunks.
Results equal the oracle's, weights bit for bit."""
import numpy as np
import pytest

import lmgen
import oracle
from tests.test_gpu_contract import _case

pytestmark = pytest.mark.gpu

BOUNDS = (63, 64, 65, 255, 256, 257, 511, 512, 513, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 20001)


def _graph(bounds, merged, seed):
    """One pair {a, b} of hubs per bound, deg(a) + deg(b) the bound. merged = 1: both see the same leaves, which are
    paired among themselves (up to four fine edges a coarse edge); 0: no two entries meet; rows in random order."""
    rng = np.random.default_rng(seed)
    edges, mate, n = [], [], 0
    for u in bounds:
        a, b = n, n + 1
        da = u - u // 2
        shared = int(merged * (u // 2))
        leaves = da + u // 2 - shared
        first = n + 2
        edges += [(a, first + i) for i in range(da)] + [(b, first + (i if i < shared else da + i - shared)) for i in range(u // 2)]
        m = [b, a] + [-1] * leaves
        if merged:
            for i in range(0, leaves - 1, 2):
                m[2 + i], m[3 + i] = first + i + 1, first + i
        mate += m
        n += 2 + leaves
    relabel = rng.permutation(n)
    g = lmgen.from_edges(n, relabel[np.array(edges)], rng.random(len(edges)).astype(np.float32))
    out = np.full(n, -1, np.int32)
    mate = np.array(mate)
    out[relabel[mate >= 0]] = relabel[mate[mate >= 0]]
    order = np.concatenate([s + rng.permutation(e - s) for s, e in zip(g.row_ptr[:-1], g.row_ptr[1:])])
    return lmgen.Graph(n, g.row_ptr, g.col[order], g.w[order]), out


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


@pytest.mark.parametrize("unweighted", [False, True])
@pytest.mark.parametrize("merged", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("bounds", [BOUNDS, BOUNDS[:9], (20001,) * 40])
def test_row_bounds_equal_oracle(ctx, bounds, merged, unweighted):
    import torch
    g, mate = _graph(bounds, merged, len(bounds))
    for call in range(2):  # the second on the buffers the first left behind
        st = _case(ctx, torch.device("cuda:0"), g, mate, f"bounds {bounds[:2]}.. merged {merged}", unweighted=unweighted)
        assert st.table_rows == 0 and st.long_rows == sum(u > 512 for u in bounds)


@pytest.mark.parametrize("u", [40, 300, 900, 3000, 9000])
def test_fifth_fine_edge_is_refused(ctx, u):
    """A neighbour listed five times in one coarse row."""
    import torch
    import paper_1302_4587_amd as lm
    star = lmgen.from_edges(u + 1, [(0, i) for i in range(1, u + 1)], np.ones(u, np.float32))
    col = star.col.copy()
    col[10:14] = col[3]
    dev = [torch.from_numpy(x).cuda() for x in (star.row_ptr, col, star.w, np.full(u + 1, -1, np.int32))]
    with pytest.raises(lm.LMError) as e:
        ctx.contract(*dev)
    assert e.value.status == lm._lib.LM_EGRAPH
