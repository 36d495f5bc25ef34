"""Solves by one workgroup per graph at their limits: a batch whose phase log
takes every record it has, entries up to which one graph is solved that way, and results read from elsewhere the moment a call
returns."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


@pytest.mark.parametrize("n", [65535, 65536])
def test_as_many_phases_as_log_records(ctx, n):
    """Increasing weights along a path of the largest number of vertices: only the last edge left is matched in a phase,
    n // 2 phases in all, beside a graph that ends in the first one."""
    import torch
    g = lmgen.from_edges(n, np.stack([np.arange(n - 1), np.arange(1, n)], 1), np.arange(1, n).astype(np.float32))
    e = lmgen.from_edges(2, [(0, 1)], np.ones(1, np.float32))
    rp = np.concatenate([g.row_ptr, g.nnz + e.row_ptr[1:]]).astype(np.int64)
    dev = [torch.from_numpy(x).cuda() for x in (rp, np.concatenate([g.col, e.col]), np.concatenate([g.w, e.w]))]
    print(f"case: path n={n}", flush=True)
    mate, st, phases = ctx.match_batch([0, n, n + 2], *dev, log_cap=40000)
    want = np.full(n + 2, -1)
    top = np.arange(n - 1, 0, -2)
    want[top], want[top - 1] = top - 1, top
    want[n:] = [1, 0]
    assert np.array_equal(mate.cpu().numpy(), want)
    assert list(phases) == [n // 2, 1] and st.phases == len(st.log) == n // 2 and st.matched_edges == n // 2 + 1
    left = n - 2 * np.arange(n // 2)  # vertices of the path left in phase t
    first = np.arange(n // 2) == 0
    assert np.array_equal(st.log[:, 0], 2 * (left - 1) + 2 * first)
    assert np.array_equal(st.log[:, 1], left + 2 * first)
    assert np.array_equal(st.log[:, 2], 1 + first)


@pytest.mark.parametrize("edges", [0, 20000])
@pytest.mark.parametrize("noalloc", [False, True])
def test_result_is_complete_on_return(ctx, noalloc, edges):
    """The call returns once mate holds the result: another stream, which waits for nothing, reads all of it at once."""
    import torch
    n = 60000
    g = lmgen.er(n, edges, 7)
    want = torch.from_numpy(oracle.local_max_graph(g, 5)[0].astype(np.int32)).pin_memory()
    dev = [torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)]
    if not edges:
        dev[1], dev[2] = torch.empty(0, dtype=torch.int32, device="cuda"), None
    mate, other = torch.empty(n, dtype=torch.int32, device="cuda"), torch.cuda.Stream()
    got = torch.empty(n, dtype=torch.int32).pin_memory()
    solve = ctx.match_noalloc if noalloc else ctx.match
    print(f"case: on return noalloc={noalloc} edges={edges}", flush=True)
    for k in range(20):
        mate.fill_(-7)
        torch.cuda.synchronize()
        solve(*dev, seed=5, mate=mate)
        with torch.cuda.stream(other):
            got.copy_(mate, non_blocking=True)
        other.synchronize()
        assert torch.equal(got, want), k


@pytest.mark.parametrize("renew", [False, True])
@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("shape", ["er", "star", "path"])
def test_both_sides_of_the_entry_limit(ctx, shape, weighted, renew):
    """One graph of 2^15 entries (one workgroup) and of two more (the tail kernel)."""
    import torch
    for m in (1 << 14, (1 << 14) + 1):
        if shape == "er":
            g = lmgen.er(5000, m, 5)
        else:
            a = np.arange(m)
            e = np.stack([np.zeros(m, int) if shape == "star" else a, a + 1], 1)
            g = lmgen.from_edges(m + 1, e, np.random.default_rng(m).integers(1, 60, m).astype(np.float32))
        assert g.nnz == 2 * m
        w = g.w if weighted else np.ones_like(g.w)
        want, log = oracle.local_max(g.n, g.row_ptr, g.col, w, 3, renew=renew)
        dev = [torch.from_numpy(g.row_ptr).cuda(), torch.from_numpy(g.col).cuda(), torch.from_numpy(w).cuda() if weighted else None]
        print(f"case: entry limit {shape} m={m} weighted={weighted} renew={renew}", flush=True)
        for kw in ({}, {"hip_graph": True}, {"check_graph": True}):
            mate, st = ctx.match(*dev, seed=3, renew_keys=renew, **kw)
            assert np.array_equal(mate.cpu().numpy(), want)
            assert np.array_equal(st.log[:, :3], log * [2, 1, 1])
