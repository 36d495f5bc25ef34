"""Rows of very many entries in single graphs: stars around the lengths from which
a wave's neighbours, a workgroup or several share a row, one and several of them,
their hubs next to each other and apart, among short rows. mate[] and the phase
log equal the oracle's, tolerance 0."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu


def _stars(degrees, weights, seed, shared=False):
    """Stars of the given degrees beside a path; shared: the leaves of one star also hang on the next one's hub."""
    rng = np.random.default_rng(seed)
    hubs = len(degrees)
    n = hubs + sum(degrees) + 300
    edges, at = [], hubs
    for h, d in enumerate(degrees):
        leaf = np.arange(at, at + d)
        edges.append(np.stack([np.full(d, h), leaf], 1))
        if shared and hubs > 1:
            edges.append(np.stack([np.full(d, (h + 1) % hubs), leaf], 1))
        at += d
    p = np.arange(at, n - 1)
    e = np.concatenate(edges + [np.stack([p, p + 1], 1)])
    relabel = rng.permutation(n)
    w = {"uniform": rng.random(len(e)), "tied": rng.integers(1, 3, len(e)), "signed": rng.choice([-2.5, -0.0, 0.0, 1e-40, 3.0], len(e))}[weights]
    return lmgen.from_edges(n, relabel[e], w.astype(np.float32))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


def _check(ctx, g, name, tune):
    import torch
    dev = [torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)]
    ones = np.ones_like(g.w)
    saved = ctx.tuning()
    for weighted in (True, False):
        for renew in (False, True):
            want, log = oracle.local_max(g.n, g.row_ptr, g.col, g.w if weighted else ones, 3, renew=renew)
            for t in tune:
                for kw in ({}, {"hip_graph": True}, {"asynchronous": True}):
                    print(f"case: {name} weighted={weighted} renew={renew} {t} {kw}", flush=True)
                    ctx.set_tuning(**t)
                    mate, st = ctx.match(dev[0], dev[1], dev[2] if weighted else None, seed=3, renew_keys=renew, **kw)
                    torch.cuda.synchronize()
                    ctx.set_tuning(**saved)
                    assert np.array_equal(mate.cpu().numpy(), want)
                    assert st is None or np.array_equal(st.log[:, :3], log * [2, 1, 1])


@pytest.mark.parametrize("weights", ["uniform", "tied", "signed"])
@pytest.mark.parametrize("degrees,shared", [((8191, 8192, 8193, 20000), False), ((90001,), False), ((8193, 12289, 4097, 9001) * 5, True), ((8200,) * 63, False), ((8193,) * 64, False), ((8194,) * 70, False)])
def test_tail_from_the_csr(ctx, degrees, shared, weights):
    g = _stars(degrees, weights, 7, shared)
    assert (1 << 15) < g.nnz <= 1 << 22
    _check(ctx, g, f"hub rows {len(degrees)} {degrees[:4]} {weights}", [{"tail_entries": 1 << 22}])


SEG = 1 << 17  # entries of a slice of a row that several workgroups read


@pytest.mark.parametrize("weights", ["uniform", "tied", "signed"])
@pytest.mark.parametrize("degrees,shared", [((SEG - 1, SEG, SEG + 1, 2 * SEG, 2 * SEG + 1), False), ((5 * SEG + 77, 2049, 300), True), ((150000, 140000, 3000), True)])
def test_first_argmax_of_phases(ctx, degrees, shared, weights):
    g = _stars(degrees, weights, 9, shared)
    assert g.nnz > 500000
    _check(ctx, g, f"slices {degrees} {weights}", [{"tail_entries": 5000}])


def test_time_of_a_large_star(ctx):
    """A row of half a million entries: 0.09 ms, 1.7 ms where one wave reads it."""
    import time
    import torch
    g = _stars((500000,), "uniform", 1)
    dev = [torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)]
    ctx.match(*dev, seed=3)
    t = time.perf_counter()
    for _ in range(20):
        ctx.match(*dev, seed=3)
    assert (time.perf_counter() - t) / 20 < 1e-3
