"""GPU parity of graphs solved by one workgroup each (k_solo), at the sizes
where its steps, words, size classes and limits end. Integer work: mate[],
phase counts and the phase log equal the oracle's, tolerance 0."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu


def _stars(degrees):
    """One star per degree: rows as long as a lane group's or a wave's step, one less and one more."""
    edges, n = [], 0
    for d in degrees:
        edges += [(n, n + 1 + i) for i in range(d)]
        n += d + 1
    rng = np.random.default_rng(len(degrees))
    return lmgen.from_edges(n, edges, rng.permutation(len(edges)) + 1)


def _regular(n, d, values, seed):
    """Row lengths close to 2d with weights drawn from `values` (ties, zeros of both signs, negative ones)."""
    rng = np.random.default_rng(seed)
    u = np.repeat(np.arange(n), d)
    v = (u + rng.integers(1, n, len(u))) % n
    key = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
    return lmgen.from_edges(n, np.stack([key // n, key % n], 1), rng.choice(np.array(values, np.float32), len(key)))


def _path(n):
    """Increasing weights along a path: about n / 2 phases of one edge each."""
    return lmgen.from_edges(n, [(i, i + 1) for i in range(n - 1)], np.arange(1, n))


CASES = {
    "steps": [_stars([x + e for x in (4, 8, 16, 32, 64, 128, 256, 512) for e in (-1, 0, 1)])],
    "hub": [_stars([49152])],
    "words": [lmgen.er(n, min(3 * n, n * (n - 1) // 2), n) for n in (1, 2, 31, 32, 33, 63, 64, 65, 511, 512, 513, 1023, 1024, 1025)],
    "rows": [_regular(900, d, [1.0, 2.0, 3.0], d) for d in (1, 2, 3, 5, 6, 10, 11, 12, 21, 22, 45)],
    "signs": [_regular(700, 6, [-2.5, -0.0, 0.0, 2.0**-140, 3.0], 1), _regular(700, 20, [0.0, 0.0], 2)],
    "path": [_path(2001), _path(6)],
    "limit": [lmgen.er(9000, 49152, 5)],
    "over": [lmgen.er(9000, 49153, 5)],
    "limit_unweighted": [lmgen.er(9000, 32768, 5)],
    "over_unweighted": [lmgen.er(9000, 32769, 5)],
    "classes": [lmgen.er(n, 2 * n, n) for n in (2048, 2049, 32768, 32769, 65535, 65536)] + [lmgen.er(5, 3, 1), _stars([65535])],
    "many": [lmgen.er(1 + 7 * i, min(20 * i, (1 + 7 * i) * 7 * i // 2), i) for i in range(320)] + [lmgen.er(40000, 300000, 3), _path(300)],
}


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


@pytest.mark.parametrize("renew", [False, True])
@pytest.mark.parametrize("unweighted", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_solo_equals_oracle(ctx, name, unweighted, renew):
    import torch
    graphs = CASES[name]
    off = np.cumsum([0] + [g.n for g in graphs])
    ent = np.cumsum([0] + [g.nnz for g in graphs])
    rp = np.concatenate([[0]] + [g.row_ptr[1:] + e for g, e in zip(graphs, ent)]).astype(np.int64)
    col = np.concatenate([g.col for g in graphs])
    w = np.concatenate([g.w for g in graphs])
    if unweighted:
        w = np.ones_like(w)
    seeds = np.arange(3, 3 + len(graphs), dtype=np.uint64)
    want, phases = oracle.local_max_batch(off, rp, col, w, seeds=seeds, renew=renew)
    logs = [oracle.local_max(g.n, g.row_ptr, g.col, w[a:a + g.nnz], int(s), renew=renew)[1] for g, a, s in zip(graphs, ent, seeds)]
    total = np.zeros((max(len(x) for x in logs), 3), np.int64)
    for x in logs:
        total[:len(x)] += x
    dev = [torch.from_numpy(x).cuda() for x in (rp, col, w)]
    if unweighted:
        dev[2] = None
    print(f"case: {name} unweighted={unweighted} renew={renew}", flush=True)
    for call in range(2):  # the second on the buffers the first left behind
        mate, st, got = ctx.match_batch(off, *dev, seeds=seeds, renew_keys=renew)
        assert np.array_equal(mate.cpu().numpy(), want)
        assert np.array_equal(got, phases) and st.phases == int(phases.max())
        assert np.array_equal(st.log[:, :3], total[:len(st.log)] * [2, 1, 1]) and len(st.log) == min(st.phases, 4096)
    if len(graphs) == 1:
        for solve in (ctx.match, ctx.match_noalloc):
            if renew and solve == ctx.match_noalloc:
                continue
            kw = {"renew_keys": True} if renew else {}
            mate, st = solve(*dev, seed=3, **kw)
            assert np.array_equal(mate.cpu().numpy(), want)
            assert np.array_equal(st.log[:, :3], total * [2, 1, 1])
