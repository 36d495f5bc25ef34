"""Phases of the device tail with one exchange between workgroups each: rows
one entry below, at and above a lane's row and a wave's step, vertices that end
without a partner in odd and in even phases (mate[] holds the candidates of every
other phase), one graph and unions of graphs, handed over in the first and in
later phases. mate[] (-1 where unmatched), the phase log and the per-graph
phase counts equal the oracle's, tolerance 0."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu

DEGREES = (1, 7, 8, 9, 15, 16, 17, 63, 64, 65, 255, 256, 257, 511, 513, 3001)


def _graph(n0, avg, seed, weights):
    """Stars of DEGREES and chains of falling weights (a phase each) beside an ER graph."""
    rng = np.random.default_rng(seed)
    bg = lmgen.er(n0, n0 * avg // 2, seed)
    rows = np.repeat(np.arange(n0), np.diff(bg.row_ptr))
    keep = rows < bg.col
    edges, w = [np.stack([rows[keep], bg.col[keep]], 1)], [rng.random(int(keep.sum()))]
    at = n0
    for d in DEGREES:  # the star's leaves hang on the ER graph too
        leaf = np.arange(at + 1, at + 1 + d)
        edges += [np.stack([np.full(d, at), leaf], 1), np.stack([leaf, rng.integers(0, n0, d)], 1)]
        w += [rng.random(d), rng.random(d)]
        at += 1 + d
    for k in range(3, 12):
        v = np.arange(at, at + k)
        edges.append(np.stack([v[:-1], v[1:]], 1))
        w.append(2.0 - 0.01 * np.arange(k - 1))
        at += k
    w = np.concatenate(w)
    if weights == "tied":
        w = np.ceil(w * 3)
    elif weights == "none":
        w = np.ones(len(w))
    return lmgen.from_edges(at, np.concatenate(edges), w.astype(np.float32))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


MODES = [({"tail_entries": 1 << 30}, {}), ({"tail_entries": 1 << 30}, {"hip_graph": True}),
         ({"tail_entries": 60000}, {}), ({"tail_entries": 9000}, {"asynchronous": True}), ({"tail_entries": 500}, {})]


@pytest.mark.parametrize("weights", ["uniform", "tied", "none"])
@pytest.mark.parametrize("n0,avg", [(15000, 8), (70000, 5), (9001, 60)])
def test_one_graph(ctx, n0, avg, weights):
    import torch
    g = _graph(n0, avg, avg, weights)
    assert g.nnz > 100000
    dev = [torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)]
    if weights == "none":
        dev[2] = None
    saved = ctx.tuning()
    for renew in (False, True):
        want, log = oracle.local_max_graph(g, 11, renew=renew)
        assert (want < 0).sum() > 100
        for tune, kw in MODES:
            print(f"case: tail phases n0={n0} avg={avg} {weights} renew={renew} {tune} {kw}", flush=True)
            ctx.set_tuning(**tune)
            mate, st = ctx.match(*dev, seed=11, renew_keys=renew, **kw)
            torch.cuda.synchronize()
            ctx.set_tuning(**saved)
            assert np.array_equal(mate.cpu().numpy(), want)
            if st is not None:
                assert np.array_equal(st.log[:, :3], log * [2, 1, 1])


@pytest.mark.parametrize("weights", ["uniform", "none"])
def test_union(ctx, weights):
    import torch
    gs = [_graph(n0, 6, n0, weights) for n0 in (3000, 66000, 500)]  # one above a workgroup's size
    vo = np.cumsum([0] + [g.n for g in gs])
    off = np.cumsum([0] + [g.nnz for g in gs])
    rp = np.concatenate([g.row_ptr[:-1] + o for g, o in zip(gs, off)] + [off[-1:]])
    col, w = np.concatenate([g.col for g in gs]), np.concatenate([g.w for g in gs])
    dev = [torch.from_numpy(x).cuda() for x in (rp, col, w)]
    if weights == "none":
        dev[2] = None
    saved = ctx.tuning()
    for renew in (False, True):
        want, phases = oracle.local_max_batch(vo, rp, col, w, seed0=21, renew=renew)
        for tune in ({"tail_entries": 1 << 30}, {"tail_entries": 60000}, {"tail_entries": 2000}):
            print(f"case: tail phases union {weights} renew={renew} {tune}", flush=True)
            ctx.set_tuning(**tune)
            mate, _, gp = ctx.match_batch(vo, *dev, seed0=21, renew_keys=renew)
            torch.cuda.synchronize()
            ctx.set_tuning(**saved)
            assert np.array_equal(mate.cpu().numpy(), want)
            assert np.array_equal(np.asarray(gp), phases)


@pytest.mark.parametrize("fault", ["end", "start", "falling", "beyond"])
def test_bad_offsets(ctx, fault):
    """A solve that starts in the tail reports offsets that are no CSR's, as the others do."""
    import torch
    import paper_1302_4587_amd as lm
    from paper_1302_4587_amd import _lib as L
    g = _graph(15000, 8, 3, "uniform")
    rp = g.row_ptr.copy()
    at, value = {"end": (-1, g.nnz - 1), "start": (0, 1), "falling": (777, rp[776] - 1), "beyond": (9000, g.nnz + 5)}[fault]
    rp[at] = value
    col, w = torch.from_numpy(g.col).cuda(), torch.from_numpy(g.w).cuda()
    print(f"case: bad offsets {fault}", flush=True)
    with pytest.raises(lm.LMError) as e:
        ctx.match(torch.from_numpy(rp).cuda(), col, w, seed=1)
    assert e.value.status == L.LM_EGRAPH
    mate, _ = ctx.match(torch.from_numpy(g.row_ptr).cuda(), col, w, seed=1)
    assert np.array_equal(mate.cpu().numpy(), oracle.local_max_graph(g, 1)[0])
