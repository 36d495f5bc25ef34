"""The first phase of one weighted graph by whole rows: rows one entry below,
at and above a lane group's step, the bounds from which a wave or a workgroup
takes a row, and more long rows side by side than a wave keeps for itself, in
graphs too large for a single workgroup. mate[] and the phase log equal the
oracle's, tolerance 0."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu

DEGREES = (15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 511, 512, 513, 2047, 2048, 2049, 9001)


def _graph(avg, weights, seed):
    """Stars of DEGREES (their hubs next to each other) beside an ER graph of the given mean degree."""
    rng = np.random.default_rng(seed)
    n0 = 60000 if avg < 8 else 12000
    bg = lmgen.er(n0, n0 * avg // 2, seed)
    rows = np.repeat(np.arange(n0), np.diff(bg.row_ptr))
    keep = rows < bg.col
    edges = [np.stack([rows[keep], bg.col[keep]], 1)]
    hub, leaf = n0, n0 + len(DEGREES)
    for d in DEGREES:
        edges.append(np.stack([np.full(d, hub), np.arange(leaf, leaf + d)], 1))
        hub, leaf = hub + 1, leaf + d
    e = np.concatenate(edges)
    w = {"uniform": rng.random(len(e)), "tied": rng.integers(1, 4, len(e)), "signed": rng.choice([-2.5, -0.0, 0.0, 1e-40, 3.0], len(e))}[weights]
    return lmgen.from_edges(leaf, e, w.astype(np.float32))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


@pytest.mark.parametrize("weights", ["uniform", "tied", "signed"])
@pytest.mark.parametrize("avg", [4, 10, 30, 60])
def test_rows_equal_oracle(ctx, avg, weights):
    import torch
    g = _graph(avg, weights, avg)
    assert g.nnz > 100000
    rp, w = torch.from_numpy(g.row_ptr).cuda(), torch.from_numpy(g.w).cuda()
    col = torch.from_numpy(np.concatenate([[0], g.col]).astype(np.int32)).cuda()[1:]  # 4-byte aligned only
    for renew in (False, True):
        want, log = oracle.local_max_graph(g, 7, renew=renew)
        modes = [{}, {"hip_graph": True}, {"asynchronous": True}]
        for kw in modes:
            print(f"case: rows avg={avg} {weights} renew={renew} {kw}", flush=True)
            mate, st = ctx.match(rp, col, w, seed=7, renew_keys=renew, **kw)
            torch.cuda.synchronize()
            assert np.array_equal(mate.cpu().numpy(), want)
            if st is not None:
                assert np.array_equal(st.log[:, :3], log * [2, 1, 1])
        if not renew:
            mate, st = ctx.match_noalloc(rp, col, w, seed=7)
            assert np.array_equal(mate.cpu().numpy(), want) and np.array_equal(st.log[:, :3], log * [2, 1, 1])
        saved = ctx.tuning()
        ctx.set_tuning(tail_entries=0)  # every phase by the phase kernels
        mate, st = ctx.match(rp, col, w, seed=7, renew_keys=renew)
        ctx.set_tuning(**saved)
        assert np.array_equal(mate.cpu().numpy(), want) and np.array_equal(st.log[:, :3], log * [2, 1, 1])
