"""The first compaction of one unweighted graph by one-wave ranges: rows one
entry below, at and above a lane's and a step's entries, runs of empty and of
matched rows longer than a window, rows over several ranges, an entry array that
ends inside a step, few and many ranges. mate[] and the phase log (with the
matched entries) equal the oracle's, tolerance 0."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu

DEGREES = (1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 259, 511, 512, 513, 1025, 5000, 23456)


def _graph(n0, avg, seed, extra):
    """Stars of DEGREES between empty rows and paths, beside an ER graph."""
    rng = np.random.default_rng(seed)
    bg = lmgen.er(n0, n0 * avg // 2, seed)
    rows = np.repeat(np.arange(n0), np.diff(bg.row_ptr))
    keep = rows < bg.col
    edges = [np.stack([rows[keep], bg.col[keep]], 1)]
    at = n0
    for i, d in enumerate(DEGREES):
        hub = at + (0, 1, 63, 64, 65, 200)[i % 6]  # (empty rows before it)
        edges.append(np.stack([np.full(d, hub), rng.choice(n0, d, replace=False)], 1))
        at = hub + 1
    pairs = np.arange(at, at + 600).reshape(-1, 2)  # matched at once: 600 matched rows in a row
    edges.append(pairs)
    at += 600 + extra
    e = np.concatenate(edges)
    return lmgen.from_edges(at, e, np.ones(len(e), np.float32))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


@pytest.mark.parametrize("n0,avg,extra", [(24000, 3, 0), (30001, 12, 1), (25002, 45, 130), (400000, 6, 7)])
def test_compaction_equals_oracle(ctx, n0, avg, extra):
    import torch
    g = _graph(n0, avg, avg, extra)
    rp = torch.from_numpy(g.row_ptr).cuda()
    for shift in (0, 1):  # entries aligned to 16 and to 4 bytes
        col = torch.from_numpy(np.concatenate([np.zeros(shift, np.int32), g.col]).astype(np.int32)).cuda()[shift:]
        for renew in (False, True):
            want, log = oracle.local_max_graph(g, 5, renew=renew)
            saved = ctx.tuning()
            for tune in ({"tail_entries": 0}, {"tail_entries": 0, "grid_per_cu": 1}, {"tail_entries": 3000}):
                for kw in ({}, {"hip_graph": True}, {"asynchronous": True}):
                    print(f"case: compact unw n0={n0} avg={avg} shift={shift} renew={renew} {tune} {kw}", flush=True)
                    ctx.set_tuning(**tune)
                    mate, st = ctx.match(rp, col, None, seed=5, renew_keys=renew, **kw)
                    torch.cuda.synchronize()
                    ctx.set_tuning(**saved)
                    assert np.array_equal(mate.cpu().numpy(), want)
                    if st is not None:
                        assert np.array_equal(st.log[:, :3], log * [2, 1, 1])
