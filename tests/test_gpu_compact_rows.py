"""The first compaction of one weighted graph by whole rows: rows one entry
below, at and above a lane group's step and a wave's step, empty rows, a few
long rows (taken by a wave alone) and so many that the piece windows take the
launch, with every later phase by the phase kernels or by the tail. mate[] and
the phase log equal the oracle's, tolerance 0."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu

DEGREES = (1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 511, 512, 513, 1023, 1025, 1900)


def _graph(avg, copies, weights, seed):
    """Stars of DEGREES, `copies` times, spread over an ER graph of the given mean degree with empty rows."""
    rng = np.random.default_rng(seed)
    n0 = 80000 if avg < 8 else 24001
    bg = lmgen.er(n0, n0 * avg // 2, seed)
    rows = np.repeat(np.arange(n0), np.diff(bg.row_ptr))
    keep = (rows < bg.col) & (rows % 97 != 0) & (bg.col % 97 != 0)
    edges = [np.stack([rows[keep], bg.col[keep]], 1)]
    step = n0 // (copies * len(DEGREES))
    for i in range(copies * len(DEGREES)):
        d = DEGREES[i % len(DEGREES)]
        leaf = n0 + (i * 4099 + np.arange(d)) % 4200  # leaves are shared
        edges.append(np.stack([np.full(d, i * step), leaf], 1))
    e = np.concatenate(edges)
    w = {"uniform": rng.random(len(e)), "tied": rng.integers(1, 4, len(e)),
         "signed": rng.choice([-2.5, -0.0, 0.0, 1e-40, 3.0], len(e))}[weights]
    return lmgen.from_edges(n0 + 4200, e, w.astype(np.float32))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1302_4587_amd as lm
    with lm.Context(0) as c:
        yield c


@pytest.mark.parametrize("weights", ["uniform", "tied", "signed"])
@pytest.mark.parametrize("avg,copies", [(3, 1), (10, 1), (10, 90), (30, 4), (60, 1)])
def test_compaction_equals_oracle(ctx, avg, copies, weights):
    import torch
    g = _graph(avg, copies, weights, avg + copies)
    assert g.nnz > 100000
    rp, w = torch.from_numpy(g.row_ptr).cuda(), torch.from_numpy(g.w).cuda()
    col = torch.from_numpy(np.concatenate([[0], g.col]).astype(np.int32)).cuda()[1:]  # 4-byte aligned only
    for renew in (False, True):
        want, log = oracle.local_max_graph(g, 5, renew=renew)
        saved = ctx.tuning()
        for tune in ({}, {"tail_entries": 0}, {"grid_per_cu": 1}):
            for kw in ({}, {"hip_graph": True}, {"asynchronous": True}):
                print(f"case: compact avg={avg} copies={copies} {weights} renew={renew} {tune} {kw}", flush=True)
                ctx.set_tuning(**tune)
                mate, st = ctx.match(rp, col, w, seed=5, renew_keys=renew, **kw)
                torch.cuda.synchronize()
                ctx.set_tuning(**saved)
                assert np.array_equal(mate.cpu().numpy(), want)
                if st is not None:
                    assert np.array_equal(st.log[:, :3], log * [2, 1, 1])
