"""Batches of graphs with few vertices and many entries: the largest graph's
entries decide between one workgroup per graph and the phase kernels, on the host
where the offsets are there, on the device otherwise. mate[], the phase log and
the per-graph phase counts equal the oracle's on both sides of the line."""
import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu


def _complete(n, seed):
    rng = np.random.default_rng(seed)
    lo, hi = np.triu_indices(n, 1)
    return lmgen.from_edges(n, np.stack([lo, hi], 1), rng.integers(1, 2000, len(lo)).astype(np.float32))


# (graphs, whether the phase kernels take the batch: the limit is about 2^18 entries + 3200 sqrt(vertices) + nnz / 128,
# four fifths of it unweighted)
BATCHES = {
    "under": ([lmgen.er(300, 1200, 1), _complete(500, 2), lmgen.er(1, 0, 3), lmgen.er(90, 100, 4)], False),
    "over": ([lmgen.er(300, 1200, 1), _complete(700, 2), lmgen.er(1, 0, 3), lmgen.er(90, 100, 4)], True),
    "over_first": ([_complete(900, 5), lmgen.er(3000, 9000, 1)], True),
    "several": ([_complete(720, k) for k in range(3)] + [lmgen.er(2000, 16000, 3)], True),
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
@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_dense_batch_equals_oracle(ctx, name, weighted, renew):
    import torch
    gs, phases_take_it = BATCHES[name]
    vo = np.cumsum([0] + [g.n for g in gs])
    off = np.cumsum([0] + [g.nnz for g in gs])
    rp = np.concatenate([g.row_ptr[:-1] + o for g, o in zip(gs, off)] + [off[-1:]])
    col, w = np.concatenate([g.col for g in gs]), np.concatenate([g.w for g in gs])
    if not weighted:
        w = np.ones_like(w)
    seeds = np.arange(3, 3 + len(gs), dtype=np.uint64)
    want, phases = oracle.local_max_batch(vo, rp, col, w, seeds=seeds, renew=renew)
    host = [rp, col, w if weighted else None]
    dev = [torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda(), torch.from_numpy(w).cuda() if weighted else None]
    for args, kw in ((dev, {}), (dev, {"hip_graph": False}), (dev, {"check_graph": True}), (dev, {"profile": True}), (host, {}), (dev, {})):
        print(f"case: dense batch {name} weighted={weighted} renew={renew} host={args is host} {kw}", flush=True)
        mate, st, gp = ctx.match_batch(vo, *args, seeds=seeds, renew_keys=renew, **kw)
        assert np.array_equal(mate if args is host else mate.cpu().numpy(), want)
        assert np.array_equal(gp, phases) and st.phases == phases.max() == len(st.log)
        assert st.log[0, 0] == len(col) and 2 * st.log[:, 2].sum() == (want >= 0).sum()
        if kw.get("profile"):
            assert (st.kernel_launches["init"] > 0) == phases_take_it
    mate = torch.full((vo[-1],), -7, dtype=torch.int32, device="cuda")
    for _ in range(3):  # behind each other on the stream
        print(f"case: dense batch {name} weighted={weighted} renew={renew} asynchronous", flush=True)
        ctx.match_batch(vo, *dev, seeds=seeds, renew_keys=renew, asynchronous=True, mate=mate)
        got = mate.clone()
        mate.fill_(-7)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), want)
