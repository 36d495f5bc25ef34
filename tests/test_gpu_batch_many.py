"""Batches of many small graphs: the phase log is summed in copies that workgroups share, its first phases apart from
the later ones, and equals the oracle's."""
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


def _path(n):  # increasing weights: one pair a phase, n // 2 phases
    return lmgen.from_edges(n, np.stack([np.arange(n - 1), np.arange(1, n)], 1), np.arange(1, n).astype(np.float32))


def _solve(ctx, gs, weighted=True, **kw):
    """(stats, whether mate, the phases of each graph and the phase log equal the oracle's)"""
    import torch
    vo = np.cumsum([0] + [g.n for g in gs])
    off = np.cumsum([0] + [g.nnz for g in gs])
    rp = np.concatenate([g.row_ptr[:-1] + o for g, o in zip(gs, off)] + [off[-1:]])
    col, w = np.concatenate([g.col for g in gs]), np.concatenate([g.w for g in gs])
    seeds = np.arange(3, 3 + len(gs), dtype=np.uint64)
    want, phases = oracle.local_max_batch(vo, rp, col, w if weighted else np.ones_like(w), seeds=seeds)
    dev = [torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda(), torch.from_numpy(w).cuda() if weighted else None]
    mate, st, gp = ctx.match_batch(vo, *dev, seeds=seeds, **kw)
    assert np.array_equal(mate.cpu().numpy(), want)
    assert np.array_equal(gp, phases) and st.phases == phases.max() == len(st.log)
    assert st.matched_edges == st.log[:, 2].sum() == (want >= 0).sum() // 2
    return st, phases


@pytest.mark.parametrize("graphs", [2, 63, 64, 65, 300])
@pytest.mark.parametrize("longest", [60, 62, 63, 64, 66, 200])
def test_log_of_paths(ctx, graphs, longest):
    """Paths of up to `longest` vertices: phase t matches one edge of every path that has a phase t and leaves two
    vertices fewer, on both sides of the phases that are summed apart."""
    sizes = [longest - (7 * i) % (longest // 2) for i in range(graphs)]
    print(f"case: paths graphs={graphs} longest={longest}", flush=True)
    st, phases = _solve(ctx, [_path(n) for n in sizes])
    for t, rec in enumerate(st.log):
        left = [n - 2 * t for n in sizes if n - 2 * t >= 2]
        assert list(rec[:3]) == [2 * (sum(left) - len(left)), sum(left), len(left)], t


@pytest.mark.parametrize("weighted", [True, False])
def test_many_small_graphs(ctx, weighted):
    gs = [lmgen.er(2 + i % 37, (i * 5) % 60 if i % 37 > 10 else i % 2, i) for i in range(3000)]
    print(f"case: many small graphs weighted={weighted}", flush=True)
    _solve(ctx, gs, weighted)
    _solve(ctx, gs, weighted, check_graph=True)


@pytest.mark.parametrize("graphs,phase_kernels", [(16000, False), (16500, True)])
def test_number_of_graphs(ctx, graphs, phase_kernels):
    """On both sides of the number of graphs (2^14 and one for every 512 vertices) past which the phase kernels solve a
    batch."""
    gs = [lmgen.er(2, 1, 0), lmgen.er(3, 2, 1), lmgen.er(1, 0, 2), lmgen.er(4, 4, 3)]
    print(f"case: {graphs} graphs", flush=True)
    st, _ = _solve(ctx, [gs[i % 4] for i in range(graphs)], profile=True)
    assert (st.kernel_launches["init"] > 0) == phase_kernels


@pytest.mark.parametrize("n", [300, 400])
@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("renew", [False, True])
def test_stream_ordered_dense(ctx, n, weighted, renew):
    """On both sides of the entries (2^17 and a few for the batch's size) past which the device leaves a stream-ordered batch
    to the phase kernels."""
    import torch
    a = np.triu_indices(n, 1)
    g = lmgen.from_edges(n, np.stack(a, 1), (np.arange(len(a[0])) * 7919 % 2003 + 1).astype(np.float32))
    gs = [lmgen.er(300, 1200, 1), g, lmgen.er(1, 0, 3), g]
    vo, off = np.cumsum([0] + [g.n for g in gs]), np.cumsum([0] + [g.nnz for g in gs])
    rp = np.concatenate([g.row_ptr[:-1] + o for g, o in zip(gs, off)] + [off[-1:]])
    col, w = np.concatenate([g.col for g in gs]), np.concatenate([g.w for g in gs])
    seeds = np.arange(3, 3 + len(gs), dtype=np.uint64)
    want, _ = oracle.local_max_batch(vo, rp, col, w if weighted else np.ones_like(w), seeds=seeds, renew=renew)
    dev = [torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda(), torch.from_numpy(w).cuda() if weighted else None]
    mate = torch.full((vo[-1],), -7, dtype=torch.int32, device="cuda")
    for _ in range(3):
        print(f"case: stream-ordered n={n} weighted={weighted} renew={renew}", flush=True)
        ctx.match_batch(vo, *dev, seeds=seeds, renew_keys=renew, asynchronous=True, mate=mate)
        got = mate.clone()
        mate.fill_(-7)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), want)
