"""Solves of several threads at once, a context and a stream each: the tails of
graphs of up to 2^20 entries take a quarter of the resident workgroups at most, so
that four of them are resident together; larger graphs' tails take half, two of
them together. Every result equals the oracle's."""
import threading

import numpy as np
import pytest

import lmgen
import oracle

pytestmark = pytest.mark.gpu


def _run(jobs):
    """Each job (graph, keyword arguments, entry point's name) solved 12 times by a thread of its own."""
    import torch
    import paper_1302_4587_amd as lm
    wants = [torch.from_numpy(oracle.local_max_graph(g, 3)[0].astype(np.int32)).cuda() for g, _, _ in jobs]
    devs = [[torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)] for g, _, _ in jobs]
    torch.cuda.synchronize()
    start, errors = threading.Barrier(len(jobs)), []

    def work(i):
        try:
            torch.cuda.set_device(0)
            g, kw, name = jobs[i]
            with lm.Context(0) as ctx, torch.cuda.stream(torch.cuda.Stream()):
                mate = torch.empty(g.n, dtype=torch.int32, device="cuda")
                start.wait()
                for k in range(12):
                    mate.fill_(-7)
                    getattr(ctx, name)(*devs[i], seed=3, mate=mate, **kw)
                    if int((mate != wants[i]).sum()):
                        errors.append((i, k))
        except Exception as e:  # the thread's failure is the test's
            errors.append((i, repr(e)))
            start.abort()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_four_tails_from_the_csr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: four threads, tails from the CSR", flush=True)
    gs = [lmgen.er(60000, 450000, 1), lmgen.rgg(90000, 10.0, seed=2), lmgen.er(30000, 240000, 3), lmgen.rgg(100000, 10.0, seed=4)]
    assert all(1 << 18 < g.nnz <= 1 << 20 for g in gs)
    _run([(gs[0], {}, "match"), (gs[1], {"asynchronous": True}, "match"), (gs[2], {"hip_graph": True}, "match"), (gs[3], {}, "match_noalloc")])


def test_two_solves_by_phases():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: two threads, phases and a tail each", flush=True)
    gs = [lmgen.er(300000, 2400000, 5), lmgen.rgg(400000, 10.0, seed=6)]
    _run([(gs[0], {"asynchronous": True}, "match"), (gs[1], {}, "match")])


def test_one_workgroup_each():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: six threads, one workgroup each", flush=True)
    _run([(lmgen.er(300 * k, 1500 * k, k), {}, "match") for k in range(1, 7)])
