"""The work a program has this library do, as cases that can be timed.

Four kinds of call, each through the public binding:

* ``match``    one graph solved on the GPU (``Context.match``), or by the
               allocation-free entry point (``Context.match_noalloc``);
* ``batch``    many small graphs in one call (``Context.match_batch``);
* ``contract`` one coarsening step by a matching (``Context.contract``);
* ``serve``    host graphs submitted to a ``Server`` and waited for.

The graphs are the families of the tests and the benchmark (Erdos-Renyi with
uniform weights, 2-D random geometric graphs with weight 1 - distance, R-MAT
with skewed degrees, unweighted or with uniform weights), drawn on the GPU from
the case's seed. The sizes of what comes back belong to the case: the sizes of
a batch's graphs and of the requests do not depend on the seed, and a graph to
be contracted keeps its structure and its pairs while the seed renumbers its
vertices and draws its weights. The matching seed is 1, as in the benchmark.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1302_4587_amd as lm

DEV = "cuda:0"
SEED = 1  # matching seed
M64 = (1 << 64) - 1
LOG_ROWS = 128  # phases of a solve vary by a few with the seed: the log comes back in a table of this many rows


def listed():
    return [
        # The smallest call a program makes: one block of a partitioned problem, latency only.
        {"name": "er_300", "kind": "match", "family": "er", "n": 300, "degree": 8.0, "weighted": True, "mode": "plain"},
        # The smallest configuration of the tests and the smoke run: n = 4096, m = 32768.
        {"name": "er_4096", "kind": "match", "family": "er", "n": 4096, "degree": 16.0, "weighted": True, "mode": "plain"},
        # A solve inside a program that may not allocate, at an odd size.
        {"name": "noalloc_rgg_60k", "kind": "match", "family": "rgg", "n": 60013, "degree": 10.0, "weighted": True, "mode": "noalloc"},
        # A mid-size solve enqueued on the caller's stream, the next work queued behind it.
        {"name": "async_rgg_1m", "kind": "match", "family": "rgg", "n": 1000003, "degree": 10.0, "weighted": True, "mode": "async"},
        # Skewed degrees, unweighted, keys renewed in every phase.
        {"name": "renew_rmat_20", "kind": "match", "family": "rmat", "scale": 20, "weighted": False, "mode": "renew"},
        # The benchmark's weighted graph: RGG with 2^24 vertices.
        {"name": "rgg_2p24", "kind": "match", "family": "rgg", "n": 1 << 24, "degree": 10.0, "weighted": True, "mode": "plain"},
        # The benchmark's headline: R-MAT scale 24, unweighted.
        {"name": "rmat_24", "kind": "match", "family": "rmat", "scale": 24, "weighted": False, "mode": "plain"},
        # A small batch of small unweighted graphs.
        {"name": "batch_64_unweighted", "kind": "batch", "graphs": 64, "lg_lo": 8.0, "lg_hi": 12.0, "d_lo": 4.0, "d_hi": 32.0, "weighted": False},
        # The benchmark's batch: 4096 weighted graphs of 2^8 to 2^16 vertices, average degree 4 to 32.
        {"name": "batch_4096", "kind": "batch", "graphs": 4096, "lg_lo": 8.0, "lg_hi": 16.0, "d_lo": 4.0, "d_hi": 32.0, "weighted": True},
        # A late level of multilevel coarsening: small, weighted, with vertex weights.
        {"name": "contract_rgg_30k", "kind": "contract", "family": "rgg", "n": 30011, "degree": 10.0, "weighted": True, "vwgt": True},
        # The benchmark's skewed contraction: R-MAT scale 24, unweighted.
        {"name": "contract_rmat_24", "kind": "contract", "family": "rmat", "scale": 24, "weighted": False, "vwgt": False},
        # The serving trace's mix, all requests at once: RGG and weighted R-MAT of 2^10 to 2^18 vertices from host memory.
        {"name": "serve_24", "kind": "serve", "requests": 24, "lg_lo": 10.0, "lg_hi": 18.0},
    ]


def _log(rng, lo, hi):
    return int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))


def _draw_graph(rng, lg_lo, lg_hi, weighted=None):
    family = rng.choice(["er", "rgg", "rmat"])
    weighted = (family != "rmat" or rng.random() < 0.5) if weighted is None else weighted
    if family == "rmat":
        return {"family": family, "scale": rng.randint(math.ceil(lg_lo), math.floor(lg_hi)), "weighted": weighted}
    degree = 10.0 if family == "rgg" else round(rng.uniform(4.0, 32.0), 2)
    return {"family": family, "n": _log(rng, 2.0 ** lg_lo, 2.0 ** lg_hi), "degree": degree, "weighted": weighted}


def draw(rng):
    kind = rng.choice(["match", "match", "match", "match", "batch", "batch", "contract", "contract", "serve"])
    if kind == "match":
        mode = rng.choice(["plain", "plain", "async", "graph", "noalloc", "renew"])
        # The allocation-free call holds 64 MiB: 2^16 vertices of any family fit.
        g = _draw_graph(rng, 8.0, 16.0 if mode == "noalloc" else 22.0, None if rng.random() < 0.7 else False)
        return {"kind": kind, "mode": mode, **g}
    if kind == "batch":
        lo = rng.uniform(6.0, 10.0)
        hi = rng.uniform(lo + 1.0, 16.0)
        graphs = _log(rng, 2, max(4, min(4096, 2 ** 26 / 2 ** hi)))
        return {"kind": kind, "graphs": graphs, "lg_lo": round(lo, 3), "lg_hi": round(hi, 3), "d_lo": 4.0, "d_hi": round(rng.uniform(6.0, 32.0), 2),
                "weighted": rng.random() < 0.7}
    if kind == "contract":
        g = _draw_graph(rng, 8.0, 22.0)
        return {"kind": kind, "vwgt": rng.random() < 0.5, **g}
    lo = rng.uniform(8.0, 12.0)
    return {"kind": kind, "requests": rng.randint(4, 40), "lg_lo": round(lo, 3), "lg_hi": round(rng.uniform(lo + 1.0, 18.0), 3)}


# ------------------------------------------------------------------ inputs


def _i64(x):
    """The 64-bit pattern x as a signed Python int, as torch wants it."""
    x &= M64
    return x - (1 << 64) if x >> 63 else x


def _lsr(x, s):
    return (x >> s) & ((1 << (64 - s)) - 1)


def _mix(x):
    """SplitMix64's output function on int64 tensors (products wrap)."""
    x = (x ^ _lsr(x, 30)) * _i64(0xBF58476D1CE4E5B9)
    x = (x ^ _lsr(x, 27)) * _i64(0x94D049BB133111EB)
    return x ^ _lsr(x, 31)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 2654435761 + 12345) & 0x7FFFFFFFFFFF)
    return g


def _pair_weights(row, col, seed):
    """k * 2^-24 with k uniform in [1, 2^24], equal for (u, v) and (v, u)."""
    key = (torch.minimum(row, col) << 32) | torch.maximum(row, col)
    return (_lsr(_mix(key ^ _i64(0x9E3779B97F4A7C15 * (2 * int(seed) + 1))), 40) + 1).float() * 2.0 ** -24


def _symmetric(lo, hi, n, bits):
    """CSR of the undirected pairs (lo < hi, possibly repeated)."""
    key = torch.unique((lo << bits) | hi)
    mask = (1 << bits) - 1
    key = torch.cat([key, ((key & mask) << bits) | (key >> bits)]).sort().values
    rp = torch.searchsorted(key, torch.arange(n + 1, device=DEV) << bits)
    return rp, key


def _er(n, degree, gen):
    m = int(n * degree / 2)
    u = torch.randint(0, n, (m,), device=DEV, generator=gen)
    v = torch.randint(0, n, (m,), device=DEV, generator=gen)
    ok = u != v
    return torch.minimum(u, v)[ok], torch.maximum(u, v)[ok]


def _rmat(scale, gen, edge_factor=16, a=0.57, b=0.19, c=0.19):
    lo, hi = [], []
    total, step = edge_factor << scale, 1 << 26
    for first in range(0, total, step):
        k = min(step, total - first)
        u = torch.zeros(k, dtype=torch.int64, device=DEV)
        v = torch.zeros(k, dtype=torch.int64, device=DEV)
        for _ in range(scale):
            r = torch.rand(k, device=DEV, generator=gen)
            down = r >= a + b
            right = (r >= a) & ~(down & (r < a + b + c))
            u = (u << 1) | down
            v = (v << 1) | right
        ok = u != v
        lo.append(torch.minimum(u, v)[ok])
        hi.append(torch.maximum(u, v)[ok])
    return torch.cat(lo), torch.cat(hi)


def _rgg(n, degree, gen):
    """Points in the unit square, ids in grid-cell order, an edge below the radius of the given mean degree."""
    r = math.sqrt(degree / (math.pi * n))
    cells = max(1, int(1.0 / r))
    x = torch.rand(n, device=DEV, generator=gen, dtype=torch.float64)
    y = torch.rand(n, device=DEV, generator=gen, dtype=torch.float64)
    cell = (y * cells).long().clamp_(max=cells - 1) * cells + (x * cells).long().clamp_(max=cells - 1)
    cell, order = cell.sort()
    x, y = x[order], y[order]
    start = torch.searchsorted(cell, torch.arange(cells * cells + 1, device=DEV))
    deg = torch.zeros(n, dtype=torch.int64, device=DEV)
    cols, ws = [], []
    for p0 in range(0, n, 1 << 21):
        p = torch.arange(p0, min(n, p0 + (1 << 21)), device=DEV)
        cx, cy = cell[p] % cells, cell[p] // cells
        rows = torch.stack([cy - 1, cy, cy + 1], 1)  # the cells of one row of three are neighbours in id order
        inside = (rows >= 0) & (rows < cells)
        rows = rows.clamp(0, cells - 1) * cells
        first = start[rows + (cx - 1).clamp(min=0)[:, None]]
        count = torch.where(inside, start[rows + (cx + 1).clamp(max=cells - 1)[:, None] + 1] - first, 0).reshape(-1)
        first = first.reshape(-1)
        end = count.cumsum(0)
        which = torch.repeat_interleave(torch.arange(len(count), device=DEV), count)
        q = first[which] + torch.arange(len(which), device=DEV) - (end - count)[which]
        src = p[which // 3]
        d2 = (x[src] - x[q]).square() + (y[src] - y[q]).square()
        ok = (d2 < r * r) & (src != q)
        deg += torch.bincount(src[ok], minlength=n)
        cols.append(q[ok].int())
        ws.append((1.0 - d2[ok].sqrt()).float())
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=rp[1:])
    return rp, torch.cat(cols), torch.cat(ws)


def _graph(case, seed, structure=None, shift=0):
    """(row_ptr int64, col int32, w float32 or None) on the GPU. structure: the seed of the edges where it is not the weights'; vertex v gets id (v + shift) mod n."""
    gen = _gen(seed if structure is None else structure)
    if case["family"] == "rgg":
        rp, col, w = _rgg(case["n"], case["degree"], gen)
        if shift:
            n, deg = case["n"], rp.diff()
            head = len(col) - int(rp[n - shift])  # the entries of the last `shift` vertices come first
            rp = torch.zeros_like(rp)
            torch.cumsum(deg.roll(shift), 0, out=rp[1:])
            col, w = ((col + shift) % n).roll(head), w.roll(head)
        return rp, col, w if case["weighted"] else None
    if case["family"] == "er":
        n = case["n"]
        lo, hi = _er(n, case["degree"], gen)
    else:
        n = 1 << case["scale"]
        lo, hi = _rmat(case["scale"], gen)
    if shift:
        lo, hi = (lo + shift) % n, (hi + shift) % n
        lo, hi = torch.minimum(lo, hi), torch.maximum(lo, hi)
    bits = max(1, (n - 1).bit_length())
    rp, key = _symmetric(lo, hi, n, bits)
    del lo, hi
    mask = (1 << bits) - 1
    w = _pair_weights(key >> bits, key & mask, seed) if case["weighted"] else None
    return rp, (key & mask).int(), w


def _batch(case, seed):
    """(vtx_off on the host, row_ptr, local col, w or None): n log-uniform, average degree uniform."""
    G = case["graphs"]
    u = torch.rand(2, G, generator=torch.Generator().manual_seed(17), dtype=torch.float64)
    sizes = torch.round(2.0 ** (case["lg_lo"] + (case["lg_hi"] - case["lg_lo"]) * u[0])).long()
    edges = (sizes * (case["d_lo"] + (case["d_hi"] - case["d_lo"]) * u[1]) / 2).long()
    off = torch.zeros(G + 1, dtype=torch.int64)
    torch.cumsum(sizes, 0, out=off[1:])
    gen, N = _gen(seed), int(off[-1])
    g = torch.repeat_interleave(torch.arange(G, device=DEV), edges.to(DEV))
    n = sizes.to(DEV)[g]
    base = off.to(DEV)[g]
    a = base + (torch.rand(len(g), device=DEV, generator=gen, dtype=torch.float64) * n).long()
    b = base + (torch.rand(len(g), device=DEV, generator=gen, dtype=torch.float64) * n).long()
    del g, n, base
    ok = a != b
    a, b = torch.minimum(a, b)[ok], torch.maximum(a, b)[ok]
    bits = max(1, (N - 1).bit_length())
    rp, key = _symmetric(a, b, N, bits)
    del a, b
    mask = (1 << bits) - 1
    row, col = key >> bits, key & mask
    w = _pair_weights(row, col, seed) if case["weighted"] else None
    col -= torch.repeat_interleave(off[:-1], sizes).to(DEV)[row]
    return off.numpy(), rp, col.int(), w


def _matching(rp, col, shift):
    """A maximal matching (mate int32) of the kind a coarsening program contracts: repeatedly match the edges whose random key beats every neighbour's.
    The keys are those of the ids before the shift."""
    n = len(rp) - 1
    mate = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    row = torch.repeat_interleave(torch.arange(n, device=DEV), rp.diff())
    col = col.long()
    while len(row):
        u, v = (row - shift) % n, (col - shift) % n
        key = _lsr(_mix((torch.minimum(u, v) << 32) | torch.maximum(u, v)), 1)
        best = torch.full((n,), -1, dtype=torch.int64, device=DEV).scatter_reduce_(0, row, key, "amax")
        hit = (best[row] == key) & (best[col] == key)
        mate[row[hit]] = col[hit]
        live = (mate[row] < 0) & (mate[col] < 0)
        row, col = row[live], col[live]
    return mate.int()


def _requests(case, seed):
    u = torch.rand(2, case["requests"], generator=torch.Generator().manual_seed(5), dtype=torch.float64)
    out = []
    for i in range(case["requests"]):
        lg = case["lg_lo"] + (case["lg_hi"] - case["lg_lo"]) * float(u[0, i])
        if u[1, i] < 0.5:
            g = {"family": "rgg", "n": int(round(2.0 ** lg)), "degree": 10.0, "weighted": True}
        else:
            g = {"family": "rmat", "scale": int(round(lg)), "weighted": True}
        out.append(tuple(t.cpu().numpy() for t in _graph(g, int(seed) * 1000 + i)))
    return out


def _contract_inputs(case, seed):
    shift = (int(seed) * 2654435761 + 1) % _size(case)[0]
    rp, col, w = _graph(case, seed, structure=1, shift=shift)
    vwgt = torch.randint(1, 9, (len(rp) - 1,), device=DEV, generator=_gen(seed)) if case["vwgt"] else None
    return rp, col, w, _matching(rp, col, shift), vwgt


def prepare(case, seed):
    state = {"case": case}
    if case["kind"] == "match":
        state["in"] = _graph(case, seed)
    elif case["kind"] == "batch":
        state["in"] = _batch(case, seed)
    elif case["kind"] == "contract":
        state["in"] = _contract_inputs(case, seed)
    else:
        state["in"] = _requests(case, seed)
    torch.cuda.empty_cache()  # what drawing the inputs took is the library's to use
    state["ctx"] = lm.Context(0)
    if case["kind"] == "serve":
        state["server"] = lm.Server(state["ctx"])
    return state


# ------------------------------------------------------------------ one pass


def _log_table(log):
    table = np.zeros((LOG_ROWS, 4), dtype=np.int64)
    table[:len(log)] = log
    return table


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["kind"] == "match":
        rp, col, w = state["in"]
        if case["mode"] == "async":
            mate, _ = ctx.match(rp, col, w, seed=SEED, asynchronous=True)
            return {"mate": mate}
        if case["mode"] == "noalloc":
            mate, st = ctx.match_noalloc(rp, col, w, seed=SEED)
        else:
            mate, st = ctx.match(rp, col, w, seed=SEED, hip_graph=case["mode"] == "graph", renew_keys=case["mode"] == "renew")
        return {"mate": mate, "log": _log_table(st.log), "matched_edges": st.matched_edges}
    if case["kind"] == "batch":
        off, rp, col, w = state["in"]
        mate, st, phases = ctx.match_batch(off, rp, col, w, seed0=SEED)
        return {"mate": mate, "log": _log_table(st.log), "matched_edges": st.matched_edges, "graph_phases": phases}
    if case["kind"] == "contract":
        rp, col, w, mate, vwgt = state["in"]
        cmap, crp, ccol, cw, cvw, _ = ctx.contract(rp, col, w, mate, vwgt, want_vwgt=case["vwgt"])
        return {"cmap": cmap, "row_ptr": crp, "col": ccol, "w": cw, **({"vwgt": cvw} if case["vwgt"] else {})}
    server = state["server"]
    tickets = [server.submit(rp, col, w, seed=SEED) for rp, col, w in state["in"]]
    got = [server.wait(t) for t in tickets]
    return {"mate": [m for m, _ in got], "phases": [st["phases"] for _, st in got][:16]}


# ------------------------------------------------------------------ what a pass cannot do without


def _size(case):
    """(vertices, entries) of a drawn graph, near enough: R-MAT loses more samples to repeats the smaller it is."""
    if case["family"] == "rmat":
        return 1 << case["scale"], (1.0 - 0.5 * 0.89 ** case["scale"]) * (32 << case["scale"])
    return case["n"], case["n"] * case["degree"]


def work(case):
    if case["kind"] == "match":
        n, nnz = _size(case)
        return {"bytes": 8.0 * (n + 1) + (8 if case["weighted"] else 4) * nnz + 4.0 * n, "flops": nnz}
    if case["kind"] == "batch":
        lo, hi = 2.0 ** case["lg_lo"], 2.0 ** case["lg_hi"]
        n = case["graphs"] * (hi - lo) / math.log(hi / lo)
        nnz = n * (case["d_lo"] + case["d_hi"]) / 2
        return {"bytes": 8.0 * n + (8 if case["weighted"] else 4) * nnz + 4.0 * n, "flops": nnz}
    if case["kind"] == "contract":
        n, nnz = _size(case)
        # Coarse sizes as the benchmark's graphs have them: R-MAT keeps nearly all, the others about half the vertices and most entries that no pair merges.
        nc, mc = (0.9 * n, 0.98 * nnz) if case["family"] == "rmat" else (0.53 * n, (0.36 if case["family"] == "rgg" else 0.9) * nnz)
        return {"bytes": 8.0 * n + 4.0 * n + (8 if case["weighted"] else 4) * nnz + 4.0 * n + 8.0 * nc + 8.0 * mc + (8.0 * (n + nc) if case["vwgt"] else 0), "flops": nnz}
    lo, hi = 2.0 ** case["lg_lo"], 2.0 ** case["lg_hi"]
    n = case["requests"] * (hi - lo) / math.log(hi / lo)
    return {"bytes": 8.0 * n + 8 * 0.5 * (10 + 27) * n + 4.0 * n, "flops": 0.5 * (10 + 27) * n}


# ------------------------------------------------------------------ the same in 64 bits


def exact(case, seed):
    """The coarse edge weights of a contraction; everything else that a pass returns is whole numbers."""
    if case["kind"] != "contract":
        return None
    rp, col, w, mate, vwgt = _contract_inputs(case, seed)
    n = len(rp) - 1
    ids, mate = torch.arange(n, device=DEV), mate.long()
    rep = torch.where((mate >= 0) & (mate < ids), mate, ids)
    cmap = ((rep == ids).long().cumsum(0) - 1)[rep]
    nc = int(cmap.max()) + 1
    c = cmap[torch.repeat_interleave(ids, rp.diff())]
    d = cmap[col.long()]
    at = (c != d).nonzero()[:, 0]  # a pair's smaller vertex comes first, so entry order is the order of its two rows
    key, group = torch.unique(c[at] * nc + d[at], return_inverse=True)
    first = torch.full((len(key),), len(col), dtype=torch.int64, device=DEV).scatter_reduce_(0, group, at, "amin")
    total = torch.zeros(len(key), dtype=torch.float64, device=DEV).scatter_add_(0, group, torch.ones_like(at, dtype=torch.float64) if w is None else w[at].double())
    by_first = first.sort().indices
    order = by_first[(key[by_first] // nc).sort(stable=True).indices]
    return {"cmap": None, "row_ptr": None, "col": None, "w": total[order], **({"vwgt": None} if case["vwgt"] else {})}
