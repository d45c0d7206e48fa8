"""Cases by which the speed of this library is followed.

Each case is one call, or one short sequence of calls, that a program makes
through ``paper_1601_05527_amd.api``: the whole single-level path on graphs
small enough that launches count, the relaxation and the distances of large
graphs in each storage type, the selections on given distances, the ingest of
an edge list, the property comparison, the multilevel cycle, a captured batch
of graphs, and the derivative with respect to the edge weights.  ``listed()``
takes its sizes from ``paper_1601_05527_amd/workloads.py`` and the tests;
``draw()`` gives more of the same ranges, odd sizes among them.

Graphs are the repository's own seeded generators, drawn on the GPU where it
has a device form.  Distances handed to a selection are those of Gaussian
vertex vectors whose spread falls with the degree (hubs relax towards the
mean first), the shape that relaxed vectors have.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1601_05527_amd import api, graphs

OMEGA = 0.5
DEV = "cuda"


# ----------------------------------------------------------------- cases ---

def listed():
    return [
        # the smallest call of the path: a G(n, m) graph with unit weights, FP64 throughout, fixed exponent
        dict(name="path-gnm-2k-f64", kind="path", graph="gnm", n=2000, m=10_000, R=10, k=20, store="f64",
             orient=0, e=0.5, target=0.0),
        # a small power-law graph, FP32 with its FP64 tail, exponent fitted to a retention
        dict(name="path-chunglu-4k-f32-fit", kind="path", graph="chunglu", n=4096, m=40_000, R=16, k=20,
             store="f32", orient=0, e=0.0, target=0.3),
        # an ordinary graph in the reference precision: FP64 distances ranked in rows of every length
        dict(name="path-chunglu-65k-f64-fit", kind="path", graph="chunglu", n=1 << 16, m=500_000, R=16, k=20,
             store="f64", orient=1, e=0.0, target=0.3),
        # relaxation and distances of the benchmark's power-law graph
        dict(name="relax-chunglu-1m-f32", kind="relax", graph="chunglu", n=1 << 20, m=16_000_000, R=16, k=20,
             store="f32", tail32=0, tail64=3),
        # the same of an R-MAT graph with BF16 storage of the test vectors and its wider last sweeps
        dict(name="relax-rmat-2m-bf16", kind="relax", graph="rmat", n=1 << 21, m=1 << 25, R=16, k=30,
             store="bf16", tail32=12, tail64=1),
        # LOCAL and GLOBAL selections fitted to a retention, from one ranking of given distances
        dict(name="fit-both-chunglu-1m", kind="select", n=1 << 20, m=16_000_000, R=16, dtype="f32", mode="both",
             e=0.0, target=0.3),
        # selection with binning, fitted
        dict(name="binned-chunglu-1m-fit", kind="binned", n=1 << 20, m=16_000_000, R=16, dtype="f32", e=0.0,
             target=0.3),
        # an edge list with some repeats and loops made into the stored graph and its components
        dict(name="ingest-chunglu-16m", kind="ingest", n=1 << 20, m=16_000_000, weighted=True, order="degree"),
        # the sparsified graph compared with the original: subgraph, triangles, components, rank correlations
        dict(name="properties-chunglu-1m", kind="properties", n=1 << 20, m=16_000_000, target=0.3),
        # the multilevel cycle on the benchmark's graph
        dict(name="multilevel-chunglu-1m", kind="multilevel", n=1 << 20, m=16_000_000, R=16, k=20, levels=9,
             n_min=1000, span=3),
        # many graphs of mixed sizes relaxed, measured and sparsified by one captured launch sequence
        dict(name="batch-chunglu-64", kind="batch", G=64, n_lo=1000, n_hi=200_000, R=8, k=20, e=0.5, tail64=3),
        # forward and backward: the gradient with respect to the edge weights of a mesh with long-range edges
        dict(name="adjoint-grid-512", kind="adjoint", side=512, n_long=2616, R=8, k=20, ckpt=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["path", "path", "path", "relax", "relax", "select", "select", "binned", "ingest",
                       "properties", "multilevel", "batch", "adjoint"])

    def size(lo, hi):
        n = _log_int(rng, lo, hi)
        return n, int(n * rng.uniform(4.0, 16.0))

    if kind == "path":
        graph = rng.choice(["gnm", "chunglu", "grid"])
        n, m = size(500, 100_000)
        fit = rng.random() < 0.5
        return dict(kind=kind, graph=graph, n=n, m=m, R=rng.randint(4, 24), k=rng.randint(10, 30),
                    store=rng.choice(["f32", "f64"]), orient=rng.randint(0, 1),
                    e=0.0 if fit else round(rng.uniform(0.2, 0.8), 3), target=round(rng.uniform(0.2, 0.5), 3) if fit else 0.0)
    if kind == "relax":
        store = rng.choice(["f32", "f32", "bf16", "f64"])
        graph = rng.choice(["chunglu", "rmat"])
        n, m = size(20_000, 1_000_000)
        if graph == "rmat":
            n = 1 << max(14, min(20, n.bit_length() - 1))
        return dict(kind=kind, graph=graph, n=n, m=m, R=rng.randint(4, 24), k=rng.randint(16, 30), store=store,
                    tail32=12 if store == "bf16" else 0,
                    tail64={"f32": 3, "bf16": 1, "f64": 0}[store])
    if kind == "select":
        dtype = rng.choice(["f32", "f32", "f64"])
        n, m = size(2000, 1_000_000 if dtype == "f32" else 200_000)
        mode = rng.choice(["both", "local", "global"])
        fit = mode == "both" or rng.random() < 0.5
        return dict(kind=kind, n=n, m=m, R=16, dtype=dtype, mode=mode,
                    e=0.0 if fit else round(rng.uniform(0.2, 0.8), 3), target=round(rng.uniform(0.2, 0.5), 3) if fit else 0.0)
    if kind == "binned":
        n, m = size(2000, 1_000_000)
        fit = rng.random() < 0.5
        return dict(kind=kind, n=n, m=m, R=16, dtype=rng.choice(["f32", "f32", "f64"]),
                    e=0.0 if fit else round(rng.uniform(0.2, 0.8), 3), target=round(rng.uniform(0.2, 0.5), 3) if fit else 0.0)
    if kind == "ingest":
        n, m = size(2000, 1_000_000)
        return dict(kind=kind, n=n, m=m, weighted=rng.random() < 0.7, order=rng.choice(["degree", "degree", "listed"]))
    if kind == "properties":
        n, m = size(2000, 1_000_000)
        return dict(kind=kind, n=n, m=m, target=round(rng.uniform(0.2, 0.5), 3))
    if kind == "multilevel":
        n, m = size(5000, 500_000)
        return dict(kind=kind, n=n, m=m, R=rng.choice([8, 10, 16]), k=rng.randint(10, 20), levels=rng.randint(4, 9),
                    n_min=rng.choice([200, 500, 1000]), span=rng.randint(1, 3))
    if kind == "batch":
        return dict(kind=kind, G=rng.randint(4, 64), n_lo=1000, n_hi=_log_int(rng, 5000, 200_000),
                    R=rng.choice([6, 8, 10, 16]), k=rng.randint(10, 20), e=round(rng.uniform(0.3, 0.7), 3), tail64=3)
    side = _log_int(rng, 32, 512)
    return dict(kind=kind, side=side, n_long=max(1, int(0.01 * side * side)), R=rng.randint(4, 12),
                k=rng.randint(10, 24), ckpt=rng.randint(3, 7))


# --------------------------------------------------------------- prepare ---

def _graph(case, seed):
    """The case's graph as a device dict: row_ptr, col, w, eid, orig_id, edge_u, edge_v, edge_w."""
    kind = case.get("graph", "chunglu")
    if kind == "chunglu":
        return graphs.chung_lu_device(case["n"], case["m"], seed=seed, device=DEV)
    if kind == "rmat":
        return graphs.rmat_device(case["n"].bit_length() - 1, case["m"], seed=seed, device=DEV)
    if kind == "gnm":
        g = graphs.gnm(case["n"], case["m"], seed=seed)
    else:
        side = case.get("side", int(math.isqrt(case.get("n", 1))))
        g = graphs.grid_long_range(side, case.get("n_long", max(1, side * side // 100)), seed=seed)

    def t(a):
        return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(DEV)

    return dict(n=g.n, m=g.m, row_ptr=t(g.row_ptr), col=t(g.col), w=t(g.w), eid=t(g.eid), orig_id=t(g.orig_id),
                edge_u=t(g.edge_u).long(), edge_v=t(g.edge_v).long(), edge_w=t(g.edge_w), d_max=g.d_max)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _distances(d, R, dtype, seed):
    """Distances of Gaussian vertex vectors with spread 1 / sqrt(degree), [m]."""
    dt = torch.float64 if dtype == "f64" else torch.float32
    deg = (d["row_ptr"][1:] - d["row_ptr"][:-1]).clamp(min=1).to(dt)
    z = torch.randn(d["n"], R, generator=_gen(seed), device=DEV, dtype=dt) / deg.sqrt()[:, None]
    rho = torch.empty(d["m"], device=DEV, dtype=dt)
    for a in range(0, d["m"], 1 << 22):
        b = min(d["m"], a + (1 << 22))
        rho[a:b] = (z[d["edge_u"][a:b]] - z[d["edge_v"][a:b]]).square().sum(1).sqrt()
    return rho


def _edge_list(case, seed):
    """The graph's edges under random labels in random order, 2% of them listed twice, 0.5% loops more."""
    d = graphs.chung_lu_device(case["n"], case["m"], seed=seed, device=DEV, degree_order=False)
    g = _gen(seed + 1)
    n, m = d["n"], d["m"]
    u, v, w = d["edge_u"].to(torch.int32), d["edge_v"].to(torch.int32), d["edge_w"]
    twice = torch.randint(0, m, (m // 50,), generator=g, device=DEV)
    loops = torch.randint(0, n, (m // 200,), generator=g, device=DEV, dtype=torch.int32)
    u2, v2 = torch.cat([u, v[twice], loops]), torch.cat([v, u[twice], loops])
    w2 = torch.cat([w, torch.rand(u2.numel() - m, generator=g, device=DEV) + 0.5])
    p = torch.randperm(u2.numel(), generator=g, device=DEV)
    return u2[p].contiguous(), v2[p].contiguous(), w2[p].contiguous() if case["weighted"] else None


def _batch_graphs(case, seed):
    rng = np.random.default_rng(case["G"])       # the sizes are the case's, the graphs the seed's
    ns = np.round(np.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), case["G"]))).astype(np.int64)
    ms = np.round(ns * rng.uniform(8.0, 32.0, case["G"]) / 2).astype(np.int64)
    return [graphs.chung_lu_device(int(n), int(m), seed=seed * 1_000_003 + q, device=DEV)
            for q, (n, m) in enumerate(zip(ns, ms))]


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, seed=seed)
    if kind == "ingest":
        s["u"], s["v"], s["w"] = _edge_list(case, seed)
        return s
    if kind == "batch":
        s["batch"] = api.Batch([api.DeviceGraph.from_tensors(d) for d in _batch_graphs(case, seed)], case["R"],
                               case["k"], OMEGA, seed=seed, e=case["e"], autotune=False, fp64_tail=case["tail64"])
        return s
    d = _graph(dict(case, graph="grid") if kind == "adjoint" else case, seed)
    dg = s["dg"] = api.DeviceGraph.from_tensors(d)
    if kind in ("path", "relax", "adjoint"):
        dg.components()                      # grouped once per graph, like its layout
    if kind in ("select", "binned"):
        s["rho"] = _distances(d, case["R"], case["dtype"], seed + 1)
    if kind == "properties":
        s["keep"] = api.sparsify_fit(dg, _distances(d, 16, "f32", seed + 1), api.AD_LOCAL, case["target"])[0]
    if kind == "adjoint":
        s["w"] = d["edge_w"].clone().requires_grad_(True)
        s["c"] = torch.randn(d["m"], generator=_gen(seed + 1), device=DEV)
    return s


# ------------------------------------------------------------------- run ---

def run(s):
    case, seed = s["case"], s["seed"]
    kind, dg = case["kind"], s.get("dg")
    if kind == "path":
        r = api.sparsify_graph(dg, case["R"], case["k"], case["orient"], e=case["e"],
                               target=case["target"] if case["target"] > 0 else None, omega=OMEGA, seed=seed,
                               store=case["store"], fp64_tail=3)
        return dict(rho=r["rho"], keep=r["keep"], n_kept=r["n_kept"], e=r["e"], x=r["relax"].x,
                    minmax=r["relax"].minmax)
    if kind == "relax":
        res = api.relax(dg, case["R"], case["k"], OMEGA, seed, store=case["store"], fp32_tail=case["tail32"],
                        fp64_tail=case["tail64"])
        return dict(rho=api.distances(dg, res), x=res.x, minmax=res.minmax)
    if kind == "select":
        if case["mode"] == "both":
            kl, kg, nk, (el, eg) = api.sparsify_fit_both(dg, s["rho"], case["target"])
            return dict(keep_local=kl, keep_global=kg, n_kept=nk, e_local=el, e_global=eg)
        orient = api.AD_LOCAL if case["mode"] == "local" else api.AD_GLOBAL
        if case["target"] > 0:
            keep, nk, e = api.sparsify_fit(dg, s["rho"], orient, case["target"])
            return dict(keep=keep, n_kept=nk, e=e)
        keep, nk = api.sparsify(dg, s["rho"], orient, case["e"])
        return dict(keep=keep, n_kept=nk)
    if kind == "binned":
        keep, nk, e = api.sparsify_binned(dg, s["rho"], seed=seed, e=case["e"], target=case["target"])
        return dict(keep=keep, n_kept=nk, e=e)
    if kind == "ingest":
        g = api.ingest(case["n"], s["u"], s["v"], s["w"], order=case["order"])
        c = g.components()
        out = dict(row_ptr=g.row_ptr, col=g.col, eid=g.eid, orig_id=g.orig_id, col_orig=g.col_orig,
                   comp_of=c.comp_of)
        if g.w is not None:
            out["w"] = g.w
        return out
    if kind == "properties":
        return {k: float(v) for k, v in api.compare_properties(dg, s["keep"]).items()}
    if kind == "multilevel":
        keep, kept, depth = api.ml_sparsify(dg, case["R"], case["k"], omega=OMEGA, seed=seed, levels=case["levels"],
                                            n_min=case["n_min"], bin_seed=17, fit=True, span=case["span"], segment=2,
                                            span_value=0.3, fp64_tail=3)
        return dict(keep=keep, n_kept=kept, depth=depth)
    if kind == "batch":
        s["batch"].run()
        rho, keep, nk, mm = s["batch"].fetch()
        return dict(rho=rho, keep=keep, n_kept=nk, minmax=mm)
    rho = api.AlgDist.apply(s["w"], dg, case["R"], case["k"], OMEGA, seed, case["ckpt"])
    gw, = torch.autograd.grad(rho, s["w"], s["c"])
    return dict(rho=rho.detach(), grad_w=gw)


# ------------------------------------------------------------------ work ---

def work(case):
    kind = case["kind"]
    if kind == "batch":
        span = math.log(case["n_hi"] / case["n_lo"])
        n = case["G"] * (case["n_hi"] - case["n_lo"]) / span
        m = 10.0 * n
        b, f = _relax_work(n, m, case["R"], case["k"], 4, True)
        return dict(bytes=b + _dist_bytes(n, m, case["R"], 8) + _select_bytes(n, m, 4), flops=f)
    if kind == "adjoint":
        n, m = case["side"] ** 2, 2 * case["side"] * (case["side"] - 1) + case["n_long"]
        b, f = _relax_work(n, m, case["R"], case["k"], 4, True)
        return dict(bytes=3 * b + 2 * _dist_bytes(n, m, case["R"], 4), flops=4 * f)
    n, m = case["n"], case["m"]
    if case.get("graph") == "grid":
        m = 2 * n
    if kind in ("path", "relax"):
        wide = 8 if case["store"] == "f64" else (2 if case["store"] == "bf16" else 4)
        b, f = _relax_work(n, m, case["R"], case["k"], wide, case["graph"] != "gnm")
        b += _dist_bytes(n, m, case["R"], 8)
        if kind == "path":
            b += _select_bytes(n, m, 8 if case["store"] == "f64" else 4)
        return dict(bytes=b, flops=f + 3 * m * case["R"])
    if kind in ("select", "binned"):
        return dict(bytes=_select_bytes(n, m, 8 if case["dtype"] == "f64" else 4), flops=2 * m * 10)
    if kind == "ingest":                     # the list read, the CSR, ids and components written
        return dict(bytes=m * (12 if case["weighted"] else 8) + 2 * m * (16 if case["weighted"] else 12) + n * 28,
                    flops=m)
    if kind == "properties":                 # the rows read once for each graph, the flags, the scores
        return dict(bytes=2 * m * 8 * (1 + case["target"]) + m + n * 48, flops=2 * m)
    # multilevel: distances on levels whose sizes shrink, twice on the finest three, and the merges between
    b, f = _relax_work(n, m, case["R"], case["k"], 4, True)
    return dict(bytes=2 * (b + _dist_bytes(n, m, case["R"], 8) + _select_bytes(n, m, 4)), flops=2 * f)


def _relax_work(n, m, R, k, wide, weighted):
    per = 2 * m * (8 if weighted else 4) + 12 * n + 2 * n * R * wide
    return float(k * per), float(k * 2 * m * R * 2)


def _dist_bytes(n, m, R, wide):
    return float(8 * n + 4 * 2 * m + 4 * m + n * R * wide + 4 * m)


def _select_bytes(n, m, wide):
    # columns, edge ids and neighbour names of the entries, the distances, the flags
    return float(8 * n + 2 * m * 12 + m * wide + m)


# ----------------------------------------------------------------- exact ---

def exact(case, seed):
    kind = case["kind"]
    if kind == "path":
        d = _graph(case, seed)
        rho, mm, _ = _exact_rho(d, case["R"], case["k"], seed, 0)
        return dict(rho=rho, keep=None, n_kept=None, e=None, x=None, minmax=mm)
    if kind == "relax":
        d = _graph(case, seed)
        rho, mm, _ = _exact_rho(d, case["R"], case["k"], seed, 0)
        return dict(rho=rho, x=None, minmax=mm)
    if kind == "batch":
        got = [_exact_rho(d, case["R"], case["k"], seed, q) for q, d in enumerate(_batch_graphs(case, seed))]
        return dict(rho=torch.cat([g[0] for g in got]), keep=None, n_kept=None,
                    minmax=torch.stack([g[1] for g in got]))
    if kind == "ingest":
        if not case["weighted"]:
            return None
        return dict(row_ptr=None, col=None, eid=None, orig_id=None, col_orig=None, comp_of=None,
                    w=_exact_merge(case, seed))
    if kind == "adjoint":
        return _exact_adjoint(case, seed)
    return None                              # whole numbers, and scores derived from them


def _mulhi(a, b):
    """High 64 bits of the unsigned product of a Python constant and an int64 tensor."""
    mask = 0xffffffff
    al, ah = a & mask, a >> 32
    bl, bh = b & mask, (b >> 32) & mask
    ll, hl, lh, hh = al * bl, ah * bl, al * bh, ah * bh
    cross = ((ll >> 32) & mask) + (hl & mask) + lh
    return ((hl >> 32) & mask) + ((cross >> 32) & mask) + hh


def _signed(c):
    c &= (1 << 64) - 1
    return c - (1 << 64) if c >> 63 else c


def _start(ids, R, seed, gid):
    """x^(0) [n, R]: Philox4x64-10 words, 24 bits each, in [-1/2, 1/2)."""
    nq = (R + 3) // 4
    c0 = ids.long()[:, None].expand(-1, nq).contiguous()
    c1 = torch.arange(nq, device=ids.device)[None, :].expand(ids.numel(), -1).contiguous()
    c2, c3 = torch.zeros_like(c0), torch.zeros_like(c0)
    m0, m1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    k0, k1 = seed, gid
    for _ in range(10):
        n0 = _mulhi(m1, c2) ^ c1 ^ _signed(k0)
        n2 = _mulhi(m0, c0) ^ c3 ^ _signed(k1)
        c0, c1, c2, c3 = n0, c2 * _signed(m1), n2, c0 * _signed(m0)
        k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
    w = torch.stack([c0, c1, c2, c3], 2).reshape(ids.numel(), 4 * nq)[:, :R]
    return ((w >> 40) & 0xffffff).double() * 2.0 ** -24 - 0.5


def _row_sums(values, row_ptr):
    return torch.segment_reduce(values, "sum", offsets=row_ptr, axis=0, initial=0)


def _exact_rho(d, R, k, seed, gid):
    """(rho [m], min then max [2R], x [n, R]) in FP64, one vector at a time."""
    col, rp = d["col"].long(), d["row_ptr"]
    live = rp[1:] > rp[:-1]
    w = torch.ones(col.numel(), dtype=torch.float64, device=col.device) if d["w"] is None else d["w"].double()
    s = torch.where(live, _row_sums(w, rp), torch.ones((), dtype=torch.float64, device=col.device))
    x0 = _start(d["orig_id"], R, seed, gid)
    cols, mm, ss = [], [], torch.zeros(d["m"], dtype=torch.float64, device=col.device)
    for r in range(R):
        x = x0[:, r].contiguous()
        for _ in range(k):
            x = torch.where(live, (1 - OMEGA) * x + OMEGA * _row_sums(w * x[col], rp) / s, x)
        lo, hi = x[live].min(), x[live].max()
        inv = torch.where(hi > lo, 1.0 / (hi - lo), torch.zeros_like(hi))
        ss += ((x[d["edge_u"]] - x[d["edge_v"]]) * inv).square()
        cols.append(x)
        mm.append((lo, hi))
    return ss.sqrt(), torch.stack([p[0] for p in mm] + [p[1] for p in mm]), cols


def _exact_merge(case, seed):
    """The merged weight of every stored entry: FP64 sums of the listed weights, in the CSR's order."""
    u, v, w = _edge_list(case, seed)
    n = case["n"]
    a, b = torch.minimum(u, v).long(), torch.maximum(u, v).long()
    ok = a != b
    key, inv = torch.unique(a[ok] * n + b[ok], return_inverse=True)
    ew = torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, inv, w[ok].double())
    lo, hi = key // n, key % n
    new = torch.arange(n, device=DEV)
    if case["order"] == "degree":
        deg = torch.bincount(torch.cat([lo, hi]), minlength=n)
        new[torch.argsort(-deg * n + torch.arange(n, device=DEV))] = torch.arange(n, device=DEV)
    x, y = new[lo], new[hi]
    return torch.cat([ew, ew])[torch.argsort(torch.cat([x * n + y, y * n + x]))]


def _exact_adjoint(case, seed):
    """FP64 autograd through the sweeps, the rescale and the distances."""
    d = _graph(dict(case, graph="grid"), seed)
    c = torch.randn(d["m"], generator=_gen(seed + 1), device=DEV).double()
    we = d["edge_w"].double().requires_grad_(True)
    rows = torch.repeat_interleave(torch.arange(d["n"], device=DEV), d["row_ptr"][1:] - d["row_ptr"][:-1])
    col, w = d["col"].long(), we[d["eid"].long()]
    s = torch.zeros(d["n"], dtype=torch.float64, device=DEV).index_add(0, rows, w)
    x = _start(d["orig_id"], case["R"], seed, 0)
    for _ in range(case["k"]):
        y = torch.zeros_like(x).index_add(0, rows, w[:, None] * x[col])
        x = (1 - OMEGA) * x + OMEGA * y / s[:, None]
    lo, hi = x.min(0).values, x.max(0).values
    rho = (((x[d["edge_u"]] - x[d["edge_v"]]) / (hi - lo)).square().sum(1)).sqrt()
    grad, = torch.autograd.grad(rho, we, c)
    return dict(rho=rho.detach(), grad_w=grad)
