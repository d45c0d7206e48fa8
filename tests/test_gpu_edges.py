"""Kernels at the sizes where they can go wrong: edges of tiles and chunks,
remainders, the smallest and largest sizes of a path.  Results that are whole
numbers equal the oracle's; others carry the tolerance stated with the test.
"""
import numpy as np
import pytest

import oracle
from paper_1601_05527_amd import graphs as G

from gpu_helpers import announce

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    from paper_1601_05527_amd import api as _api
    return _api


def _np(t):
    return t.detach().cpu().numpy()


# -------------------------------------------------------------- triangles --

@pytest.mark.parametrize("edge", [2, 15, 16, 31, 32, 63, 1023, 8191])
def test_triangles_at_class_edges(api, edge):
    """Six mutually joined vertices of exactly edge .. edge + 3 and 64, 65
    entries (at least) around an edge of a row class, their other neighbours drawn from one
    pool, so that most triangles lie on two of them; the pool's own rows stay
    short.  Counts are whole numbers."""
    announce(f"triangles at rows of {edge}")
    rng = np.random.default_rng(edge)
    k = 6
    degs = [max(k, d) for d in (edge, edge + 1, edge + 2, edge + 3, 64, 65)]
    pool = max(degs) + 40
    hubs = rng.choice(pool + k, size=k, replace=False)
    rest = np.setdiff1d(np.arange(pool + k), hubs)
    us, vs = [], []
    a, b = np.triu_indices(k, 1)
    us.append(hubs[a])
    vs.append(hubs[b])
    for h, d in zip(hubs, degs):
        x = rng.choice(rest, size=d - (k - 1), replace=False)
        us.append(np.full(x.size, h))
        vs.append(x)
    ring = rng.permutation(rest)
    us.append(ring)
    vs.append(np.roll(ring, 1))
    g = G.from_edges(pool + k, np.concatenate(us), np.concatenate(vs))
    np.testing.assert_array_equal(np.diff(g.row_ptr)[hubs], degs)
    pr = api.graph_properties(api.DeviceGraph.from_host(g, "cuda"))
    ref = oracle.properties(g.n, g.row_ptr, g.col)
    assert ref["lambda"].sum() > 0
    np.testing.assert_array_equal(_np(pr["lambda"]), ref["lambda"])
    np.testing.assert_array_equal(_np(pr["c"]), ref["c"])


@pytest.mark.parametrize("k", [2, 3, 17, 65, 66, 513, 514, 1025, 1026, 1600])
def test_triangles_of_cliques(api, k):
    """Every length of upper-neighbour list up to k - 1 at once: below, at and
    above one table, and several tables.  k vertices have C(k - 1, 2) triangles
    each, a pendant vertex none."""
    announce(f"triangles of a clique of {k}")
    a, b = np.triu_indices(k, 1)
    g = G.from_edges(k + 1, np.append(a, 0), np.append(b, k))
    pr = api.graph_properties(api.DeviceGraph.from_host(g, "cuda"))
    lam = _np(pr["lambda"])
    np.testing.assert_array_equal(lam[:k], np.full(k, (k - 1) * (k - 2) // 2))
    assert lam[k] == 0


@pytest.mark.parametrize("k,leaves", [(2049, 0), (2050, 0), (2200, 0), (1200, 3000)])
def test_triangles_of_wide_cliques(api, k, leaves):
    """Lists of upper neighbours up to, at and past the wide table, the last on rows of
    several workgroups (every vertex of the clique with leaves of its own)."""
    announce(f"triangles of a clique of {k} with {leaves} leaves each")
    a, b = np.triu_indices(k, 1)
    hub = np.repeat(np.arange(k), leaves)
    g = G.from_edges(k + hub.size, np.concatenate([a, hub]), np.concatenate([b, k + np.arange(hub.size)]))
    lam = _np(api.graph_properties(api.DeviceGraph.from_host(g, "cuda"))["lambda"])
    np.testing.assert_array_equal(lam[:k], np.full(k, (k - 1) * (k - 2) // 2))
    assert not lam[k:].any()


def test_triangles_of_hubs(api):
    """Rows beyond one workgroup: two joined hubs that share 9,000 neighbours,
    consecutive ones of which are joined."""
    announce("triangles of hubs")
    n = 9_002
    leaf = np.arange(2, n)
    u = np.concatenate([[0], np.zeros(leaf.size, int), np.ones(leaf.size, int), leaf[:-1]])
    v = np.concatenate([[1], leaf, leaf, leaf[1:]])
    g = G.from_edges(n, u, v)
    pr = api.graph_properties(api.DeviceGraph.from_host(g, "cuda"))
    ref = oracle.properties(g.n, g.row_ptr, g.col)
    np.testing.assert_array_equal(_np(pr["lambda"]), ref["lambda"])


# ------------------------------------------------------------- components --

def _component_graph(kind):
    rng = np.random.default_rng(5)
    if kind == "star-hub-last":                      # no vertex hangs under 0 but through the hub
        n = 70_001
        return G.from_edges(n, np.arange(n - 1), np.full(n - 1, n - 1))
    if kind == "giant-without-0":                    # vertex 0 isolated, a random graph on the rest
        u, v = rng.integers(1, 20_000, 60_000), rng.integers(1, 20_000, 60_000)
        key = np.unique(np.minimum(u, v) * 20_000 + np.maximum(u, v))
        key = key[key // 20_000 != key % 20_000]
        return G.from_edges(20_000, key // 20_000, key % 20_000)
    if kind == "tree":                               # a random tree under random labels
        n = 50_000
        parent = np.array([0] + [rng.integers(max(0, i - 7), i) for i in range(1, n)])
        p = rng.permutation(n)
        return G.from_edges(n, p[np.arange(1, n)], p[parent[1:]])
    if kind == "pairs":                              # thousands of two-vertex components
        n = 12_346
        p = rng.permutation(n)
        return G.from_edges(n, p[0::2], p[1::2])
    # a chain of cliques: long paths of joins between hubs of equal degree
    us, vs = [], []
    for c in range(600):
        a, b = np.triu_indices(9, 1)
        us.append(9 * c + a)
        vs.append(9 * c + b)
        if c:
            us.append(np.array([9 * c - 1]))
            vs.append(np.array([9 * c]))
    g = G.from_edges(9 * 600, np.concatenate(us), np.concatenate(vs))
    return G.relabel(g, rng.permutation(g.n))


@pytest.mark.parametrize("kind", ["star-hub-last", "giant-without-0", "tree", "pairs", "cliques"])
def test_component_labels(api, kind):
    announce(f"component labels {kind}")
    g = _component_graph(kind)
    ref = oracle.properties(g.n, g.row_ptr, g.col)
    got = api.graph_properties(api.DeviceGraph.from_host(g, "cuda"))
    np.testing.assert_array_equal(_np(got["comp"]), ref["comp"])
    assert got["n_components"] == ref["n_components"]


@pytest.mark.parametrize("n", [2, 4095, 4096, 4097, 8193, 70_001])
@pytest.mark.parametrize("stride", [1, 3, 64, 5000])
def test_component_labels_of_banded_orders(api, n, stride):
    """Paths through every stride-th vertex, with cuts, stored in order: chains of parents inside
    and across the workgroups' ranges of 4,096 vertices.  A vertex's label is the smallest of its path."""
    announce(f"component labels of bands n={n} stride={stride}")
    u = np.arange(max(0, n - stride))
    u = u[(u // stride) % 1777 != 1776]
    if u.size == 0:
        u = np.array([0])
    g = G.from_edges(n, u, np.minimum(u + stride, n - 1))
    want = np.arange(n)
    for a, b in zip(g.edge_u, g.edge_v):               # ascending
        want[b] = want[a]
    dg = api.DeviceGraph.from_host(g, "cuda")
    got = api.graph_properties(dg)
    np.testing.assert_array_equal(_np(got["comp"]), want)
    assert got["n_components"] == np.unique(want).size
    c = dg.components()
    live = np.diff(g.row_ptr) > 0
    assert c.n_comp == np.unique(want[live]).size
    np.testing.assert_array_equal(_np(c.comp_of)[:n] >= 0, live)


# ------------------------------------------------------------------ batch --

@pytest.mark.parametrize("sizes", [(16384, 1, 16383, 15, 17, 16385), (3, 5, 7, 40_000, 2), (32768,)])
def test_batch_counts_at_chunk_edges(api, sizes):
    """Kept counts of graphs whose edge ranges start and end at, before and
    after the counting kernel's chunks of 16,384 edges."""
    announce(f"batch counts {sizes}")
    dgs = [api.DeviceGraph.from_host(G.gnm(m // 3, m, q) if m > 20 else
                                     G.from_edges(m + 1, np.arange(m), np.arange(1, m + 1)), "cuda")
           for q, m in enumerate(sizes)]
    b = api.Batch(dgs, 4, 5, seed=1, e=0.4, autotune=False)
    b.run()
    _, keep, n_kept, _ = [_np(t) for t in b.fetch()]
    for q in range(len(sizes)):
        assert n_kept[q] == keep[b.edge_off[q]:b.edge_off[q + 1]].sum(), q
    b.close()


# --------------------------------------------------- FP64 distances ranked --

def _counted_ranks(g, rho, i):
    """(LOCAL, GLOBAL) ranks of row i's entries by counting comparisons (a NaN
    compares with nothing), ties by the neighbour's id."""
    p = slice(g.row_ptr[i], g.row_ptr[i + 1])
    r, ids = rho[g.eid[p]], g.orig_id[g.col[p]]
    d = len(r)
    order = np.argsort(r, kind="stable")
    s = r[order]
    n_num = d - int(np.isnan(r).sum())
    lt = np.searchsorted(s[:n_num], r, "left")
    eq = np.searchsorted(s[:n_num], r, "right") - lt
    eqlt = np.zeros(d, np.int64)
    for k in np.nonzero(eq > 1)[0]:
        eqlt[k] = np.sum((r == r[k]) & (ids < ids[k]))
    lt[np.isnan(r)] = 0
    eq[np.isnan(r)] = 0
    return lt + eqlt, d - lt - eq + eqlt


@pytest.mark.parametrize("values", ["distances", "quantised", "special"])
def test_fp64_rows_of_every_length(api, values):
    """FP64 selection on rows at the bounds of every sort and of the bucket
    partition (up to 40,000 entries), with ties, and with infinities, signed
    zeros, negative values and NaNs, against ranks counted on the host."""
    announce(f"fp64 rows {values}")
    rng = np.random.default_rng(8)
    degs = [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 12_000, 40_000]
    us, vs, n = [], [], 0
    leaf = len(degs)
    for q, d in enumerate(degs):                       # stars, whose leaves are chained in threes
        us.append(np.full(d, q))
        vs.append(np.arange(leaf, leaf + d))
        leaf += d
    chain = np.arange(len(degs), leaf - 1)
    chain = chain[chain % 3 != 0]
    g = G.from_edges(leaf, np.concatenate(us + [chain]), np.concatenate(vs + [chain + 1]))
    rho = rng.random(g.m)
    if values == "quantised":
        rho = np.round(rho, 2)
    elif values == "special":
        pick = rng.integers(0, 12, g.m)
        for k, v in enumerate([np.nan, np.inf, -np.inf, 0.0, -0.0, -0.25]):
            rho[pick == k] = v
    dg = api.DeviceGraph.from_host(g, "cuda")
    t = torch.from_numpy(rho).cuda()
    for orient, e in ((0, 0.5), (1, 0.7)):
        keep, nk = api.sparsify(dg, t, orient, e)
        bud = api.budget_table(g.d_max, e)
        ref = np.zeros(g.m, np.uint8)
        for i in range(g.n):
            p = slice(g.row_ptr[i], g.row_ptr[i + 1])
            rank = _counted_ranks(g, rho, i)[orient]
            ref[g.eid[p][rank < bud[p.stop - p.start]]] = 1
        np.testing.assert_array_equal(_np(keep), ref)
        assert int(nk.item()) == ref.sum()


@pytest.mark.parametrize("d", [8196, 8448, 20_000])
@pytest.mark.parametrize("values", [1, 2, 40])
def test_fp64_long_rows_of_equal_distances(api, d, values):
    """A hub whose distances take a few values, so that a bucket holds thousands of ties, which
    names decide; its neighbours, joined in fours, never choose the hub's edge.  Kept edges
    equal those of ranks counted on the host."""
    announce(f"fp64 ties d={d} values={values}")
    rng = np.random.default_rng(d + values)
    leaf = np.arange(1, d + 1)
    a, b = np.triu_indices(4, 1)
    quad = 1 + 4 * np.arange(d // 4)[:, None]
    g = G.from_edges(d + 1, np.concatenate([np.zeros(d, int), (quad + a).ravel()]),
                     np.concatenate([leaf, (quad + b).ravel()]))
    g = G.relabel(g, rng.permutation(g.n))
    hub = int(np.argmax(np.diff(g.row_ptr)))
    of_hub = (g.edge_u == hub) | (g.edge_v == hub)
    dg = api.DeviceGraph.from_host(g, "cuda")
    for orient in (0, 1):
        rho = np.where(of_hub, 2.0 + rng.integers(0, values, g.m), rng.random(g.m) + (0.0 if orient == 0 else 1000.0))
        if values == 40:
            rho[of_hub & (rng.random(g.m) < 0.3)] = np.nan
        keep, nk = api.sparsify(dg, torch.from_numpy(rho).cuda(), orient, 0.4)
        bud = api.budget_table(g.d_max, 0.4)
        ref = np.zeros(g.m, np.uint8)
        for i in range(g.n):
            p = slice(g.row_ptr[i], g.row_ptr[i + 1])
            ref[g.eid[p][_counted_ranks(g, rho, i)[orient] < bud[p.stop - p.start]]] = 1
        assert ref[of_hub].sum() < d and (orient == 1 or ref[of_hub].sum() > 0)    # the GLOBAL order ranks NaNs first
        np.testing.assert_array_equal(_np(keep), ref)
        assert int(nk.item()) == ref.sum()


# ------------------------------------------------- plan of the short rows --

@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1025, 70_000])
def test_short_row_packing(api, n):
    """Rows packed into waves at the edges of tiles: rows that fill a wave
    exactly, rows closed by long ones, runs of isolated rows, and tiles
    without any short row; the fit over both orders equals the oracle's."""
    announce(f"short rows n={n}")
    rng = np.random.default_rng(n)
    hubs = max(1, n // 40)                             # long rows (above 64 where n allows) between short ones
    u = rng.integers(0, hubs, 6 * n) * 40 % max(1, n)
    v = rng.integers(0, n, 6 * n)
    iso = (np.arange(n) // 64) % 5 == 3                # every fifth tile isolated
    ok = (u != v) & ~iso[u] & ~iso[v]
    key = np.unique(np.minimum(u, v)[ok] * np.int64(n) + np.maximum(u, v)[ok])
    g = G.from_edges(n, key // max(n, 1), key % max(n, 1))
    rho = np.round(rng.random(g.m), 3).astype(np.float32)
    dg = api.DeviceGraph.from_host(g, "cuda")
    if g.m == 0:
        keep, nk = api.sparsify(dg, torch.empty(0, device="cuda"), 0, 0.5)
        assert int(nk.item()) == 0
        return
    t = torch.from_numpy(rho).cuda()
    kl, kg, nk, (el, eg) = api.sparsify_fit_both(dg, t, 0.4)
    for o, (keep, e) in enumerate([(kl, el), (kg, eg)]):
        e_o, keep_o, kept_o = oracle.fit_exponent(g, rho.astype(np.float64), o, 0.4)
        assert e == e_o
        np.testing.assert_array_equal(_np(keep), keep_o)
        assert int(_np(nk)[o]) == kept_o
        # a keep buffer that starts one byte past a 16-byte boundary
        buf = torch.full((g.m + 32,), 7, dtype=torch.uint8, device="cuda")
        k1, n1 = api.sparsify(dg, t, o, e, keep=buf[1:1 + g.m])
        keep_f, kept_f = oracle.sparsify(g, rho.astype(np.float64), o, e)
        np.testing.assert_array_equal(_np(k1), keep_f)
        assert int(n1.item()) == kept_f
        assert int(buf[0]) == 7 and bool((buf[1 + g.m:] == 7).all())


# --------------------------------------------------- selection with binning --

@pytest.mark.parametrize("values", ["f32", "f64", "one-bin", "many-bins"])
def test_binned_rows_of_every_length(api, values):
    """Rows at the bounds of the packed waves, of every sort and of the bucket
    partition; all values of a row in one bin, and rows whose one outlier
    gives them as many bins as their length allows."""
    announce(f"binned rows {values}")
    rng = np.random.default_rng(9)
    degs = [1, 2, 31, 32, 33, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 20_000]
    us, vs = [], []
    leaf = len(degs)
    for q, d in enumerate(degs):
        us.append(np.full(d, q))
        vs.append(np.arange(leaf, leaf + d))
        leaf += d
    chain = np.arange(len(degs), leaf - 1)
    chain = chain[chain % 3 != 0]
    g = G.from_edges(leaf, np.concatenate(us + [chain]), np.concatenate(vs + [chain + 1]))
    rho = rng.random(g.m) + 0.1
    if values == "one-bin":
        rho[:] = 0.7
    elif values == "many-bins":
        rho = 0.5 + 1e-4 * rng.random(g.m)
        for q in range(len(degs)):
            rho[g.eid[g.row_ptr[q]]] = 40.0
    rho = rho if values == "f64" else rho.astype(np.float32)
    dg = api.DeviceGraph.from_host(g, "cuda")
    t = torch.from_numpy(rho).cuda()
    for e in (0.35, 0.8):
        keep, nk, _ = api.sparsify_binned(dg, t, seed=5, e=e)
        keep_o, kept_o = oracle.sparsify_binned(g, rho.astype(np.float64), e, 5)
        np.testing.assert_array_equal(_np(keep), keep_o)
        assert int(nk.item()) == kept_o
    keep, nk, e_fit = api.sparsify_binned(dg, t, seed=6, target=0.4)
    e_o, keep_o, kept_o = oracle.fit_exponent_binned(g, rho.astype(np.float64), 0.4, 6)
    assert e_fit == e_o
    np.testing.assert_array_equal(_np(keep), keep_o)


# ------------------------------------------ selections on the helper streams --

_FORK_DEGS = [64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 20_000]


def _fork_graph():
    """Just above 2^21 stored entries: rows at the bounds of every class, 20 of each, their
    neighbours drawn from one pool (rows of about 18), under random names."""
    rng = np.random.default_rng(21)
    degs = np.repeat(_FORK_DEGS, 20)
    pool = degs.size + np.arange(60_000)
    u = np.repeat(np.arange(degs.size), degs)
    v = np.concatenate([rng.choice(pool, size=d, replace=False) for d in degs])
    g = G.from_edges(degs.size + pool.size, u, v)
    assert 1 << 21 <= 2 * g.m < 1.1 * (1 << 21)
    g.orig_id = rng.permutation(g.n).astype(np.int32)
    return g


@pytest.fixture(scope="module")
def fork_graph():
    return _fork_graph()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("ties", [False, True])
def test_selection_on_helper_streams(api, fork_graph, prec, ties):
    """Every class's launch of the forked dispatch (FP64 rankings stay on one stream), with distinct
    and with tied distances: masks, counts and exponents of the oracle."""
    announce(f"forked selection {prec} ties={ties}")
    g = fork_graph
    rng = np.random.default_rng(5)
    rho = rng.integers(1, 200, g.m) / 64.0 if ties else (1.0 + rng.permutation(g.m)) / (1 << 21)
    rho = rho.astype(np.float32 if prec == "f32" else np.float64)
    ref = rho.astype(np.float64)
    dg = api.DeviceGraph.from_host(g, "cuda")
    t = torch.from_numpy(rho).cuda()
    for orient, e in ((0, 0.45), (1, 0.8)):
        keep, nk = api.sparsify(dg, t, orient, e)
        keep_o, kept_o = oracle.sparsify(g, ref, orient, e)
        np.testing.assert_array_equal(_np(keep), keep_o)
        assert int(nk.item()) == kept_o
    kl, kg, nk, es = api.sparsify_fit_both(dg, t, 0.35)
    for orient, keep in ((0, kl), (1, kg)):
        e_o, keep_o, kept_o = oracle.fit_exponent(g, ref, orient, 0.35)
        assert es[orient] == e_o and int(_np(nk)[orient]) == kept_o
        np.testing.assert_array_equal(_np(keep), keep_o)
    keep, nk, _ = api.sparsify_binned(dg, t, seed=5, e=0.6)
    keep_o, kept_o = oracle.sparsify_binned(g, ref, 0.6, 5)
    np.testing.assert_array_equal(_np(keep), keep_o)
    assert int(nk.item()) == kept_o


# ----------------------------------------------------------------- ingest --

@pytest.mark.parametrize("n", [2, 3, 4, 255, 256, 257, 4096, 4097, 65536, 65537, 1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize("order", [0, 1])
def test_ingest_at_id_widths(api, n, order):
    """Ids that fill their key bits: the largest ids joined to each other, to 0 and
    looped (the largest id's loop has the code of no pair), each pair listed once, twice or 17
    times."""
    announce(f"ingest n={n} order={order}")
    rng = np.random.default_rng(n)
    top = np.arange(max(0, n - 12), n)
    u = np.concatenate([top, np.repeat(top, 17), rng.integers(0, n, 300), top])
    v = np.concatenate([top, np.repeat(top[::-1], 17), rng.integers(0, n, 300), np.zeros(top.size, int)])
    p = rng.permutation(u.size)
    u, v = u[p].astype(np.int32), v[p].astype(np.int32)
    w = rng.lognormal(0.0, 1.0, u.size).astype(np.float32)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for ww in (None, w):
        dg = api.ingest(n, cu(u), cu(v), None if ww is None else cu(ww), by_degree=order == 1)
        row_ptr, col, we, eid, orig, m, dropped = oracle.ingest(n, u, v, ww, order=order)
        assert dg.m == m and dg.n_dropped == dropped
        for got, want in ((dg.row_ptr, row_ptr), (dg.col, col), (dg.eid, eid), (dg.orig_id, orig)):
            np.testing.assert_array_equal(_np(got), want)
        if ww is not None:
            np.testing.assert_array_equal(_np(dg.w), we)


@pytest.mark.parametrize("off", [1, 2, 3])
@pytest.mark.parametrize("m", [500, 70_000])
def test_inputs_off_their_vector_alignment(api, off, m):
    """Edge lists, weights and scores that start `off` elements into an allocation: sorted where
    they are, equal to the oracle's."""
    announce(f"inputs off={off} m={m}")
    rng = np.random.default_rng(off)
    n = 700

    def view(a):
        buf = torch.zeros(a.size + 8, dtype=torch.from_numpy(a).dtype, device="cuda")
        buf[off:off + a.size] = torch.from_numpy(a).cuda()
        t = buf[off:off + a.size]
        assert t.is_contiguous() and t.data_ptr() % 16 == off * a.itemsize % 16
        return t

    u, v = (rng.integers(0, n, m).astype(np.int32) for _ in range(2))
    w = rng.lognormal(0.0, 1.0, m).astype(np.float32)
    for order in (0, 1):
        dg = api.ingest(n, view(u), view(v), view(w), by_degree=order == 1)
        row_ptr, col, we, eid, orig, m_o, dropped = oracle.ingest(n, u, v, w, order=order)
        assert dg.m == m_o
        np.testing.assert_array_equal(_np(dg.row_ptr), row_ptr)
        np.testing.assert_array_equal(_np(dg.col), col)
        np.testing.assert_array_equal(_np(dg.w), we)
    x, y = rng.integers(0, 50, m).astype(np.float64), rng.random(m)
    assert api.spearman(view(x), view(y)) == api.spearman(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())


# ---------------------------------------------------------------- adjoint --

@pytest.mark.parametrize("R", [1, 2, 4, 6, 8, 12, 24, 33, 64])
@pytest.mark.parametrize("kind", ["rows", "sparse"])
def test_adjoint_rows_of_every_kind(api, R, kind):
    """The reverse step's vector widths and lanes per row, on rows of one chunk, of
    several and of a workgroup (the two hubs, 300 and 700 entries), and
    isolated vertices.  Bounds: those of the adjoint tests on grids, which are k
    FP32 roundings on the scale of the largest gradients."""
    announce(f"adjoint {kind} R={R}")
    rng = np.random.default_rng(7)
    n, k = 1500, 6
    if kind == "rows":
        us, vs = [np.arange(n - 3)], [np.arange(1, n - 2)]
        for h, d in ((3, 300), (700, 700), (11, 64), (12, 65), (13, 40), (14, 17)):
            us.append(np.full(d, h))
            vs.append(rng.choice(np.setdiff1d(np.arange(n - 3), [h - 1, h, h + 1]), size=d, replace=False))
        u, v = np.concatenate(us), np.concatenate(vs)
        key = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
        g = G.from_edges(n, key // n, key % n)
    else:
        g = G.from_edges(n, np.arange(0, n - 2, 2), np.arange(1, n - 1, 2))
        g = G.from_edges(n, np.concatenate([g.edge_u, np.arange(0, n - 4, 4)]),
                         np.concatenate([g.edge_v, np.arange(2, n - 2, 4)]))
    g = G.with_weights(g, rng.uniform(0.5, 2.0, g.m).astype(np.float32))
    c = rng.normal(size=g.m)
    dg = api.DeviceGraph.from_host(g, "cuda")
    w = torch.from_numpy(g.edge_w.astype(np.float32)).cuda().requires_grad_(True)
    rho = api.AlgDist.apply(w, dg, R, k, 0.5, 3, 4)
    (torch.from_numpy(c.astype(np.float32)).cuda() * rho).sum().backward()
    got = _np(w.grad).astype(np.float64)
    want = oracle.grad_weights(g, c, R, k, 0.5, x0=oracle.start_vectors(g.n, R, 3, 0, g.orig_id))
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    per = np.abs(got - want) / (np.abs(want) + 1e-3 * np.abs(want).max())
    print(f"rel L2 {err:.3e}  max per-edge {per.max():.3e}")
    assert err <= 1e-4
    assert per.max() <= 1e-3


@pytest.mark.parametrize("n", [262_144, 262_145, 600_001])
def test_adjoint_of_more_rows_than_lanes_in_flight(api, n):
    """R = 33 takes 64 lanes a row: from 262,145 rows on, a workgroup of the reverse step handles
    several blocks of rows.  Bounds as above."""
    announce(f"adjoint n={n}")
    rng = np.random.default_rng(n)
    R, k = 33, 3
    hub = rng.choice(np.arange(3, n), size=700, replace=False)
    u, v = np.concatenate([np.arange(n - 1), np.full(700, 1)]), np.concatenate([np.arange(1, n), hub])
    g = G.from_edges(n, u, v)
    g = G.with_weights(g, rng.uniform(0.5, 2.0, g.m).astype(np.float32))
    c = rng.normal(size=g.m)
    dg = api.DeviceGraph.from_host(g, "cuda")
    w = torch.from_numpy(g.edge_w.astype(np.float32)).cuda().requires_grad_(True)
    rho = api.AlgDist.apply(w, dg, R, k, 0.5, 3, 2)
    (torch.from_numpy(c.astype(np.float32)).cuda() * rho).sum().backward()
    got = _np(w.grad).astype(np.float64)
    want = oracle.grad_weights(g, c, R, k, 0.5, x0=oracle.start_vectors(g.n, R, 3, 0, g.orig_id))
    per = np.abs(got - want) / (np.abs(want) + 1e-3 * np.abs(want).max())
    print(f"rel L2 {np.linalg.norm(got - want) / np.linalg.norm(want):.3e}  max per-edge {per.max():.3e}")
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
    assert per.max() <= 1e-3


# ------------------------------------------- launch plans and set-up passes --

@pytest.mark.parametrize("n", [3, 64, 65, 1024, 1025, 2048, 2049, 32_768, 32_769, 262_144, 262_145])
@pytest.mark.parametrize("R", [2, 7])
def test_plans_at_their_sizes(api, n, R):
    """Graphs at the tile counts where the launch plan, its single workgroup, the
    min / max split and the two plan forms change over; rows of a workgroup (300
    and 600 entries; the last vertex is one) where they fit, and hub
    bounds that make every row one.  FP64 storage: the values are the oracle's up
    to the summation order of a row (600 terms of 1.1e-16) over 3 sweeps."""
    announce(f"plans n={n} R={R}")
    rng = np.random.default_rng(n)
    us, vs = [np.arange(n - 1)], [np.arange(1, n)]
    if n > 1000:
        for h, d in ((n - 1, 600), (7, 300), (n // 2, 600)):
            us.append(np.full(d, h))
            vs.append(rng.choice(n, size=d, replace=False))
    u, v = np.concatenate(us), np.concatenate(vs)
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique((lo * n + hi)[lo != hi])
    g = G.from_edges(n, key // n, key % n)
    dg = api.DeviceGraph.from_host(g, "cuda")
    want = oracle.algebraic_distance(g, R, 3, 0.5, seed=4)
    for hub in (0, 1):
        res = api.relax(dg, R, 3, omega=0.5, seed=4, store="f64", hub_degree=hub)
        rho = _np(api.edge_dist(dg, res.x, res.minmax))
        np.testing.assert_allclose(rho, want, rtol=1e-11, atol=1e-12)


@pytest.mark.parametrize("n", [(1 << 20) - 63, 1 << 20, (1 << 20) + 1])
def test_plans_of_a_thousand_workgroups(api, n):
    """The plan's two-launch form up to the last workgroup whose predecessors' sums are one per
    thread, and the general form after it; long rows at both ends.  Tolerance as above."""
    announce(f"plans n={n}")
    rng = np.random.default_rng(n)
    us, vs = [np.arange(n - 1)], [np.arange(1, n)]
    for h, d in ((n - 1, 600), (7, 300), (n // 2, 5000)):
        us.append(np.full(d, h))
        vs.append(rng.choice(n, size=d, replace=False))
    u, v = np.concatenate(us), np.concatenate(vs)
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique((lo * n + hi)[lo != hi])
    g = G.from_edges(n, key // n, key % n)
    dg = api.DeviceGraph.from_host(g, "cuda")
    want = oracle.algebraic_distance(g, 2, 3, 0.5, seed=4)
    for hub in (0, 1):
        res = api.relax(dg, 2, 3, omega=0.5, seed=4, store="f64", hub_degree=hub)
        rho = _np(api.edge_dist(dg, res.x, res.minmax))
        np.testing.assert_allclose(rho, want, rtol=1e-11, atol=1e-12)


# ------------------------------------------------------ centring of components --

@pytest.mark.parametrize("chunks", [1, 2047, 2048, 2049])
@pytest.mark.parametrize("R", [3, 16])
def test_centring_at_chunk_counts(api, chunks, R):
    """One component of so many chunks (256 members each) and as many components of one, around
    the count where a chunk goes from several waves to one.  FP64 storage: the
    oracle's values up to the summation order of a mean, as for the plans."""
    announce(f"centring chunks={chunks} R={R}")
    for kind in ("one", "each"):
        n = 256 * chunks - 3 if kind == "one" else 3 * chunks
        u, v = np.arange(n - 1), np.arange(1, n)
        if kind == "each":
            u, v = u[v % 3 != 0], v[v % 3 != 0]
        g = G.from_edges(n, u, v)
        dg = api.DeviceGraph.from_host(g, "cuda")
        c = dg.components()
        assert (c.n_comp, c.n_chunks) == ((1, chunks) if kind == "one" else (chunks, chunks))
        res = api.relax(dg, R, 3, omega=0.5, seed=4, store="f64")
        rho = _np(api.edge_dist(dg, res.x, res.minmax))
        np.testing.assert_allclose(rho, oracle.algebraic_distance(g, R, 3, 0.5, seed=4), rtol=1e-11, atol=1e-12)


@pytest.mark.parametrize("store", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("R", [6, 16])
def test_centring_sums_of_either_layout(api, store, R):
    """Small components relax to the same bits beside a component of a thousand chunks
    (whose sums lie by vector) and without it (by chunk)."""
    announce(f"centring layouts {store} R={R}")
    small = np.arange(0, 900)
    u, v = small[:-1][small[1:] % 3 != 0], small[1:][small[1:] % 3 != 0]
    long_ = np.arange(900, 900 + 256 * 1000)
    both = G.from_edges(long_[-1] + 1, np.concatenate([u, long_[:-1]]), np.concatenate([v, long_[1:]]))
    out = []
    for g in (G.from_edges(900, u, v), both):
        dg = api.DeviceGraph.from_host(g, "cuda")
        c = dg.components()
        assert c.n_comp == (300 if g.n == 900 else 301) and c.n_chunks == (300 if g.n == 900 else 1300)
        kw = dict(fp32_tail=3, fp64_tail=1) if store == "bf16" else {}
        res = api.relax(dg, R, 12, omega=0.5, seed=9, store=store, **kw)
        out.append((_np(res.x)[:900], _np(res.shift)[_np(c.comp_of)[:900]]))
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])


# ------------------------------------------------------------ retention fit --

@pytest.mark.parametrize("target", [1e-9, 0.34, 0.999999, 1.0])
@pytest.mark.parametrize("kind", ["edge", "three", "star", "cycle", "equal"])
def test_fit_at_extreme_ranks(api, kind, target):
    """The select's digits at the first and the last rank, on graphs whose threshold
    indices are all equal, all distinct or one number apart.  Exponents and
    masks equal the oracle's."""
    announce(f"fit {kind} target={target}")
    rng = np.random.default_rng(2)
    if kind == "edge":
        g = G.from_edges(2, np.array([0]), np.array([1]))
    elif kind == "three":
        g = G.from_edges(5, np.array([0, 0, 2]), np.array([1, 2, 4]))
    elif kind == "star":
        g = G.from_edges(5000, np.zeros(4999, int), np.arange(1, 5000))
    elif kind == "cycle":
        g = G.from_edges(3000, np.arange(3000), np.roll(np.arange(3000), -1))
    else:
        g = G.chung_lu(800, 9000, seed=6)
    rho = np.full(g.m, 0.5, np.float32) if kind == "equal" else rng.uniform(0.1, 1.0, g.m).astype(np.float32)
    dg = api.DeviceGraph.from_host(g, "cuda")
    for o in (0, 1):
        keep, n_kept, e = api.sparsify_fit(dg, torch.from_numpy(rho).cuda(), o, target)
        e_o, keep_o, kept_o = oracle.fit_exponent(g, rho.astype(np.float64), o, target)
        assert e == e_o and int(_np(n_kept)[0]) == kept_o
        np.testing.assert_array_equal(_np(keep), keep_o)


def test_fit_stages_flushed_between_steps(api):
    """2^24 edges of which the select's first digit and the exact check list whole steps of the
    same workgroups (isolated edges, kept at every e, in 64 of every 2,048 blocks of 1,024 edges;
    K_{128,128} elsewhere), so that the staged appends are flushed inside the loops while
    the lists stay complete.  The smallest exponent is 0 with one edge a vertex; others are
    checked against the selection at the exponent and one grid step (2^-40) below it."""
    announce("fit stages")
    P, d = 8, 128
    per_n = 2 * 65_536 + 124 * 2 * d
    a = torch.arange(65_536, device="cuda")
    left = torch.arange(d, device="cuda").repeat_interleave(d)
    right = d + torch.arange(d, device="cuda").repeat(d)
    base = 2 * 65_536 + 2 * d * torch.arange(124, device="cuda")
    u1 = torch.cat([2 * a, (base[:, None] + left).reshape(-1)])
    v1 = torch.cat([2 * a + 1, (base[:, None] + right).reshape(-1)])
    off = per_n * torch.arange(P, device="cuda")[:, None]
    u, v = (off + u1).reshape(-1), (off + v1).reshape(-1)              # ascending: the edge ids
    n, m = P * per_n, u.numel()
    assert m == 1 << 24
    e = torch.arange(m, device="cuda", dtype=torch.int32)
    src, dst = torch.cat([u, v]), torch.cat([v, u])
    o = torch.argsort(src * n + dst)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    dg = api.DeviceGraph.from_tensors(dict(n=n, m=m, d_max=d, row_ptr=row_ptr, col=dst[o].to(torch.int32), w=None,
                                           eid=torch.cat([e, e])[o], orig_id=torch.arange(n, device="cuda", dtype=torch.int32)))
    gen = torch.Generator(device="cuda").manual_seed(3)
    rho = torch.randperm(m, generator=gen, device="cuda").float()       # distinct
    for target in (0.01, 0.045, 0.3):
        kl, kg, nk, es = api.sparsify_fit_both(dg, rho, target)
        K = int(np.ceil(target * m))
        for orient, keep, e_fit, kept in ((0, kl, es[0], int(nk[0])), (1, kg, es[1], int(nk[1]))):
            want, n_want = api.sparsify(dg, rho, orient, e_fit)
            assert torch.equal(keep, want) and kept == int(n_want) == int(keep.sum(dtype=torch.int64))
            assert kept >= K
            if target == 0.01:
                assert e_fit == 0.0
                best = torch.full((n,), np.inf, device="cuda").scatter_reduce(
                    0, src, torch.cat([rho, rho]) * (1 if orient == 0 else -1), "amin")
                r = rho * (1 if orient == 0 else -1)
                assert torch.equal(keep.bool(), (r == best[u]) | (r == best[v]))
            else:
                assert int(api.sparsify(dg, rho, orient, e_fit - 2.0 ** -40)[1]) < K


# --------------------------------------------------- merging and coarsening --

@pytest.mark.parametrize("spread", [1.0, 1e30])
def test_merged_runs_across_waves(api, spread):
    """Runs of 1 to 40 listed copies of a pair, so that runs of every length up to and past
    the short ones start at every lane and cross waves and workgroups; with the large
    spread most sums need the exact digits.  Weights equal the oracle's."""
    announce(f"merged runs spread={spread}")
    rng = np.random.default_rng(3)
    lens = np.concatenate([np.arange(1, 41), rng.integers(1, 41, 4000)])
    n = 3000
    key = np.sort(rng.choice(n * n, size=3 * lens.size, replace=False))
    key = key[key // n < key % n][:lens.size]
    u, v = np.repeat(key // n, lens[:key.size]), np.repeat(key % n, lens[:key.size])
    w = np.exp(rng.uniform(-np.log(spread), np.log(spread), u.size) + rng.normal(size=u.size)).astype(np.float32)
    p = rng.permutation(u.size)
    u, v, w = u[p].astype(np.int32), v[p].astype(np.int32), w[p]
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dg = api.ingest(n, cu(u), cu(v), cu(w), by_degree=False)
    row_ptr, col, we, eid, orig, m, dropped = oracle.ingest(n, u, v, w, order=0)
    assert dg.m == m
    np.testing.assert_array_equal(_np(dg.col), col)
    np.testing.assert_array_equal(_np(dg.w), we)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("edge", [15, 63, 255, 2047])
def test_coarsening_at_row_classes(api, edge, prec):
    """Rows of edge .. edge + 3 entries around the lengths where a row goes from
    one step to several, from 16 lanes to a wave and from a wave to a workgroup,
    with distances in steps so that ties occur.  Seeds and aggregates equal the oracle's."""
    announce(f"coarsening rows of {edge} {prec}")
    rng = np.random.default_rng(edge)
    n = max(400, 2 * edge)
    us, vs = [np.arange(8, n - 1)], [np.arange(9, n)]
    for h, d in enumerate((edge, edge + 1, edge + 2, edge + 3)):
        us.append(np.full(d, h))
        vs.append(rng.choice(np.arange(8, n), size=d, replace=False))
    u, v = np.concatenate(us), np.concatenate(vs)
    g = G.relabel(G.from_edges(n, u, v), rng.permutation(n)) if edge == 63 else G.from_edges(n, u, v)
    rho = rng.integers(1, 40, g.m) / 64.0
    rho = rho.astype(np.float32 if prec == "f32" else np.float64)
    dg = api.DeviceGraph.from_host(g, "cuda")
    for theta in (0.3, 0.9):
        agg, is_seed, nc = api.ml_aggregate(dg, torch.from_numpy(rho).cuda(), 1e-12, theta)
        seeds_o = oracle.ml_seeds(g, rho.astype(np.float64), 1e-12, theta)
        agg_o, nc_o = oracle.ml_aggregates(g, rho.astype(np.float64), seeds_o, 1e-12)
        assert nc == nc_o
        np.testing.assert_array_equal(_np(is_seed), seeds_o)
        np.testing.assert_array_equal(_np(agg), agg_o)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("d", [5, 40, 200, 700, 3000])
def test_coarsening_passes_over_nan_distances(api, d, prec):
    """Rows of one step, of several, of a wave and of a workgroup with distances that
    are NaN, infinite and tied: a vertex joins the seed neighbour of largest strength
    among those that compare (NaN compares with nothing), ties by the smaller name.  Seeds equal the oracle's,
    aggregates the rule's."""
    announce(f"coarsening nan rows of {d} {prec}")
    rng = np.random.default_rng(d)
    n = 4 * d + 200
    us, vs = [np.arange(8, n - 1)], [np.arange(9, n)]
    for h in range(8):
        us.append(np.full(d, h))
        vs.append(rng.choice(np.arange(8, n), size=d, replace=False))
    g = G.from_edges(n, np.concatenate(us), np.concatenate(vs))
    g = G.relabel(g, rng.permutation(n))
    rho = rng.integers(1, 6, g.m) / 8.0
    pick = rng.integers(0, 4, g.m)
    rho[pick == 0] = np.nan
    rho[pick == 1] = np.inf
    rho = rho.astype(np.float32 if prec == "f32" else np.float64)
    agg, is_seed, nc = api.ml_aggregate(api.DeviceGraph.from_host(g, "cuda"), torch.from_numpy(rho).cuda(), 1e-12, 0.5)
    seeds = oracle.ml_seeds(g, rho.astype(np.float64), 1e-12, 0.5)
    np.testing.assert_array_equal(_np(is_seed), seeds)
    rank = np.cumsum(seeds) - 1
    want = np.where(seeds == 1, rank, -1)
    r = rho.astype(np.float64)
    delta = 1.0 / np.sqrt(r * r + 1e-12)
    for i in np.nonzero(seeds == 0)[0]:
        p = np.arange(g.row_ptr[i], g.row_ptr[i + 1])
        p = p[(seeds[g.col[p]] == 1) & ~np.isnan(delta[g.eid[p]])]
        if p.size:
            want[i] = rank[g.col[p][np.lexsort((g.orig_id[g.col[p]], -delta[g.eid[p]]))[0]]]
    assert nc == seeds.sum()
    np.testing.assert_array_equal(_np(agg), want)


@pytest.mark.parametrize("d_max", [(1 << 21) - 1, 1 << 21])
def test_fit_side_records_of_both_widths(api, d_max):
    """The largest degree (a bound: tables are sized by it) picks 64-bit or 128-bit side
    records and puts the fit's log tables in memory; fits of either give the masks,
    counts and exponents of the exact bound, on rows of every class."""
    import dataclasses
    announce(f"fit d_max={d_max}")
    g = G.chung_lu(4000, 120_000, seed=31)
    rho = np.random.default_rng(8).integers(1, 4000, g.m).astype(np.float32)      # with ties
    dg = api.DeviceGraph.from_host(g, "cuda")
    wide = dataclasses.replace(dg, d_max=d_max)
    rt = torch.from_numpy(rho).cuda()
    for target in (0.05, 0.4):
        kl, kg, nk, (el, eg) = api.sparsify_fit_both(wide, rt, target)
        for o, keep, e in ((0, kl, el), (1, kg, eg)):
            keep1, n1, e1 = api.sparsify_fit(dg, rt, o, target)
            keep2, n2, e2 = api.sparsify_fit(wide, rt, o, target)
            assert e == e1 == e2
            assert int(_np(nk)[o]) == int(_np(n1)[0]) == int(_np(n2)[0])
            np.testing.assert_array_equal(_np(keep), _np(keep1))
            np.testing.assert_array_equal(_np(keep2), _np(keep1))


# ---------------------------------------------------------------- comparison --

@pytest.mark.parametrize("n", [3, 100, 4097, 70_001])
def test_degree_ranks_by_their_leading_bits(api, n):
    """ad_compare_properties ranks degrees by the bits a whole number up to 2m can
    have: the correlation equals that of the same degrees as general scores (the
    same ranks; the mean's partial sums too), from isolated vertices to the hub
    whose row is every other vertex."""
    announce(f"degree ranks n={n}")
    rng = np.random.default_rng(n)
    u = np.concatenate([np.zeros(n - 1, int), rng.integers(1, n, 2 * n)])
    v = np.concatenate([np.arange(1, n), rng.integers(1, n, 2 * n)])
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique((lo * n + hi)[lo != hi])
    g = G.from_edges(n, key // n, key % n)
    keep = (rng.random(g.m) < 0.4).astype(np.uint8)
    cmp = api.compare_properties(api.DeviceGraph.from_host(g, "cuda"), torch.from_numpy(keep).cuda())
    rp = oracle.subgraph(g, keep)[0]
    deg = lambda p: torch.from_numpy(np.diff(p).astype(np.float64)).cuda()
    got = [x for k, x in cmp.items() if "degree" in k and "spearman" in k]
    assert got == [api.spearman(deg(g.row_ptr), deg(rp))]
