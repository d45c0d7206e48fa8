"""Run in a subprocess by test_launches_cpu.py: calls entry points of libad.so on the runtime of
fake_hip.c (no device, no kernel runs) with made-up device addresses, and prints one
JSON line per call: its status and what it enqueued.

    fake_launches.py SHIM LIBRARY '[{"call": ..., ...}, ...]'
"""
import ctypes
import json
import os
import sys

shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.fake_log.restype = ctypes.c_char_p
shim.fake_reset.argtypes = [ctypes.c_long]
lib = ctypes.CDLL(sys.argv[2])
P, I32, I64, U64, F64, SZ = (ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_uint64, ctypes.c_double,
                             ctypes.c_size_t)
STREAM = 7
_next = 1 << 44


def dev(nbytes=1 << 40):
    """An address that nothing reads."""
    global _next
    _next += (nbytes + 4095) // 4096 * 4096
    return _next - (nbytes + 4095) // 4096 * 4096


class Graph(ctypes.Structure):
    _fields_ = [("n", I64), ("m", I64), ("row_ptr", P), ("col", P), ("w", P), ("eid", P), ("orig_id", P),
                ("d_max", I32), ("col_orig", P)]


class Comp(ctypes.Structure):
    _fields_ = [("n_comp", I64), ("n_chunks", I64), ("comp_of", P), ("members", P), ("comp_start", P),
                ("chunk_start", P)]


class Relax(ctypes.Structure):
    _fields_ = [("R", I32), ("k", I32), ("omega", F64), ("seed", U64), ("graph_id", U64), ("store", ctypes.c_int),
                ("fp32_tail", I32), ("ckpt_every", I32), ("rows_per_wave", I32), ("hub_degree", I32),
                ("fp64_tail", I32), ("comp", ctypes.POINTER(Comp))]


def graph(c):
    return Graph(c["n"], c["m"], dev(), dev(), dev(), dev(), dev(), c["d_max"], dev())


def size(f, *args):
    fn = getattr(lib, f)
    fn.restype = SZ
    return fn(*args)


def sparsify(c):
    g = graph(c)
    ws = size("ad_sparsify_workspace_size", ctypes.byref(g))
    return lib.ad_sparsify(ctypes.byref(g), c["dtype"], P(dev()), 0, P(dev()), P(dev()), P(dev()), P(dev()), SZ(ws),
                           P(STREAM))


def binned(c):
    g = graph(c)
    ws = size("ad_sparsify_binned_workspace_size", ctypes.byref(g))
    e = F64(0)
    return lib.ad_sparsify_binned(ctypes.byref(g), c["dtype"], P(dev()), U64(1), U64(0), F64(0.5), F64(0.0), P(dev()),
                                  P(dev()), ctypes.byref(e), P(dev()), SZ(ws), P(STREAM))


def relax_opts(c):
    comp = Comp(c["n_comp"], c["n_chunks"], dev(), dev(), dev(), dev())
    o = Relax(c["R"], c["k"], 0.5, 1, 0, c["store"], 2, c.get("ckpt", 0), 0, 0, 0, ctypes.pointer(comp))
    o._comp = comp
    return o


def relax(c):
    g, o = graph(c), relax_opts(c)
    ws = size("ad_relax_workspace_size", ctypes.byref(g), ctypes.byref(o))
    return lib.ad_relax(ctypes.byref(g), ctypes.byref(o), None, P(dev()), P(dev()), P(dev()), P(dev()), P(dev()),
                        SZ(ws), P(STREAM))


def backward(c):
    g, o = graph(c), relax_opts(c)
    ws = size("ad_relax_backward_workspace_size", ctypes.byref(g), ctypes.byref(o))
    return lib.ad_relax_backward(ctypes.byref(g), ctypes.byref(o), P(dev()), P(dev()), P(dev()), P(dev()), P(dev()),
                                 P(dev()), P(dev()), SZ(ws), P(STREAM))


def dist_noalloc(c):
    return lib.ad_edge_dist_noalloc(ctypes.byref(graph(c)), 16, 1, P(dev()), P(dev()), 1, P(dev()), P(STREAM))


def dist(c):
    g = graph(c)
    ws = size("ad_edge_dist_workspace_size", ctypes.byref(g)) - c.get("short", 0)
    return lib.ad_edge_dist(ctypes.byref(g), 16, 1, P(dev()), P(dev()), 1, P(dev()), P(dev()), SZ(ws), P(STREAM))


for c in json.loads(sys.argv[3]):
    shim.fake_reset(c.get("fail_at", -1))
    status = globals()[c["call"]](c)
    log = [l.split() for l in shim.fake_log().decode().splitlines()]
    print(json.dumps(dict(status=status, log=log, pending=shim.fake_pending_error())), flush=True)
os._exit(0)
