"""What calls enqueue, looked at without a device (fake_hip.c): the helper streams of a
selection whose launch fails, and launch shapes at sizes beyond any test's memory."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1601_05527_amd", "libad.so")
STREAM = "7"


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None or not os.path.exists(LIB):
        pytest.skip("needs a C compiler and the built library")
    shim = str(tmp_path_factory.mktemp("hip") / "libfake_hip.so")
    subprocess.run([cc, "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.c"), "-o", shim], check=True)

    def call(*calls):
        r = subprocess.run([sys.executable, os.path.join(HERE, "fake_launches.py"), shim, LIB, json.dumps(calls)],
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        return [json.loads(line) for line in r.stdout.splitlines()]

    return call


def _unjoined(log):
    """Streams with work of this call that the caller's stream does not wait for at its end."""
    last, event_of, joined = {}, {}, {}
    for at, (what, *a) in enumerate(log):
        if what == "launch":
            last[a[0]] = at
        elif what == "wait" and a[0] != STREAM:
            last[a[0]] = at
        elif what == "record":
            event_of[a[1]] = (a[0], at)
        elif what == "wait" and a[1] in event_of:
            joined[event_of[a[1]][0]] = event_of[a[1]][1]
    return [s for s, at in last.items() if s != STREAM and joined.get(s, -1) < at]


@pytest.mark.parametrize("call,dtype", [("sparsify", 1), ("binned", 1), ("binned", 0)])
def test_helper_streams_joined_when_a_launch_fails(run, call, dtype):
    """Whichever launch of a selection on helper streams fails, the caller's stream waits for what
    the helper streams were given before the call returns its error."""
    c = dict(call=call, dtype=dtype, n=1 << 20, m=1 << 24, d_max=20_000)
    whole = run(c)[0]
    assert whole["status"] == 0 and not _unjoined(whole["log"])
    n = sum(x[0] == "launch" for x in whole["log"])
    assert n > 10 and len({x[1] for x in whole["log"] if x[0] == "launch"}) == 4
    for at, r in enumerate(run(*[dict(c, fail_at=k) for k in range(1, n + 1)]), 1):
        assert r["status"] != 0, at
        assert not _unjoined(r["log"]), (at, r["log"])
        assert r["pending"] == 0, at


def _check_shapes(r):
    """The runtime takes fewer than 2^32 threads per grid dimension, and none empty."""
    assert r["status"] == 0
    for x in r["log"]:
        if x[0] == "launch":
            g = [int(v) for v in x[3:9]]
            assert all(0 < g[i] * g[i + 3] < 1 << 32 for i in range(3)), x


@pytest.mark.parametrize("store", [0, 1, 2])
@pytest.mark.parametrize("R", [16, 20, 64])
def test_relaxation_of_many_components_launches(run, store, R):
    n_comp = 1 << 24                      # of two vertices each
    _check_shapes(run(dict(call="relax", n=2 * n_comp, m=1 << 28, d_max=5000, R=R, k=3, store=store, n_comp=n_comp,
                           n_chunks=n_comp))[0])


@pytest.mark.parametrize("n,m,R", [(1 << 27, 1 << 30, 16), ((1 << 26) + 5, 1 << 26, 33), ((1 << 26) + 5, 1 << 20, 63),
                                   (1 << 30, 1 << 30, 8)])
def test_gradient_of_many_rows_launches(run, n, m, R):
    _check_shapes(run(dict(call="backward", n=n, m=m, d_max=5000, R=R, k=4, store=1, ckpt=2, n_comp=1,
                           n_chunks=n // 256 + 1))[0])


def test_long_rows_take_no_room_from_the_fixed_scratch(run):
    """The largest graph that the allocation-free distances accept does not depend on its edges,
    and a graph at that bound goes without the list of its long rows' items."""
    def most(m, d_max):
        lo, hi = 1 << 20, 1 << 23                     # accepted, refused
        while lo + 1 < hi:
            cut = sorted({lo + (hi - lo) * k // 65 for k in range(1, 65)} - {lo, hi})
            got = [r["status"] == 0 for r in run(*[dict(call="dist_noalloc", n=n, m=m, d_max=d_max) for n in cut])]
            assert got == sorted(got, reverse=True)
            k = sum(got)
            lo, hi = (cut[k - 1] if k else lo), (cut[k] if k < len(cut) else hi)
        return lo

    n = most(10, 3)
    assert n > 2_400_000 and most(1 << 22, 5000) == n
    few, many = run(*[dict(call="dist_noalloc", n=k, m=1 << 22, d_max=5000) for k in (n, n // 2)])
    assert few["status"] == many["status"] == 0
    assert [any("k_hub_first" in x[2] for x in r["log"]) for r in (few, many)] == [False, True]
    _check_shapes(few)


def test_distances_without_room_for_the_list(run):
    """A workspace that holds the plan alone still serves; a shorter one is refused."""
    c = dict(call="dist", n=300_000, m=1 << 21, d_max=9000)
    rows = min(300_000, (1 << 22) // 513)
    room = (4 * (rows + 1) + 255) // 256 * 256
    whole, plan, short = run(c, dict(c, short=room), dict(c, short=room + 1))
    assert whole["status"] == plan["status"] == 0 and short["status"] == 3
