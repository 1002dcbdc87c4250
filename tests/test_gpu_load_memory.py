"""Device memory.  A load: a graph fits where its own arrays fit, without the
load's temporaries beside them; in memory for one of two graphs, each loads
over the other.  An update call that runs out: the handle holds what it held,
and goes on.  The library's hipMalloc goes through a counter with a cap, in a
process of its own."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))

HEAD = r"""
import ctypes, os, sys
import numpy as np
import torch
assert torch.cuda.is_available()
torch.zeros(1, device="cuda:0")
hip = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64.so" in l)
cap = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
for f in ("cap_held", "cap_peak"):
    getattr(cap, f).restype = ctypes.c_size_t
cap.cap_set.argtypes = [ctypes.c_size_t]
assert cap.cap_init(hip.encode()) == 0
import graphgen
import paper_1612_09368_amd as cm

def graph(n, m):
    s, d = graphgen.er_graph(n, m, graphgen.rng_for("load-memory", n))
    return n, torch.from_numpy(s).to("cuda:0"), torch.from_numpy(d).to("cuda:0"), keys(s, d)

def keys(s, d):
    return np.sort(np.minimum(s, d).astype(np.int64) << 32 | np.maximum(s, d))

NONE = 2 ** 64 - 1

def load(g, gr, most=NONE):
    # (no decomposition: cooperative launches belong to the process that runs the tests)
    cap.cap_set(most)
    try:
        g.load(*gr[:3])
    finally:
        cap.cap_set(NONE)
    held = cap.cap_held()
    assert np.array_equal(keys(*g.export_edges()), gr[3])
    assert cap.cap_held() == held <= most
"""

LOAD = HEAD + r"""
# 2 m a power of two: the duplicate test's hash is as small as it gets
big, small = graph(1 << 14, 1 << 18), graph(1 << 13, 1 << 15)
held = {}
for gr in (big, small):
    base = cap.cap_held()
    with cm.Graph() as g:
        load(g, gr)
        held[gr[0]] = cap.cap_held() - base
    assert held[gr[0]] > 0 and cap.cap_held() == base
print("held", held, flush=True)
base = cap.cap_held()
with cm.Graph() as g:
    for gr in (big, big, small, big, small, small, big):
        load(g, gr, base + held[big[0]])
        print("loaded", gr[0], cap.cap_held() - base, flush=True)
assert cap.cap_held() == base
# with less than its arrays need a load is refused, and the handle goes on
half = base + held[big[0]] // 2
with cm.Graph() as g:
    load(g, small, half)
    try:
        load(g, big, half)
        raise SystemExit("too large a graph was accepted")
    except cm.CoreMaintError as e:
        assert e.status == cm.E_NOMEM, e
    load(g, small, half)
assert cap.cap_held() == base
print("load memory: ok", flush=True)
"""

# A handle restored from a snapshot takes validation and reservation without a
# cooperative launch: batches of over 1,024 edges, up to the point where they
# would run.
UPDATE = HEAD + r"""
def state(g):
    return keys(*g.export_edges()), g.cores(), g.superior_degrees()

def same(x, y):
    return all(np.array_equal(a, b) for a, b in zip(x, y))

base = cap.cap_held()
with cm.Graph.restore(sys.argv[2]) as g:
    n, _ = g.num_vertices()
    before = state(g)
    s, d = g.export_edges()
    present = before[0]
    rng = np.random.RandomState(3)

    def refused(call, most, code, a, b):
        held = cap.cap_held()
        cap.cap_set(held + most)
        st, stats = call(a, b, check=False)
        cap.cap_set(NONE)
        assert st == code and stats.applied == 0, (st, code)
        assert same(before, state(g))
        return cap.cap_held() - held

    def missing(k, hub):
        u = np.full(4 * k, hub) if hub >= 0 else rng.randint(0, n, 4 * k)
        v = rng.randint(0, n, 4 * k)
        x = np.unique((np.minimum(u, v).astype(np.int64) << 32 | np.maximum(u, v))[u != v])
        x = rng.permutation(x[~np.isin(x, present)])[:k]
        return (x >> 32).astype(np.int32), (x & 0xffffffff).astype(np.int32)

    # 1: the batch arrays do not fit (a deletion of edges that are there)
    k = s.size
    assert refused(g.delete_edges, 8 * k, cm.E_NOMEM, s, d) <= 8 * k
    # ... a smaller batch gets arrays of its size, and is looked at: the last edge is missing
    a, b = missing(1, 5)
    x, y = np.append(s[:3000], a), np.append(d[:3000], b)
    refused(g.delete_edges, NONE >> 1, cm.E_MISSING, x, y)
    # 2: the pool is full and a larger one does not fit; every list grows past its slots
    u, v = missing(min(n * 12, 60000), -1)
    x, y = np.append(u, s[0]), np.append(v, d[0])
    refused(g.insert_edges, NONE >> 1, cm.E_EXISTS, x, y)  # (room for the batch arrays)
    # nothing, the scan's arrays, the lists' array, one of the two beside it
    for most in range(0, 3250001, 250000):
        assert refused(g.insert_edges, most, cm.E_NOMEM, u, v) == 0, most
        print("refused with", most, flush=True)
    refused(g.insert_edges, NONE >> 1, cm.E_EXISTS, x, y)
assert cap.cap_held() == base
print("update memory: ok", flush=True)
"""


def _child(tmp_path, code, *args):
    so = tmp_path / "alloc_cap.so"
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "host", "alloc_cap.c"), "-o", str(so),
                           "-ldl", "-lpthread"])
    out = subprocess.run([sys.executable, "-c", code, str(so), *args], cwd=os.path.dirname(HERE), capture_output=True,
                         text=True, timeout=110)
    assert out.returncode == 0, (out.stdout[-2000:], out.stderr[-3000:])
    return out.stdout


def test_a_load_fits_where_its_arrays_fit(tmp_path):
    assert "load memory: ok" in _child(tmp_path, LOAD)


def test_an_update_that_does_not_fit_changes_nothing(tmp_path):
    import torch
    assert torch.cuda.is_available()
    import graphgen
    import paper_1612_09368_amd as cm
    n = 5000
    s, d = graphgen.er_graph(n, 40000, graphgen.rng_for("update-memory"))
    with cm.Graph() as g:
        g.load(n, s, d)
        g.decompose()
        g.snapshot(tmp_path / "snap")
    assert "update memory: ok" in _child(tmp_path, UPDATE, str(tmp_path / "snap"))
