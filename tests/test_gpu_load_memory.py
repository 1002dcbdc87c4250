"""Device memory of a load: a graph fits where its own arrays fit, without the
load's temporaries beside them; in memory for one of two graphs, each loads
over the other.  The library's hipMalloc goes through a counter with a cap, in
a process of its own."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r"""
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


def test_a_load_fits_where_its_arrays_fit(tmp_path):
    so = tmp_path / "alloc_cap.so"
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "host", "alloc_cap.c"), "-o", str(so),
                           "-ldl", "-lpthread"])
    out = subprocess.run([sys.executable, "-c", CHILD, str(so)], cwd=os.path.dirname(HERE), capture_output=True,
                         text=True, timeout=110)
    assert out.returncode == 0, (out.stdout[-2000:], out.stderr[-3000:])
    assert "load memory: ok" in out.stdout
