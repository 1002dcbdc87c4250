"""Workgroup 0 runs chains of small steps while the other workgroups still
look at the counters of the barrier before: the counters' rotation on the host
(cm_steps.h), and updates that go from whole-grid rounds into such chains and
back at every level, against a recount from scratch."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_late_looks_at_the_counters(tmp_path):
    exe = tmp_path / "chain_check"
    subprocess.check_call(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                           os.path.join(HERE, "host", "chain_check.cpp"), "-o", str(exe)],
                          stderr=subprocess.DEVNULL)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    assert "chain: ok" in out.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("items", [1, 8, 64])
@pytest.mark.parametrize("mode", [0, 1], ids=["plain", "persistent"])
def test_grid_rounds_into_chains_and_back(mode, items):
    """Arms of lengths 1 to 700 on one ring vertex, cut in the middle: rounds
    narrow from hundreds of vertices to one, so that the cascade leaves the grid
    for workgroup 0; the next batch starts wide again.  The decomposition of
    the same graph narrows and widens with its levels."""
    import oracle
    import torch
    import paper_1612_09368_amd as cm
    assert torch.cuda.is_available()
    s, d, cut, nxt = [], [], [], 1
    for arm in [*range(3, 120), *range(120, 700, 29)]:
        ids = [0, *range(nxt, nxt + arm), 0]
        nxt += arm
        e = list(zip(ids, ids[1:]))
        cut.append(e[len(e) // 2])
        s += [min(p) for p in e]
        d += [max(p) for p in e]
    for k in (5, 9, 30):  # cliques: levels above
        i, j = np.triu_indices(k, 1)
        s += (nxt + i).tolist()
        d += (nxt + j).tolist()
        nxt += k
    s, d = np.asarray(s, np.int32), np.asarray(d, np.int32)
    a, b = np.sort(np.asarray(cut, np.int32), axis=1).T.copy()
    ref = oracle.DynamicGraph(nxt, s, d)
    with cm.Graph(mode=mode, local_items=items) as g:
        for _ in range(3):
            g.load(nxt, s, d)
            g.decompose()
            assert np.array_equal(g.cores(), ref.cores())
            for _ in range(3):
                st = g.delete_edges(a, b)
                ref.delete_edges(a, b)
                assert np.array_equal(g.cores(), ref.cores())
                assert st.local_steps > 0 and (items == 64 or st.grid_steps > 0)
                g.insert_edges(a, b)
                ref.insert_edges(a, b)
                assert np.array_equal(g.cores(), ref.cores())


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 1], ids=["plain", "persistent"])
def test_chains_of_long_steps(mode):
    """Bounds that keep every step in workgroup 0, whatever its size: the chain
    looks at its slice after each step, hands back to the grid and goes on."""
    import graphgen
    import oracle
    import paper_1612_09368_amd as cm
    import torch
    assert torch.cuda.is_available()
    n = 20_000
    s, d = graphgen.er_graph(n, 100_000, graphgen.rng_for("chain-long"))
    es = graphgen.EdgeSet(s, d)
    a, b = graphgen.uniform_non_edges(n, 5000, es, graphgen.rng_for("chain-long", 1))
    ref = oracle.DynamicGraph(n, s, d)
    big = (1 << 31) - 1
    with cm.Graph(mode=mode, local_edges=big, local_items=big, local_work=big) as g:
        g.load(n, s, d)
        g.decompose()
        assert np.array_equal(g.cores(), ref.cores())
        for _ in range(2):
            for call, model in ((g.insert_edges, ref.insert_edges), (g.delete_edges, ref.delete_edges)):
                st = call(a, b)
                model(a, b)
                assert np.array_equal(g.cores(), ref.cores())
                assert st.local_steps > 0 and st.grid_steps == 0
