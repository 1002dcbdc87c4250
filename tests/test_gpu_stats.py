"""What the calls report of themselves: step counts and launch times of the
vertex operations in the plain form, steps of program batches."""
import numpy as np
import pytest
import torch

import graphgen
import paper_1612_09368_amd as cm

pytestmark = pytest.mark.gpu


def _graph(n=3000, m=15000):
    assert torch.cuda.is_available()
    rng = graphgen.rng_for("stats")
    s, d = graphgen.er_graph(n, m, rng)
    return n, s, d, graphgen.uniform_non_edges(n, 600, graphgen.EdgeSet(s, d), rng)


@pytest.mark.parametrize("use_graph", [0, 1])
def test_plain_vertex_operations_report_steps_and_time(use_graph):
    n, s, d, _ = _graph()
    off = np.arange(0, 41 * 8, 8, dtype=np.int64)
    nb = np.concatenate([np.random.RandomState(i).permutation(n)[:8] for i in range(40)]).astype(np.int32)
    with cm.Graph(mode=cm.MODE_PLAIN, use_graph=use_graph) as g:
        g.load(n, s, d)
        g.decompose()
        _, ins = g.insert_vertices(off, nb)
        for st in (ins, g.delete_vertices(np.arange(n, n + 40, dtype=np.int32))):
            assert st.launches == 1 and st.iterations > 0 and st.applied == 320
            assert 0.0 < st.kernel_ms <= st.ms_total
            assert st.grid_steps > 0  # the star steps are the grid's
            assert st.graph_launch == 0


@pytest.mark.parametrize("use_graph", [0, 1])
def test_program_batches_report_both_kinds_of_steps(use_graph):
    n, s, d, (a, b) = _graph()
    for cfg in (dict(), dict(local_edges=1, local_items=1)):
        with cm.Graph(mode=cm.MODE_PERSISTENT, use_graph=use_graph, **cfg) as g:
            g.load(n, s, d)
            g.decompose()
            res, _ = g.run_batches([cm.BATCH_INSERT, cm.BATCH_DELETE], [0, a.size, 2 * a.size],
                                   np.concatenate([a, a]), np.concatenate([b, b]))
            for st in res:
                assert st.applied == a.size
                assert st.grid_steps > 0 if cfg else st.local_steps > 0


@pytest.mark.parametrize("mode", [cm.MODE_PLAIN, cm.MODE_PERSISTENT])
def test_phase_clock_of_small_batches(mode):
    """Validation, reservation and compaction run inside the maintenance launch
    of a small batch, and show in the phase clock: once per batch."""
    n, s, d, (a, b) = _graph()
    with cm.Graph(mode=mode, timing=True) as g:
        g.load(n, s, d)
        g.decompose()
        for k in (1, 600):
            g.phase_times(reset=True)
            ins = g.insert_edges(a[:k], b[:k])
            ph = g.phase_times(reset=True)
            assert [ph[p][1] for p in ("validate", "reserve", "compact")] == [1, 1, 0]
            assert all(0.0 < ph[p][0] < ins.kernel_ms for p in ("validate", "reserve"))
            dele = g.delete_edges(a[:k], b[:k])
            ph = g.phase_times(reset=True)
            assert [ph[p][1] for p in ("validate", "reserve", "compact")] == [1, 1, 1]
            assert all(0.0 < ph[p][0] < dele.kernel_ms for p in ("validate", "reserve", "compact"))
        with pytest.raises(cm.CoreMaintError):
            g.insert_edges(s[:1], d[:1])
        ph = g.phase_times()
        assert [ph[p][1] for p in ("validate", "reserve", "compact")] == [1, 0, 0]
