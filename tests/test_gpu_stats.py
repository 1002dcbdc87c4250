"""What the calls report of themselves: step counts and launch times of the
vertex operations in the plain form, steps of program batches."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
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


@pytest.mark.parametrize("mode", [cm.MODE_PLAIN, cm.MODE_PERSISTENT])
@pytest.mark.parametrize("k", [1023, 1024, 1025, 2048])
def test_largest_batch_prepared_inside_its_launch(k, mode):
    """Up to 1,024 items workgroup 0 prepares the batch; above that the whole
    grid's own kernels are faster, and take it."""
    n, s, d, _ = _graph()
    es = graphgen.EdgeSet(s, d)
    a, b = graphgen.uniform_non_edges(n, k, es, graphgen.rng_for("stats-k", k))
    ref = oracle.DynamicGraph(n, s, d)
    with cm.Graph(mode=mode) as g:
        g.load(n, s, d)
        g.decompose()
        for call, model in ((g.insert_edges, ref.insert_edges), (g.delete_edges, ref.delete_edges)):
            g.phase_times(reset=True)
            call(a, b)
            model(a, b)
            ph = g.phase_times()
            assert [ph[p][1] for p in ("validate", "reserve")] == ([1, 1] if k <= 1024 else [0, 0])
            assert np.array_equal(g.cores(), ref.cores())


@pytest.mark.parametrize("mode", [cm.MODE_PLAIN, cm.MODE_PERSISTENT])
@pytest.mark.parametrize("lists", [1, 16, 17])
def test_moved_lists(lists, mode):
    """Full lists of lengths around one wave step and one group of steps of the
    copy, moved by one more entry each: in workgroup 0 and by the grid."""
    size = [1, 4, 60, 64, 68, 448, 455, 456, 508, 512, 516, 1024, 1028, 1536, 3000, 8192, 12000][:lists]
    n = lists + 16000
    c = [(x + max(x >> 3, 4) + 3) & ~3 for x in size]  # slots of a list loaded with x entries
    h = np.arange(lists, dtype=np.int32)
    s = np.repeat(h, c)
    d = np.concatenate([lists + np.arange(x) for x in c]).astype(np.int32)
    first = np.concatenate([np.arange(x) < y for x, y in zip(c, size)])
    ref = oracle.DynamicGraph(n, s, d)
    with cm.Graph(mode=mode) as g:
        g.load(n, s[first], d[first])
        g.decompose()
        g.insert_edges(s[~first], d[~first])
        top = np.full(lists, n - 1, np.int32)
        for call, model in ((g.insert_edges, ref.insert_edges), (g.delete_edges, ref.delete_edges)):
            call(h, top)
            model(h, top)
            assert np.array_equal(g.cores(), ref.cores())
            got, want = g.export_edges(), ref.edges()
            key = [np.sort(np.minimum(x, y).astype(np.int64) * n + np.maximum(x, y)) for x, y in (got, want)]
            assert np.array_equal(*key)


@pytest.mark.parametrize("mode", [cm.MODE_PLAIN, cm.MODE_PERSISTENT])
def test_vertices_without_edges_leave_in_counted_steps(mode):
    """Their steps are theirs, not the next batch's."""
    n, s, d, _ = _graph()
    with cm.Graph(mode=mode) as g:
        g.load(n + 100, s, d)
        g.decompose()
        st = g.delete_vertices(np.arange(n, n + 100, 3, dtype=np.int32))
        assert st.iterations > 0 and st.applied == 0
        assert st.grid_steps >= st.iterations
        ref = oracle.DynamicGraph(n, s, d)
        assert np.array_equal(g.cores()[:n], ref.cores())
        left = g.cores()[n:]
        assert (left[::3] == -1).all() and (np.delete(left, np.arange(0, 100, 3)) == 0).all()
        assert g.num_vertices() == (n + 100, n + 100 - 34)
