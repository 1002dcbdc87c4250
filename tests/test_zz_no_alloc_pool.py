"""The allocation-free entry point with a full adjacency pool: a batch whose
lists cannot move is refused with CM_E_CAPACITY and nothing applied, in batches
of one edge (no launch queued behind the first), of a few and of the most that
one launch prepares (one queued), and larger ones (prepared by kernels of
their own); deletions go on, and the allocating entry point takes the same
batch."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _state(g):
    s, d = g.export_edges()
    order = np.lexsort((np.maximum(s, d), np.minimum(s, d)))
    return (g.cores(), g.superior_degrees(), np.minimum(s, d)[order], np.maximum(s, d)[order],
            np.array([g.num_edges()]))


def _check(g, ref):
    assert np.array_equal(g.cores(), ref.cores())
    s, d = ref.edges()
    c = ref.cores()
    sd = np.zeros(ref.n, np.int64)
    np.add.at(sd, s, c[d] >= c[s])
    np.add.at(sd, d, c[s] >= c[d])
    assert np.array_equal(g.superior_degrees(), sd)
    assert g.num_edges() == ref.num_edges()


@pytest.mark.parametrize("s", [1, 2, 300, 1024, 1025, 4096, 4097])
@pytest.mark.parametrize("mode", [0, 1], ids=["plain", "persistent"])
def test_full_pool(mode, s):
    import torch
    assert torch.cuda.is_available()
    import paper_1612_09368_amd as cm

    def dev(x):
        return torch.from_numpy(np.ascontiguousarray(x, np.int32)).to("cuda:0")

    rng = np.random.RandomState(s)
    n = 2000
    i, j = np.triu_indices(n, 1)
    order = rng.permutation(i.size)[:120_000]
    i, j = i[order].astype(np.int32), j[order].astype(np.int32)
    m = 6000
    ref = oracle.DynamicGraph(n, i[:m], j[:m])
    with cm.Graph(mode=mode, timing=True) as g:
        g.load(n, i[:m], j[:m])
        g.decompose()
        # fill: batches until one is refused, then ones of s items
        at, k, full = m, 500, False
        while at + 4 * s < i.size:
            a, b = i[at:at + k], j[at:at + k]
            before = _state(g)
            st, stats = g.update_edges_noalloc(cm.BATCH_INSERT, dev(a), dev(b), check=False)
            if st == cm.OK:
                assert not full or k < 500  # a single edge may still find room in its two lists
                ref.insert_edges(a, b)
                at += k
                continue
            assert st == cm.E_CAPACITY
            assert stats.applied == 0 and stats.launches == 0 and stats.kernel_ms == 0.0
            assert all(np.array_equal(x, y) for x, y in zip(before, _state(g)))
            if full:
                break
            full, k = True, s
        else:
            raise AssertionError("the pool never filled")
        _check(g, ref)
        # a deletion needs no room
        x, y = ref.edges()
        pick = rng.permutation(x.size)[:min(s, 1000)]
        x, y = x[pick].astype(np.int32), y[pick].astype(np.int32)
        g.update_edges_noalloc(cm.BATCH_DELETE, dev(x), dev(y))
        ref.delete_edges(x, y)
        _check(g, ref)
        # the refused batch through the allocating call, and then without allocation again
        g.insert_edges(a, b)
        ref.insert_edges(a, b)
        _check(g, ref)
        g.update_edges_noalloc(cm.BATCH_INSERT, dev(x), dev(y))
        ref.insert_edges(x, y)
        _check(g, ref)
