"""Cascades at the edges of the walks that run them: chains that end inside,
at and past the steps a wave walks of its own finds in one round, and lists
around one wave step, one group of steps, one chunk and the longest list a
wave walks alone; every result against a recount from scratch."""
import numpy as np
import pytest
import torch

import oracle
import paper_1612_09368_amd as cm

pytestmark = pytest.mark.gpu

FORMS = [dict(mode=cm.MODE_PLAIN), dict(mode=cm.MODE_PERSISTENT), dict(mode=cm.MODE_PERSISTENT, expand_mode=2),
         dict(mode=cm.MODE_PERSISTENT, expand_mode=3, large_degree=16, chunk=32)]


def _check(g, ref):
    assert np.array_equal(g.cores(), ref.cores())
    n, s, d = ref.n, *ref.edges()
    c = ref.cores()
    sd = np.zeros(n, np.int64)
    np.add.at(sd, s, c[d] >= c[s])
    np.add.at(sd, d, c[s] >= c[d])
    assert np.array_equal(g.superior_degrees(), np.where(c >= 0, sd, 0))


def _round_trip(n, s, d, batch, cfg):
    """Delete the batch, insert it again, checked after load and each half."""
    assert torch.cuda.is_available()
    s, d = np.asarray(s, np.int32), np.asarray(d, np.int32)
    b = np.asarray(batch, np.int32).reshape(-1, 2)
    ref = oracle.DynamicGraph(n, s, d)
    with cm.Graph(**cfg) as g:
        g.load(n, s, d)
        g.decompose()
        _check(g, ref)
        for _ in range(2):
            g.delete_edges(b[:, 0], b[:, 1])
            ref.delete_edges(b[:, 0].copy(), b[:, 1].copy())
            _check(g, ref)
            g.insert_edges(b[:, 0], b[:, 1])
            ref.insert_edges(b[:, 0].copy(), b[:, 1].copy())
            _check(g, ref)


@pytest.mark.parametrize("cfg", FORMS, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
@pytest.mark.parametrize("n", [3, 8, 15, 16, 17, 18, 19, 33, 65, 129, 1000])
def test_chain_depth(n, cfg):
    """A cycle loses one edge: the peel runs down both arms; putting it back
    expands over the whole cycle.  A second cycle keeps its cores."""
    s = np.concatenate([np.arange(n), n + np.arange(n)])
    d = np.concatenate([(np.arange(n) + 1) % n, n + (np.arange(n) + 1) % n])
    _round_trip(2 * n, np.minimum(s, d), np.maximum(s, d), [(0, 1)], cfg)


@pytest.mark.parametrize("cfg", FORMS, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
@pytest.mark.parametrize("width", [1, 7, 12, 13, 63, 64, 65, 200])
def test_wide_then_narrow(width, cfg):
    """Cycles that share a vertex: one deletion peels `width` arms at once,
    then each arm alone."""
    arm = 24
    s, d = [], []
    nxt = 1
    for _ in range(width):
        ids = [0, *range(nxt, nxt + arm), 0]
        nxt += arm
        for a, b in zip(ids, ids[1:]):
            s.append(min(a, b))
            d.append(max(a, b))
    cut = [(s[i * (arm + 1) + arm // 2], d[i * (arm + 1) + arm // 2]) for i in range(width)]
    _round_trip(nxt, s, d, cut, cfg)


@pytest.mark.parametrize("cfg", FORMS, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
@pytest.mark.parametrize("deg", [62, 63, 64, 65, 128, 255, 256, 257, 511, 512, 513, 1030])
def test_hub_lists(deg, cfg):
    """Hubs of about `deg` neighbours along a chain: every hub's list holds a
    wheel (rim vertices at core 3) and its two chain neighbours, so that rim
    edges pull hubs and rims across a level."""
    hubs, s, d = 4, [], []
    rim0 = hubs
    cut = []
    for h in range(hubs):
        r = np.arange(rim0 + h * deg, rim0 + (h + 1) * deg)
        for a, b in zip(r, np.roll(r, -1)):
            s.append(min(a, b))
            d.append(max(a, b))
        s += [h] * deg
        d += r.tolist()
        cut.append((int(r[0]), int(r[1])))
        cut.append((int(r[deg // 2]), int(r[deg // 2 + 1])))
        if h:
            s.append(h - 1)
            d.append(h)
    _round_trip(hubs + hubs * deg, s, d, cut, cfg)


def _cliques(sizes):
    s, d, base = [], [], 0
    for k in sizes:
        i, j = np.triu_indices(k, 1)
        s.append(base + i)
        d.append(base + j)
        base += k
    return base, np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32)


@pytest.mark.parametrize("sizes", [[2], [9, 10], [8, 9, 10, 17, 18, 19], [2, 200], [70, 71, 72, 80, 90, 300],
                                   list(range(2, 60)), [3] * 1364 + [4], [3] * 1365 + [4], [2] * 2048 + [40]],
                         ids=lambda x: f"{len(x)}cliques{max(x)}")
def test_decompose_level_gaps(sizes):
    """Cliques of chosen sizes: empty levels inside and past the near list's
    window, and vertex counts around the sweeps that one workgroup runs."""
    n, s, d = _cliques(sizes)
    n += 1  # an isolated id
    with cm.Graph() as g:
        g.load(n, s, d)
        g.decompose()
        ref = oracle.DynamicGraph(n, s, d)
        _check(g, ref)
        # dead ids and tombstones, then from scratch again
        gone = np.arange(0, n, 7, dtype=np.int32)
        g.delete_vertices(gone)
        ref.delete_vertices(gone)
        g.decompose()
        _check(g, ref)


@pytest.mark.parametrize("joint", [0, 1, 10 ** 6], ids=["apart", "one", "matched"])
@pytest.mark.parametrize("sizes", [[3, 4, 5], list(range(3, 30)), [9, 10, 11, 12, 13], [63, 64, 65, 66, 67],
                                   [512, 513, 514], [700, 701, 702, 703]], ids=lambda x: f"{x[0]}to{x[-1]}")
def test_decompose_two_levels_a_sweep(sizes, joint):
    """Cliques of successive sizes, joined by edges to the next: a level's
    removals lower the next level's vertices to its degree, short and long
    lists.  A path and a hub of paths: all that level 2 has listed goes with
    level 1."""
    n, s, d = _cliques(sizes)
    s, d = [s], [d]
    base = 0
    for x in sizes[:-1]:
        i = np.arange(min(x, joint))
        s.append(base + i)
        d.append(base + x + i)
        base += x
    p = n + np.arange(2999)
    s.append(p)
    d.append(p + 1)
    hub = n + 3000
    arm = hub + 1 + np.arange(600)
    s += [np.full(600, hub), arm]
    d += [arm, arm + 600]
    n = hub + 1201
    s, d = np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32)
    ref = oracle.DynamicGraph(n, s, d)
    with cm.Graph() as g:
        g.load(n, s, d)
        for _ in range(2):
            g.decompose()
            _check(g, ref)


@pytest.mark.parametrize("mode", [cm.MODE_PLAIN, cm.MODE_PERSISTENT])
def test_vertex_stars_filter_mode(mode):
    """One-call vertex operations with invalid items, dropped one by one."""
    rng = np.random.RandomState(5)
    n, s, d = _cliques([12, 9, 30, 5])
    off = np.array([0, 5, 5, 12, 15], np.int64)
    nb = np.concatenate([[0, 3, 3, n + 50, 20], rng.permutation(n)[:7], [n, n + 2, 1]]).astype(np.int32)
    with cm.Graph(mode=mode, strict=False) as g:
        g.load(n, s, d)
        g.decompose()
        ref = oracle.DynamicGraph(n, s, d)
        g.insert_vertices(off, nb)
        ref.insert_vertices(off, nb, strict=False)
        _check(g, ref)
        ids = np.array([0, 13, 13, n + 1, n + 99, 2], np.int32)
        g.delete_vertices(ids)
        ref.delete_vertices(ids, strict=False)
        _check(g, ref)


@pytest.mark.parametrize("bad,code", [((0, 1), cm.E_DUP), ((1, 0), cm.E_DUP), ((4, 4), cm.E_SELF_LOOP),
                                      ((0, 99), cm.E_RANGE), ((-1, 3), cm.E_RANGE)])
@pytest.mark.parametrize("where", [1, 20, -1])
def test_load_rejects_and_loads_again(bad, code, where):
    """A bad edge anywhere fails the load with its own code; the handle then
    loads graphs of other sizes, larger and smaller, over each other."""
    with cm.Graph() as g:
        for sizes in ([12, 9], [40, 30, 3], [5]):
            n, s, d = _cliques(sizes)
            if sizes[0] == 12:
                w = where if where >= 0 else len(s)
                with pytest.raises(cm.CoreMaintError) as e:
                    g.load(n, np.insert(s, w, bad[0]), np.insert(d, w, bad[1]))
                assert e.value.status == code
            for _ in range(2):
                g.load(n, s, d)
                g.decompose()
                _check(g, oracle.DynamicGraph(n, s, d))


@pytest.mark.parametrize("strict", [True, False])
@pytest.mark.parametrize("mode", [cm.MODE_PLAIN, cm.MODE_PERSISTENT])
@pytest.mark.parametrize("s", [1, 2, 511, 513, 4095, 4096, 4097])
def test_batch_sizes_around_fused_preparation(s, mode, strict):
    """Batches at the edges of the sizes prepared inside their first launch:
    hubs whose lists the locate scan reads (up to the whole grid's), lists that
    must move, the pool repacked, invalid items first and last."""
    rng = np.random.RandomState(s)
    hubs, n = 6, 9000
    keys = set()
    for h in range(hubs):
        for w in range(hubs, n, 1 + h):
            keys.add((h, w))
    base = np.array(sorted(keys), np.int32)
    ref = oracle.DynamicGraph(n, base[:, 0], base[:, 1])
    with cm.Graph(mode=mode, strict=strict) as g:
        g.load(n, base[:, 0], base[:, 1])
        g.decompose()
        for rnd in range(3):
            new = set()
            while len(new) < s:
                a, b = (rng.randint(hubs, 400), rng.randint(hubs, n)) if rnd != 1 else (rng.randint(hubs), rng.randint(n))
                if a != b and (min(a, b), max(a, b)) not in keys:
                    new.add((min(a, b), max(a, b)))
                elif rnd == 1 and len(keys) + len(new) > hubs * n - hubs * hubs:
                    break
                elif rnd == 1 and rng.rand() < 0.2:
                    new.add((int(rng.randint(hubs, 400)), int(rng.randint(400, n))))
                    new -= keys
            x = np.array(sorted(new), np.int32)
            for bad in ((0, 0), (n, 1), tuple(base[0])):
                for at in (0, len(x)):
                    y = np.insert(x, at, bad, axis=0)
                    st, stats = g.insert_edges(y[:, 0], y[:, 1], check=False)
                    want = ref.insert_edges(y[:, 0].copy(), y[:, 1].copy(), strict=strict)
                    assert st == want[0] and stats.first_bad == at
                    _check(g, ref)
                    if not strict:
                        g.delete_edges(x[:, 0], x[:, 1])
                        ref.delete_edges(x[:, 0].copy(), x[:, 1].copy())
            g.insert_edges(x[:, 0], x[:, 1])
            ref.insert_edges(x[:, 0].copy(), x[:, 1].copy())
            _check(g, ref)
            st, stats = g.delete_edges(np.append(x[:, 0], 0), np.append(x[:, 1], 1 if (0, 1) not in keys else 0), check=False)
            want = ref.delete_edges(np.append(x[:, 0], 0), np.append(x[:, 1], 1 if (0, 1) not in keys else 0), strict=strict)
            assert st == want[0] and stats.first_bad == len(x)
            _check(g, ref)
            if strict:
                g.delete_edges(x[:, 0], x[:, 1])
                ref.delete_edges(x[:, 0].copy(), x[:, 1].copy())
                _check(g, ref)


@pytest.mark.parametrize("mode", [cm.MODE_PLAIN, cm.MODE_PERSISTENT])
@pytest.mark.parametrize("s", [16384, 16385, 65536, 65537, 150001])
def test_batch_sizes_around_wave_spans(s, mode):
    """Batches at the edges of the runs a wave takes in the partition,
    validation and reservation steps."""
    rng = np.random.RandomState(s)
    n = 20000
    u, v = rng.randint(0, n, 400000), rng.randint(0, n, 400000)
    keys = np.unique((np.minimum(u, v) * n + np.maximum(u, v))[u != v])
    rng.shuffle(keys)
    first, batch = keys[:60000], keys[60000:60000 + s]
    _round_trip(n, *(x.astype(np.int32) for x in divmod(np.concatenate([first, batch]), n)),
                np.stack(divmod(batch, n), 1), dict(mode=mode))


@pytest.mark.parametrize("cfg", [dict(mode=cm.MODE_PLAIN), dict(mode=cm.MODE_PERSISTENT),
                                 dict(mode=cm.MODE_PERSISTENT, local_items=1, chunk=32),
                                 dict(mode=cm.MODE_PERSISTENT, local_items=1, chunk=64, large_degree=64)],
                         ids=["plain", "persistent", "grid-chunk32", "grid-chunk64"])
@pytest.mark.parametrize("share", [160, 200, 240])
def test_long_supporter_runs_of_neighbouring_hubs(share, cfg):
    """Hubs with successive ids, counted by many chunks each and evicted as
    soon as they are counted, with supporter runs longer than one wave step: a
    140-regular graph, and a matching on `share` of its vertices that gives no
    vertex k + 1 supporters, so all of it is a candidate and all of it falls."""
    rng = np.random.RandomState(share)
    nd, half, hubs, leaves = 300, 70, 32, 6000
    i = np.repeat(np.arange(nd), half)
    j = (i + np.tile(np.arange(1, half + 1), nd)) % nd
    s, d = [np.minimum(i, j)], [np.maximum(i, j)]
    for h in range(hubs):
        leaf = nd + rng.choice(leaves, rng.randint(300, 1400), replace=False)
        s.append(np.full(leaf.size, h))
        d.append(leaf)
    s, d = np.concatenate(s), np.concatenate(d)
    order = rng.permutation(s.size)
    n, s, d = nd + leaves, s[order].astype(np.int32), d[order].astype(np.int32)
    ref = oracle.DynamicGraph(n, s, d)
    before = ref.cores()
    assert (before[:nd] == 2 * half).all()
    with cm.Graph(**cfg) as g:
        g.load(n, s, d)
        g.decompose()
        for _ in range(4):
            # opposite vertices are no neighbours
            x = np.concatenate([np.arange(hubs), hubs + rng.permutation(nd // 2 - hubs)[:share // 2 - hubs]])
            a, b = x.astype(np.int32), (x + nd // 2).astype(np.int32)
            g.insert_edges(a, b)
            ref.insert_edges(a, b)
            _check(g, ref)
            assert np.array_equal(ref.cores(), before)
            g.delete_edges(a, b)
            ref.delete_edges(a, b)
            _check(g, ref)


@pytest.mark.parametrize("cfg", [dict(mode=cm.MODE_PLAIN), dict(mode=cm.MODE_PERSISTENT),
                                 dict(mode=cm.MODE_PERSISTENT, chunk=32), dict(mode=cm.MODE_PERSISTENT, large_degree=16)],
                         ids=["plain", "persistent", "chunk32", "large16"])
@pytest.mark.parametrize("half,pairs", [(400, 950), (120, 990)])
def test_eviction_of_a_dense_graph(half, pairs, cfg):
    """A regular graph of 2,000 vertices, nearly all of them candidates of one
    matching and evicted in one round with runs of hundreds of entries: more
    items of 64 entries than the lists have chunks."""
    nd = 2000
    i = np.repeat(np.arange(nd), half)
    j = (i + np.tile(np.arange(1, half + 1), nd)) % nd
    a = np.arange(pairs)
    _insert_first(nd, np.minimum(i, j), np.maximum(i, j), a, a + nd // 2, cfg)


def _insert_first(n, s, d, a, b, cfg):
    s, d, a, b = (np.asarray(x, np.int32) for x in (s, d, a, b))
    ref = oracle.DynamicGraph(n, s, d)
    with cm.Graph(**cfg) as g:
        g.load(n, s, d)
        g.decompose()
        for _ in range(2):
            g.insert_edges(a, b)
            ref.insert_edges(a, b)
            _check(g, ref)
            g.delete_edges(a, b)
            ref.delete_edges(a, b)
            _check(g, ref)
