// Load-balanced walks over frontier queues (gfx950, wave64).
//
// A frontier is a list of vertices plus a list of chunk items for long
// adjacency lists.  Each wave takes a batch of up to 64 queue entries and
// walks their lists laid end to end, one slot per lane per step, so short
// and medium lists keep every lane busy; lists longer than `large` never
// enter the vertex list -- the pusher splits them into chunk items that
// separate waves walk.  Pushes go through per-wave LDS buffers so that a
// queue tail takes one atomic per 64 or more entries.
#pragma once
#include "cm_internal.h"

namespace cm {

// Write the chunk items (w, 0), .., (w, nch - 1) of every lane (nch = 0 for
// none) from position `base` of a chunk queue on.  The wave writes them
// together, lane i taking items i, i + 64, ..., so a very long list does not
// serialise on its own lane.  Every lane of the wave must call it; incl =
// the inclusive scan of nch.
__device__ __forceinline__ void write_chunks(const KArgs &a, int64_t *hq, int32_t base, int32_t w, int32_t nch,
                                             int32_t incl) {
    const int32_t total = __builtin_amdgcn_readlane(incl, WAVE - 1);
    const int32_t excl = incl - nch;
    for (int32_t e0 = 0; e0 < total; e0 += WAVE) {
        const int32_t e = e0 + lane();
        // owner of item e: the last lane whose items start at or before e
        // (a lane with no items shares its start with the next lane, so
        // the owner of a valid item always has items)
        int32_t j = 0;
        for (int s = WAVE / 2; s > 0; s >>= 1) {
            const int32_t xc = __shfl(excl, j + s);
            if (xc <= e) j += s;
        }
        const int32_t xj = __shfl(excl, j);
        const int32_t wj = __shfl(w, j);
        if (e < total) {
            const int32_t pos = base + e;
            if (pos < a.q.hcap) hq[pos] = chunk_item(wj, e - xj);
            else atomicOr(&a.ctl->overflow, 1);
        }
    }
}

// Append the chunk items of every lane to a chunk queue with one tail atomic
// per wave: returning atomics on one word serialise (about 11 ns each), and
// one per long list bound the rounds that push many of them.  A wave with
// inactive lanes (the last pass of a strided loop) pushes lane by lane.
__device__ __forceinline__ void push_chunks(const KArgs &a, int64_t *hq, int32_t *htail, int32_t w,
                                            int32_t nch) {
    if (__ballot(nch > 0) == 0ull) return;
    if (__ballot(1) != ~0ull) {
        if (nch > 0) {
            const int32_t base = atomicAdd(htail, nch);
            for (int32_t c = 0; c < nch; ++c) {
                if (base + c < a.q.hcap) hq[base + c] = chunk_item(w, c);
                else atomicOr(&a.ctl->overflow, 1);
            }
        }
        return;
    }
    const int32_t incl = wave_incl_add(nch);
    int32_t base = 0;
    if (lane() == WAVE - 1) base = atomicAdd(htail, incl);
    write_chunks(a, hq, __builtin_amdgcn_readlane(base, WAVE - 1), w, nch, incl);
}

// Route a pushed vertex: short/medium lists to the vertex queue, long lists
// as `nchunks` items to the chunk queue.  All lanes may call it (pred
// selects the pushing lanes).
__device__ __forceinline__ void push_vertex(const KArgs &a, int32_t *vq, int32_t *vtail, int64_t *hq,
                                            int32_t *htail, int32_t w, bool pred) {
    int32_t L = pred ? a.g.len[w] : 0;
    bool big = pred && L > a.t.large_deg;
    push_agg<int32_t>(vq, a.q.vcap, vtail, w, pred && !big, &a.ctl->overflow);
    push_chunks(a, hq, htail, w, big ? nchunks(L, a.t.chunk) : 0);
}

// Per-wave push buffers in LDS.  A queue tail is one word that every wave
// appends to, and returning atomics on one address serialise (about 11 ns
// each on gfx950), so a traversal step that pushed with one atomic per wave
// per step was bound by that word.  A wave instead collects its pushes in
// LDS and appends them with one atomic per 64 or more entries; a round
// flushes its buffers before its barrier.  wb_push / push_vertex_wb must be
// called by every lane of the wave (pred selects the pushing lanes).
constexpr int PUSH_SLOTS = 6;
struct WaveBuf {
    int32_t *buf;  // 2 * WAVE entries of this wave's slot
    int32_t n;     // entries held (uniform over the wave)
};
__device__ __forceinline__ WaveBuf wave_buf(int slot) {
    __shared__ int32_t lds_push[PUSH_SLOTS][COOP_THREADS / WAVE][2 * WAVE];
    return WaveBuf{lds_push[slot][threadIdx.x / WAVE], 0};
}
__device__ __forceinline__ void wb_flush(WaveBuf &b, int32_t *q, int32_t qcap, int32_t *tail, int32_t *overflow) {
    if (b.n == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // other lanes' LDS writes come first
    int base = 0;
    if (lane() == 0) base = atomicAdd(tail, b.n);
    base = __shfl(base, 0);
    for (int i = lane(); i < b.n; i += WAVE) {
        const int pos = base + i;
        if (pos < qcap) q[pos] = b.buf[i];
        else atomicOr(overflow, 1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // reads done before the slots are reused
    b.n = 0;
}
__device__ __forceinline__ void wb_push(WaveBuf &b, int32_t *q, int32_t qcap, int32_t *tail, int32_t val,
                                        bool pred, int32_t *overflow) {
    const unsigned long long m = __ballot(pred);
    if (m == 0ull) return;
    if (pred) b.buf[b.n + __popcll(m & ((1ull << lane()) - 1ull))] = val;
    b.n += __popcll(m);
    if (b.n >= WAVE) wb_flush(b, q, qcap, tail, overflow);
}
// Two kinds of streams that a step pushes to: vertices to a vertex queue, and
// vertices with long walks to a chunk queue, as items of `chunk` entries of
// their walk.  Both collect in a wave buffer; a chunk stream keeps each
// vertex's walk length beside it, as its pusher had it.  The length is not read
// again at the flush: a supporter run of the expansion gets its length from
// atomics of other CUs in the same step, and a plain read may still return an
// older one from this CU's L1 (another wave of the workgroup has read a
// neighbouring word), which would leave the end of the run unwalked.
struct VStream {
    WaveBuf b;
    int32_t *q, *tail;
};
struct CStream {
    WaveBuf b;
    int32_t *len;  // walk lengths of the buffer's entries
    int64_t *q;
    int32_t *tail;
    int32_t chunk;
};
constexpr int CHUNK_STREAMS = 3;  // of one step
__device__ __forceinline__ int32_t *wave_lens(int i) {
    __shared__ int32_t lds_lens[CHUNK_STREAMS][COOP_THREADS / WAVE][2 * WAVE];
    return lds_lens[i][threadIdx.x / WAVE];
}
__device__ __forceinline__ void vs_push(const KArgs &a, VStream &s, int32_t w, bool pred) {
    wb_push(s.b, s.q, a.q.vcap, s.tail, w, pred, &a.ctl->overflow);
}
__device__ __forceinline__ void cs_flush(const KArgs &a, CStream &s) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // other lanes' LDS writes come first
    for (int i0 = 0; i0 < s.b.n; i0 += WAVE) {  // up to 2 * WAVE - 1 entries
        const bool has = i0 + lane() < s.b.n;
        const int32_t w = has ? s.b.buf[i0 + lane()] : -1;
        push_chunks(a, s.q, s.tail, w, has ? nchunks(s.len[i0 + lane()], s.chunk) : 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // reads done before the slots are reused
    s.b.n = 0;
}
__device__ __forceinline__ void cs_push(const KArgs &a, CStream &s, int32_t w, int32_t L, bool pred) {
    const unsigned long long m = __ballot(pred);
    if (m == 0ull) return;
    if (pred) {
        const int32_t i = s.b.n + __popcll(m & lanes_below());
        s.b.buf[i] = w;
        s.len[i] = L;
    }
    s.b.n += __popcll(m);
    if (s.b.n >= WAVE) cs_flush(a, s);
}

// End of a step: what is left in the waves' buffers, appended with one tail
// atomic per stream and workgroup.  One per wave is 2,048 turns on a word at
// 11 ns each, for each of the streams (which share a line): a round that gave
// every wave something to push took 20 to 60 us for it.  A buffer that reaches
// WAVE entries is flushed at once, so each holds fewer here.  Every thread of
// the workgroup must call it (workgroup barriers inside).
template <int NV, int NC>
__device__ __forceinline__ void block_flush(const KArgs &a, VStream *const (&vs)[NV], CStream *const (&cs)[NC]) {
    constexpr int N = NV + NC, NW = COOP_THREADS / WAVE;
    __shared__ int32_t cnt[PUSH_SLOTS][NW];
    __shared__ int32_t first[PUSH_SLOTS];
    static_assert(N <= PUSH_SLOTS, "one slot per stream");
    const int wv = uniform((int)(threadIdx.x / WAVE));
    const int nw = (int)(blockDim.x / WAVE);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // other lanes' LDS writes come first
    int32_t w[NC], nch[NC], incl[NC], mine[N];
#pragma unroll
    for (int i = 0; i < NV; ++i) mine[i] = vs[i]->b.n;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        CStream &s = *cs[i];
        w[i] = -1;
        nch[i] = incl[i] = mine[NV + i] = 0;
        if (s.b.n > 0) {  // uniform
            if (lane() < s.b.n) {
                w[i] = s.b.buf[lane()];
                nch[i] = nchunks(s.len[lane()], s.chunk);
            }
            incl[i] = wave_incl_add(nch[i]);
            mine[NV + i] = __builtin_amdgcn_readlane(incl[i], WAVE - 1);
        }
    }
    if (lane() == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) cnt[i][wv] = mine[i];
    }
    __syncthreads();
    if (threadIdx.x < N) {
        int32_t *tail = nullptr;
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if ((int)threadIdx.x == i) tail = vs[i]->tail;
#pragma unroll
        for (int i = 0; i < NC; ++i)
            if ((int)threadIdx.x == NV + i) tail = cs[i]->tail;
        int32_t sum = 0;
        for (int j = 0; j < nw; ++j) sum += cnt[threadIdx.x][j];
        first[threadIdx.x] = sum ? atomicAdd(tail, sum) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (mine[i] == 0) continue;  // uniform
        int32_t base = first[i];
        for (int j = 0; j < wv; ++j) base += cnt[i][j];
        if (i < NV) {
            VStream &s = *vs[i < NV ? i : 0];
            if (lane() < s.b.n) {
                const int pos = base + lane();
                if (pos < a.q.vcap) s.q[pos] = s.b.buf[lane()];
                else atomicOr(&a.ctl->overflow, 1);
            }
            s.b.n = 0;
        } else {
            constexpr int Z = NV;
            const int ci = i < NV ? 0 : i - Z;
            CStream &s = *cs[ci];
            write_chunks(a, s.q, base, w[ci], nch[ci], incl[ci]);
            s.b.n = 0;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // reads done before the slots are reused
}

// The next frontier of a cascade: walks of up to `large` entries go to v,
// longer ones of up to DEEP_LIST to m (the wave may walk them itself in this
// round, see for_batches_deep; flushed as chunk items otherwise), the others to
// h.
constexpr int DEEP_LIST = 512;
struct Pusher {
    VStream v;
    CStream m, h;
    const int32_t *lens;  // walk lengths (they do not change during the step)
    int32_t large;
};
__device__ __forceinline__ Pusher make_pusher(int32_t *vq, int32_t *vtail, int64_t *hq, int32_t *htail,
                                              const int32_t *lens, int32_t large, int32_t chunk) {
    return Pusher{VStream{wave_buf(0), vq, vtail}, CStream{wave_buf(1), wave_lens(0), hq, htail, chunk},
                  CStream{wave_buf(2), wave_lens(1), hq, htail, chunk}, lens, large};
}
__device__ __forceinline__ void push_deep(const KArgs &a, Pusher &p, int32_t w, int32_t L, bool pred) {
    vs_push(a, p.v, w, pred && L <= p.large);
    cs_push(a, p.m, w, L, pred && L > p.large && L <= DEEP_LIST);
    cs_push(a, p.h, w, L, pred && L > p.large && L > DEEP_LIST);
}
__device__ __forceinline__ void push_deep(const KArgs &a, Pusher &p, int32_t w, bool pred) {
    if (__ballot(pred) == 0ull) return;
    push_deep(a, p, w, pred ? p.lens[w] : 0, pred);
}
// A vertex whose walk is not the wave's to go on with: v or c by its length L.
__device__ __forceinline__ void push_len(const KArgs &a, VStream &v, CStream &c, int32_t w, int32_t L, bool pred,
                                         int32_t large) {
    vs_push(a, v, w, pred && L <= large);
    cs_push(a, c, w, L, pred && L > large);
}
// ... one list at a time, straight to the chunk queue (steps without streams)
__device__ __forceinline__ void push_vertex_wb(const KArgs &a, WaveBuf &b, int32_t *vq, int32_t *vtail,
                                               int64_t *hq, int32_t *htail, int32_t w, bool pred) {
    const int32_t L = pred ? a.g.len[w] : 0;
    const bool big = pred && L > a.t.large_deg;
    wb_push(b, vq, a.q.vcap, vtail, w, pred && !big, &a.ctl->overflow);
    push_chunks(a, hq, htail, w, big ? nchunks(L, a.t.chunk) : 0);
}

// Team-stride over 0 .. n-1 by whole waves: f(i) runs on every lane (i < 0
// past the end), so that it may use wave votes and wave buffers.  A wave takes
// up to SPAN_STEPS steps in a row, fewer when that would leave under 256 waves
// at work: each wave then moves its pushes with one tail atomic or few, and the
// atomics of all waves on one tail (11 ns each, one after another) stay below
// a barrier's time.
constexpr int SPAN_STEPS = 4;
__device__ __forceinline__ int32_t wave_span(int32_t n) {
    const int32_t per = ((n + 255) / 256 + WAVE - 1) / WAVE;  // steps per wave for 256 waves
    return (per < 1 ? 1 : per > SPAN_STEPS ? SPAN_STEPS : per) * WAVE;
}
template <class F>
__device__ __forceinline__ void for_span(const Team &T, int32_t n, F &&f) {
    const int32_t span = wave_span(n);
    for (int32_t base = T.wave() * span; base < n; base += T.nwaves() * span) {
#pragma unroll 1
        for (int32_t o = 0; o < span && base + o < n; o += WAVE) {
            const int32_t i = base + o + lane();
            f(i < n ? i : -1);
        }
    }
}

// Team-stride over the implicit identity list 0..n-1 (whole-graph passes).
// fl(v, L) runs on the owning lane for lists of length <= small; fw(v, L)
// runs on the whole wave (uniform) for the others, of any length.
template <class FL, class FW>
__device__ __forceinline__ void for_all_vertices(const Team &T, int32_t n, const DevGraph &g, int32_t small,
                                                 FL &&fl, FW &&fw) {
    const int step = T.nwaves() * WAVE;
    for (int32_t base = T.wave() * WAVE; base < n; base += step) {
        int32_t v = base + lane();
        bool ok = v < n && g.core[v] != -1;  // -1 marks a dead id
        int32_t L = ok ? g.len[v] : 0;
        if (ok && L <= small) fl(v, L);
        unsigned long long m = __ballot(ok && L > small);
        while (m) {
            int src = __ffsll((long long)m) - 1;
            m &= m - 1ull;
            int32_t vv = __shfl(v, src);
            int32_t LL = __shfl(L, src);
            fw(vv, LL);
        }
    }
}

// Team-stride over chunk items, one wave per item: fc(v, lo, hi, L, k, o, x)
// with v's list length L (or its length in `lens`), core number k, first slot
// o and xw[v] (-1 without xw), all in scalar registers.  An item's words are
// loaded together, and with them the next item.
template <class FC>
__device__ __forceinline__ void for_chunks(const Team &T, const int64_t *q, int32_t n, const DevGraph &g,
                                           const int32_t *lens, int32_t chunk, const int32_t *xw, FC &&fc) {
    int32_t j = T.wave();
    if (j >= n) return;  // uniform
    int64_t nx = q[j];
    while (j < n) {
        const int64_t it = uniform64(nx);
        const int32_t v = item_v(it), c = item_c(it);
        j += T.nwaves();
        if (j < n) nx = q[j];
        const int32_t L0 = lens[v], k0 = g.core[v];
        const int64_t o0 = g.off[v];
        int32_t x0 = -1;
        if (xw) x0 = xw[v];
        const int32_t L = uniform(L0), k = uniform(k0), x = uniform(x0);
        const int64_t o = uniform64(o0);
        const int32_t lo = c * chunk;
        fc(v, lo, lo + chunk < L ? lo + chunk : L, L, k, o, x);
    }
}

// Wave walk of slots [lo, hi) of v: every lane calls f(w, slot) each step
// (w < 0 for padding lanes and tombstones) so f may use wave votes.
template <class F>
__device__ __forceinline__ void wave_walk(const DevGraph &g, int32_t v, int32_t lo, int32_t hi, F &&f) {
    const int32_t *p = g.nbr + g.off[v];
    for (int32_t s = lo; s < hi; s += WAVE) {
        int32_t i = s + lane();
        int32_t w = (i < hi) ? p[i] : -1;
        f(w, i);
    }
}

// Staged walks.  A step of a walk is a chain of dependent reads (the entry,
// the neighbour's core or counter, its SD and stamp, the atomic that claims
// it); a wave that walks a few hundred entries one step at a time waits for
// that chain, 2 to 3 us, at every step.  The staged walks take WALK_STEPS
// steps together, stage by stage, so that the reads and atomics of all of them
// are in flight at once (8 batches on R-MAT 22 and back: expansion 93 to
// 78 ms, SD 21 to 15 ms).  The cooperative kernels run one workgroup of 512
// threads per CU, so a thread may have 256 VGPRs: k_maintain needs 142,
// k_decompose 87, k_serve 231; k_program needs all 256 and spills 7.  A stage
// may test what earlier stages loaded and issue the next load or atomic, but must
// not look at what it issues itself (that would wait for it before the next
// step's is issued):
//   s1(e)   first gather of entry e.w (w < 0: none or a tombstone)
//   s2(e)   second gathers, chosen by the first
//   s3(e)   the atomic
//   s4(e)   the entry's flags, into e.a
//   fin(..) votes and pushes, step by step on every lane
// The gathers may read what another wave's atomic is changing: a stale stamp
// or counter only defers to the atomic.
constexpr int WALK_STEPS = 4;
struct Ent {
    int32_t w, k;        // entry, and the k of the list it is in
    int32_t a, b, c, d;  // the stages' words
};
// The steps are written out (constant indices only), so that the entries
// stay in registers.
static_assert(WALK_STEPS == 4, "CM_STEPS and pick() write out four steps");
__device__ __forceinline__ int32_t pick(int32_t x0, int32_t x1, int32_t x2, int32_t x3, int u) {
    const int32_t lo = u == 0 ? x0 : x1, hi = u == 2 ? x2 : x3;
    return u < 2 ? lo : hi;
}
#define CM_STEPS(body)                      \
    do {                                    \
        { constexpr int u = 0; body }       \
        { constexpr int u = 1; body }       \
        { constexpr int u = 2; body }       \
        { constexpr int u = 3; body }       \
    } while (0)
template <class S1, class S2, class S3, class S4>
__device__ __forceinline__ void walk_stages(Ent (&e)[WALK_STEPS], S1 &&s1, S2 &&s2, S3 &&s3, S4 &&s4) {
    CM_STEPS(s1(e[u]););
    CM_STEPS(s2(e[u]););
    CM_STEPS(s3(e[u]););
    CM_STEPS(s4(e[u]););
}

// Staged wave walk of p[lo, hi), every entry with the same k: fin(w, flags).
template <class S1, class S2, class S3, class S4, class FIN>
__device__ __forceinline__ void wave_walk_st(const int32_t *p, int32_t lo, int32_t hi, int32_t k, S1 &&s1,
                                             S2 &&s2, S3 &&s3, S4 &&s4, FIN &&fin) {
    for (int32_t s0 = lo; s0 < hi; s0 += WALK_STEPS * WAVE) {
        Ent e[WALK_STEPS];
        CM_STEPS(
            const int32_t i = s0 + u * WAVE + lane();
            e[u].w = -1;
            e[u].k = k;
            if (i < hi) e[u].w = p[i];
        );
        walk_stages(e, s1, s2, s3, s4);
#pragma unroll 1
        for (int u = 0; u < WALK_STEPS && s0 + u * WAVE < hi; ++u)
            fin(pick(e[0].w, e[1].w, e[2].w, e[3].w, u), pick(e[0].a, e[1].a, e[2].a, e[3].a, u));
    }
}

// Staged wave walk of chunk [lo, hi) of the list at slot o through its up-list
// (ub = ubl of its owner, >= 0): the chunk's compacted up-list entries, built from slots
// [lo, min(hi, ub)) and ending at a negative entry when fewer, then the slots
// appended since (from ub on).  Returns the entries read (uniform).
template <class S1, class S2, class S3, class S4, class FIN>
__device__ __forceinline__ int32_t walk_chunk_up(const DevGraph &g, int32_t lo, int32_t hi,
                                                 int32_t ub, int32_t k, int64_t o, S1 &&s1, S2 &&s2,
                                                 S3 &&s3, S4 &&s4, FIN &&fin) {
    int32_t seen = 0;
    const int32_t hb = hi < ub ? hi : ub;
    const int32_t nb = hb - lo;  // slots of the chunk's up-list
    const int32_t *up = g.upl + o + lo;
    const int32_t *app = g.nbr + o;
    const int32_t ab = lo > ub ? lo : ub;  // first appended slot
    bool more = nb > 0;
    int32_t s0 = 0, a0 = ab;
    // one loop for both parts keeps one copy of the stages
    while (more || a0 < hi) {
        Ent e[WALK_STEPS];
        const int32_t *p = more ? up : app;
        const int32_t first = more ? s0 : a0, end = more ? nb : hi;
        CM_STEPS(
            const int32_t i = first + u * WAVE + lane();
            e[u].w = -1;
            e[u].k = k;
            if (i < end) e[u].w = p[i];
        );
        if (more) {
            CM_STEPS(
                const unsigned long long neg = more ? __ballot(e[u].w < 0) : ~0ull;
                const int32_t live = neg ? __ffsll((long long)neg) - 1 : WAVE;
                if (lane() >= live) e[u].w = -1;
                seen += live;
                if (neg) more = false;
            );
            s0 += WALK_STEPS * WAVE;
        } else {
            const int32_t got = hi - a0;
            seen += got < WALK_STEPS * WAVE ? got : WALK_STEPS * WAVE;
            a0 += WALK_STEPS * WAVE;
        }
        walk_stages(e, s1, s2, s3, s4);
#pragma unroll 1
        for (int u = 0; u < WALK_STEPS; ++u) {
            const int32_t wu = pick(e[0].w, e[1].w, e[2].w, e[3].w, u);
            if (__ballot(wu >= 0) != 0ull) fin(wu, pick(e[0].a, e[1].a, e[2].a, e[3].a, u));
        }
    }
    return seen;
}

// Team-stride over a vertex queue in batches of up to 64 entries per wave:
// a wave takes `per` consecutive entries, per = ceil(n / waves) capped at
// 64, so a queue shorter than 64 entries per wave is spread over every wave
// instead of leaving most waves idle.  fb(v) runs on the whole wave with
// lane j holding entry j of the batch (v < 0 past the end).  n must be the
// same in every thread of the team.
template <class FB>
__device__ __forceinline__ void for_batches(const Team &T, const int32_t *q, int32_t n, FB &&fb) {
    const int nw = T.nwaves();
    int per = (int)(((int64_t)n + nw - 1) / nw);
    per = per < 1 ? 1 : (per > WAVE ? WAVE : per);
    const int step = nw * per;
    for (int32_t base = T.wave() * per; base < n; base += step) {
        const int32_t i = base + lane();
        fb((lane() < per && i < n) ? q[i] : -1);
    }
}

// for_batches over a round's queue, then over what the wave itself found:
// once its share of the queue is done, the wave takes the vertices in its own
// push buffers as its next batches -- a long list alone, or the short ones
// together if they are few (a wide frontier is spread over all waves by the
// queue instead) -- as long as it has walked fewer than DEEP_STEPS steps of
// 64 entries in this round.  Cascades are order-free closures (every vertex
// is claimed, evicted or peeled exactly once through an atomic), so a vertex
// may be walked in the round that finds it.  fb(v, limit) walks the lists of
// up to `limit` entries and returns the entries it walked (uniform).
// A grid round costs about 9 us in all (barrier, first chain of reads), a wave's
// own group of steps about 3 us.  Of (4, 8), (8, 12), (12, 32) and (16, 16)
// steps and vertices, (12, 32) was taken for the long thin cascades of small
// batches, where it is 9% ahead of the next (ER 2^18, 100 edges: 1.84 ms without,
// 2.01 / 1.53 / 1.39 / 1.49 ms); on the 64-graph pool it is within 2% of the best
// (55.1 ms without, 47.6 / 46.7 / 47.5 / 47.4 ms).
constexpr int DEEP_STEPS = 12, DEEP_WIDTH = 32;
template <class FB>
__device__ __forceinline__ void for_batches_deep(const Team &T, const int32_t *q, int32_t n, Pusher &p,
                                                 FB &&fb, int deep = DEEP_STEPS, int width = DEEP_WIDTH) {
    const int nw = T.nwaves();
    int per = (int)(((int64_t)n + nw - 1) / nw);
    per = per < 1 ? 1 : (per > WAVE ? WAVE : per);
    const int step = nw * per;
    int32_t base = T.wave() * per;
    int32_t left = deep;
    for (;;) {
        int32_t v = -1, limit = p.large;
        if (base < n) {
            const int32_t i = base + lane();
            if (lane() < per && i < n) v = q[i];
            base += step;
        } else {
            if (left <= 0 || p.m.b.n + p.v.b.n == 0 || (p.m.b.n == 0 && p.v.b.n > width)) break;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // other lanes' LDS writes come first
            if (p.m.b.n > 0) {
                p.m.b.n -= 1;
                if (lane() == 0) v = p.m.b.buf[p.m.b.n];
                limit = DEEP_LIST;
            } else {
                if (lane() < p.v.b.n) v = p.v.b.buf[lane()];
                p.v.b.n = 0;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // reads done before the slots are reused
        }
        left -= (fb(v, limit) + WAVE - 1) / WAVE;
    }
}

// Flattened walk over the lists of a wave's batch: lane j holds vertex v_j
// and the number L_j of leading slots of its list to walk (0 for none).
// The lists are laid end to end and every lane takes one slot per step, so
// a batch of short and medium lists keeps all 64 lanes busy with 64 loads
// in flight instead of walking the lists one after another.  f(j, w, own)
// runs on every lane each step (it may use wave votes): j = the lane whose
// list holds the slot this lane reads (-1 when it reads none), w = the slot's
// entry (< 0 for a tombstone or none), own = the lanes that read a slot of
// THIS lane's list in this step, so that popcount(ballot(p) & own) counts p
// over this lane's slots.
template <class F>
__device__ __forceinline__ void flat_walk(const DevGraph &g, int32_t v, int32_t L, F &&f) {
    const int32_t incl = wave_incl_add(L);
    const int32_t total = __builtin_amdgcn_readlane(incl, WAVE - 1);
    const int32_t excl = incl - L;
    const int64_t off = v >= 0 ? g.off[v] : 0;  // independent of L: issues with the length load
    for (int32_t base = 0; base < total; base += WAVE) {
        const int32_t e = base + lane();
        // owner of slot e: the last lane whose list starts at or before e
        int32_t j = 0;
        for (int s = WAVE / 2; s > 0; s >>= 1) {
            const int32_t xc = __shfl(excl, j + s);
            if (xc <= e) j += s;
        }
        const int32_t xj = __shfl(excl, j);
        const int64_t oj = __shfl(off, j);
        const bool has = e < total;
        const int32_t w = has ? g.nbr[oj + (e - xj)] : -1;
        int32_t lo = excl - base, hi = incl - base;
        lo = lo < 0 ? 0 : (lo > WAVE ? WAVE : lo);
        hi = hi < 0 ? 0 : (hi > WAVE ? WAVE : hi);
        const unsigned long long own =
            hi > lo ? ((hi - lo == WAVE ? ~0ull : ((1ull << (hi - lo)) - 1ull)) << lo) : 0ull;
        f(has ? j : -1, w, own);
    }
}

// The wave's owner marks of flat_walk_st (one copy for all walks of a kernel).
__device__ __forceinline__ int32_t *mark_buf() {
    __shared__ int32_t lds_mark[COOP_THREADS / WAVE][WALK_STEPS * WAVE];
    return lds_mark[threadIdx.x / WAVE];
}

// Staged flattened walk (flat_walk, WALK_STEPS steps at a time): lane j holds
// vertex v_j, the number L_j of slots of its run in `arr` to walk and its k_j.
// fin(j, w, flags, own, oj, lo): j, w and own as f of flat_walk (j >= 0), the
// entry's flags, oj = the first slot of lane j's list and lo = the first lane
// of this step that reads from it (lanes lo .. this lane - 1 read the slots
// just before this one), for writing compacted per-list output.  The owners
// of a group's slots come from marks in LDS: every list that starts inside the
// group marks its first slot with its lane, and a running maximum spreads it
// (a binary search by shuffles cost six dependent LDS round trips per step).
// Returns the slots walked (uniform).
template <class S1, class S2, class S3, class S4, class FIN>
__device__ __forceinline__ int32_t flat_walk_st(const int32_t *arr, const DevGraph &g, int32_t v, int32_t L,
                                                int32_t k, S1 &&s1, S2 &&s2, S3 &&s3, S4 &&s4, FIN &&fin) {
    int32_t *mark = mark_buf();
    const int64_t off = v >= 0 ? g.off[v] : 0;  // independent of L: issues with the length load
    const int32_t incl = wave_incl_add(L);
    const int32_t total = __builtin_amdgcn_readlane(incl, WAVE - 1);
    const int32_t excl = incl - L;
    int32_t carry = 0;  // owner of the last slot before the group, plus one
    for (int32_t base = 0; base < total; base += WALK_STEPS * WAVE) {
        Ent e[WALK_STEPS];
        int32_t jj[WALK_STEPS];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // last group's reads come first
        CM_STEPS(mark[u * WAVE + lane()] = 0;);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (L > 0 && excl >= base && excl < base + WALK_STEPS * WAVE) mark[excl - base] = lane() + 1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        CM_STEPS(jj[u] = mark[u * WAVE + lane()];);
        CM_STEPS(
            int32_t m = wave_incl_max(jj[u]);
            m = m > carry ? m : carry;
            carry = __builtin_amdgcn_readlane(m, WAVE - 1);
            jj[u] = m - 1;
        );
        CM_STEPS(
            const int32_t i = base + u * WAVE + lane();
            const int32_t xj = __shfl(excl, jj[u]);
            const int64_t oj = __shfl(off, jj[u]);
            e[u].k = __shfl(k, jj[u]);
            e[u].w = -1;
            if (i < total) e[u].w = arr[oj + (i - xj)];
        );
        walk_stages(e, s1, s2, s3, s4);
#pragma unroll 1
        for (int u = 0; u < WALK_STEPS && base + u * WAVE < total; ++u) {
            const int32_t b0 = base + u * WAVE;
            const int32_t j = pick(jj[0], jj[1], jj[2], jj[3], u);
            const int32_t xj = __shfl(excl, j);
            const int64_t oj = __shfl(off, j);
            int32_t lo = excl - b0, hi = incl - b0;
            lo = lo < 0 ? 0 : (lo > WAVE ? WAVE : lo);
            hi = hi < 0 ? 0 : (hi > WAVE ? WAVE : hi);
            const unsigned long long own =
                hi > lo ? ((hi - lo == WAVE ? ~0ull : ((1ull << (hi - lo)) - 1ull)) << lo) : 0ull;
            fin(j, pick(e[0].w, e[1].w, e[2].w, e[3].w, u), pick(e[0].a, e[1].a, e[2].a, e[3].a, u), own, oj,
                xj - b0 > 0 ? xj - b0 : 0);
        }
    }
    return total;
}

}  // namespace cm
