// fe_walk.h -- chains of hop-passing events over per-type lists: the wave-wide
// walk shared by the counting kernels (fe_chain.hip).
//
// A machine's lists only ever matter through chains.  Let an event of node k
// be chained to the newest chained event of node k-1 that its hop allows
// (exact: tick in [t - hi, t - lo - 1]; relaxed: an earlier event with tick
// >= t - hi), node 0's events starting a chain each, and let s be the index
// of the chain's first event.  s does not decrease along a node's chained
// events, so the newest predecessor in range is the one with the largest s;
// a completion at index r empties the lists, after which exactly the chains
// with s > r are left.  So the count is: of node N-1's chained events (s, i)
// in order, take the next one with s > r, set r = i, repeat.
//   Everything before that last step is independent per event.  The walk
// goes forward: the events chained to an entry at tick t are those of the
// next type in (t + lo, min(t + hi, t' + lo)], t' the next entry's tick
// (later ones belong to t' or after), a range of the type's list.  Hops pass
// a small share of their entries, so nearly all the work is one pass over
// node 0's events, 64 at a time.
//   Layout: a wave takes one candidate (or one shared prefix); lane k holds
// node k's list and hop, read with v_readlane.  Between stages entries wait in
// rings of 128 in LDS, and the deepest stage with a full batch goes first, so
// every batch but the last few has 64 entries and no ring overflows.  The
// walk is bound by instruction issue, nearly all of it in the source stage's
// loop, so that stage has a loop of its own with its list's values in scalar
// registers, entries wait as two positions (their ticks are read again by the
// few that get on), and everything unusual -- a crowded bucket, a tie, more
// events than the four at hand -- is behind one test.
#pragma once

#include "fe_chain.h"

namespace fe {

constexpr int QCAP = 128;  // entries a ring holds: 64 waiting and one batch's output
constexpr int FAR_TICK = 0x7fffffff;
constexpr int BEFORE = -0x7fffffff - 1;

typedef int v4i __attribute__((ext_vector_type(4), aligned(4)));

// (only where all lanes are on: in a branch that some lanes skip, the register
// may have been filled for the others alone)
__device__ __forceinline__ int rdl(int v, int k) { return __builtin_amdgcn_readlane(v, k); }
__device__ __forceinline__ unsigned long long bal(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ int below(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// A value read in a rarely taken branch has to be there when the branch ends:
// where the paths join, the wait for it would be one for every read in flight.
__device__ __forceinline__ void arrived(int &v) { asm volatile("" : "+v"(v)); }

// Lane k: node k's list and hop k.
struct NodeRow {
    int start, count, boff, nb, sh, lo, hi;
    int t0;  // (uniform)
};

// Row m of a table into lanes 0..N-1 (N returned; wave-uniform).
__device__ __forceinline__ int load_row(const ChainIdx &ix, const Rows &rows, int64_t m, NodeRow &r)
{
    const int lane = __lane_id();
    const int N = rows.len ? __builtin_amdgcn_readfirstlane(rows.len[m]) : rows.N;
    const int k = lane < N ? lane : 0;
    const TypeIdx ty = ix.ty[rows.ty[m * rows.ts + k * rows.tk]];
    r.start = ty.start;
    r.count = ty.count;
    r.boff = ty.boff;
    r.nb = ty.nb;
    r.sh = ty.sh;
    r.t0 = __builtin_amdgcn_readfirstlane(ty.t0);
    r.lo = r.hi = 0;
    if (lane < N - 1) {
        r.lo = rows.lo[m * rows.hs + lane * rows.hk];
        r.hi = rows.hi[m * rows.hs + lane * rows.hk];
    }
    return N;
}

// bucket of tick x in a list's table
__device__ __forceinline__ int bucket(int x, int t0, int sh, int nb)
{
    const int b = (x - t0) >> sh;
    return b < 0 ? 0 : b < nb ? b : nb;
}

// list[i] at a 32-bit byte offset (lists hold fewer than 2^30 entries)
__device__ __forceinline__ int at(const int *list, int i)
{
    return *(const int *)((const char *)list + (size_t)((unsigned)i << 2));
}
__device__ __forceinline__ v4i at4(const int *list, int i)
{
    return *(const v4i *)((const char *)list + (size_t)((unsigned)i << 2));
}

// What only ties and crowded buckets need: stream indices of the list looked
// into and of the entries' own, the former's length.  It is made where a wave
// needs it, as a walk has more uniform values than eight waves a SIMD leave it
// registers for, and by all lanes.
struct Spare {
    const int *ei, *own;
    int count;
};

// A hop (wave-uniform): from node k's list to the next node's.
struct Hop {
    const ChainIdx &ix;
    const NodeRow &row;
    int k;
    const int *et, *tab;  // the next list and its bucket table
    int lo, hi, nb, sh, t0;

    __device__ __forceinline__ Hop(const ChainIdx &x, const NodeRow &w, int k_)
        : ix(x), row(w), k(k_), et(x.et + rdl(w.start, k_ + 1)),
          tab(x.tab + rdl(w.boff, k_ + 1)), lo(rdl(w.lo, k_)), hi(rdl(w.hi, k_)),
          nb(rdl(w.nb, k_ + 1)), sh(rdl(w.sh, k_ + 1)), t0(w.t0)
    {
    }
    __device__ __forceinline__ Spare spare() const
    {
        return Spare{ix.ei + rdl(row.start, k + 1), ix.ei + rdl(row.start, k),
                     rdl(row.count, k + 1)};
    }
};
// the tick a hop's events start at, and its place in the table
template <bool REL> __device__ __forceinline__ int from_tick(const Hop &h, int t)
{
    return REL ? t : t + h.lo + 1;
}
template <bool REL> __device__ __forceinline__ int table_at(const Hop &h, int t)
{
    // (an event's own tick is in the table; a hop's first may be past it)
    if (REL) return at(h.tab, (t - h.t0) >> h.sh);
    const int b = (t + (h.lo + 1 - h.t0)) >> h.sh;
    return at(h.tab, b < h.nb ? b : h.nb);
}

// The first event after an entry by search: from tick x on (the entry's own
// tick, relaxed: then after it by index), in x's bucket or first behind it;
// p: where it is if v's four entries reach tick x.
template <bool REL>
__device__ __forceinline__ int start_in_bucket(const Hop &h, const Spare &sp, int t, int x, int own,
                                               v4i v, int p)
{
    const int end = at(h.tab, bucket(x, h.t0, h.sh, h.nb) + 1);  // the bucket's end
    int q = p;
    if (v[3] < x) {
        int z = end;
        while (q < z) {
            const int mid = (q + z) >> 1;
            const bool before = at(h.et, mid) < x;
            q = before ? mid + 1 : q;
            z = before ? z : mid;
        }
    }
    if constexpr (REL) {
        if (at(h.et, q) == t) {
            // (the entries of tick t end by the bucket's end)
            const int i = at(sp.own, own);
            int z = end;
            while (q < z) {
                const int mid = (q + z) >> 1;
                const bool before = at(sp.ei, mid) <= i;
                q = before ? mid + 1 : q;
                z = before ? z : mid;
            }
        }
    }
    return q;
}

// The events of the next list chained to an entry: positions [p, p + c).
// Exact: ticks in (t + lo, min(t + hi, tn + lo)]; relaxed: events after the
// entry's (own: its position), up to tick t + hi and up to the next entry's
// event (tick tn, position next).  L: the table at the first tick's bucket; v:
// four entries from there on (L <= count, and LIST_PAD guards of INT_MAX,
// which stop every search, follow a list); relaxed, indices are only read
// where ticks are equal.  skip: events of lane 0's entry that have been put
// out already.  via: own and next are places in a pair's share, and their
// positions there.
template <bool REL>
__device__ __forceinline__ void events_of(const Hop &h, bool on, int t, int tn, int own, int next,
                                          int L, v4i v, int skip, int &p, int &c,
                                          const int *via = nullptr)
{
    const int x = from_tick<REL>(h, t);
    const int tl = REL ? tn : __builtin_elementwise_add_sat(tn, h.lo);
    const int lim = tl < t + h.hi ? tl : t + h.hi;
    const int k = (v[0] < x) + (v[1] < x) + (v[2] < x) + (v[3] < x);
    const int m = (v[0] <= lim) + (v[1] <= lim) + (v[2] <= lim) + (v[3] <= lim);
    p = L + k;
    c = m > k ? m - k : 0;
    bool odd = (v[3] < x) | (v[3] <= lim);
    if constexpr (REL) {
        odd |= (v[0] == t) | (v[1] == t) | (v[2] == t) | (v[3] == t);
        odd |= (v[0] == tn) | (v[1] == tn) | (v[2] == tn) | (v[3] == tn);
    }
    c = on ? c : 0;
    odd &= on;
    if (skip) odd |= __lane_id() == 0;
    if (__builtin_expect(bal(odd) != 0, 0)) {
        const Spare sp = h.spare();
        if (odd) {
            if (REL && via) own = at(via, own);
            int q = start_in_bucket<REL>(h, sp, t, x, own, v, p);
            // (those entries were in range: the place exists)
            p = q = q + (__lane_id() == 0 ? skip : 0);
            const int in =
                REL && tn != FAR_TICK ? at(sp.own, via ? at(via, next) : next) : FAR_TICK;
            auto in_range = [&](int e) {
                const int te = at(h.et, e);
                if constexpr (REL) return (te <= lim) & ((te != tn) || at(sp.ei, e) <= in);
                else return te <= lim;
            };
            // (a guard ends every range; at most a batch is put out at once)
            int step = 4;  // entries before q are in range
            while (q + step <= sp.count && q < p + WAVE && in_range(q + step - 1)) {
                q += step;
                step *= 2;
            }
            int z = q + step <= sp.count ? q + step - 1 : sp.count;  // z is not (or the end)
            if (q >= p + WAVE) z = q;
            while (q < z) {
                const int mid = (q + z) >> 1;
                const bool r = in_range(mid);
                q = r ? mid + 1 : q;
                z = r ? z : mid;
            }
            c = q - p < WAVE ? q - p : WAVE;
        }
    }
}

// The first event after an entry (of the same arguments): its position p and
// tick (FAR_TICK if there is none).
template <bool REL>
__device__ __forceinline__ int first_after(const Hop &h, bool on, int t, int own, int L, v4i v,
                                           int &p)
{
    const int x = from_tick<REL>(h, t);
    const bool b0 = v[0] < x, b1 = v[1] < x, b2 = v[2] < x;
    int f = b0 ? v[1] : v[0];
    f = b1 ? v[2] : f;
    f = b2 ? v[3] : f;
    p = L + b0 + b1 + b2;
    bool odd = f < x;
    if constexpr (REL) odd |= f == t;
    odd &= on;
    if (__builtin_expect(bal(odd) != 0, 0)) {
        const Spare sp = h.spare();
        if (odd) {
            p = start_in_bucket<REL>(h, sp, t, x, own, v, p);
            f = at(h.et, p);
            arrived(f);
        }
    }
    return f;
}

// The first hop the other way round: the newest event of node 0's list for an
// event of node 1's (tick t, position own) -- exact, the last one by tick
// t - lo - 1; relaxed, the last one before it.  A node 1 event has one
// predecessor at most, so this way there are no ranges to lay out.
struct Back {
    const ChainIdx &ix;
    const NodeRow &row;
    const int *et, *tab;  // node 0's list (from the guard before it)
    int lo, hi, nb, sh, t0;

    __device__ __forceinline__ Back(const ChainIdx &x, const NodeRow &w)
        : ix(x), row(w), et(x.et + rdl(w.start, 0) - 1), tab(x.tab + rdl(w.boff, 0)),
          lo(rdl(w.lo, 0)), hi(rdl(w.hi, 0)), nb(rdl(w.nb, 0)), sh(rdl(w.sh, 0)), t0(w.t0)
    {
    }
    __device__ __forceinline__ Spare spare() const
    {
        return Spare{ix.ei + rdl(row.start, 0), ix.ei + rdl(row.start, 1), rdl(row.count, 0)};
    }
};
template <bool REL> __device__ __forceinline__ int to_tick(const Back &h, int t)
{
    return REL ? t : t - h.lo - 1;
}
template <bool REL> __device__ __forceinline__ int table_at(const Back &h, int t)
{
    if (REL) return at(h.tab, (t - h.t0) >> h.sh);
    const int b = (t - (h.lo + 1 + h.t0)) >> h.sh;  // (may be before it)
    return at(h.tab, b > 0 ? b : 0);
}
// Its tick (the guard's, BEFORE, if there is none), from L, the table at the
// last tick's bucket, and v, four of et from L on (the entry before the
// bucket first); POS: and its position p.
template <bool REL, bool POS>
__device__ __forceinline__ int newest_before(const Back &h, bool on, int t, int own, int L, v4i v,
                                             int &p)
{
    const int y = to_tick<REL>(h, t);
    const bool b1 = v[1] <= y, b2 = v[2] <= y, b3 = v[3] <= y;
    int f = b1 ? v[1] : v[0];
    f = b2 ? v[2] : f;
    f = b3 ? v[3] : f;
    if (POS) p = L - 1 + b1 + b2 + b3;
    // (a crowded bucket, or events of the same tick)
    bool odd = b3;
    if constexpr (REL) odd |= f == t;
    odd &= on;
    if (__builtin_expect(bal(odd) != 0, 0)) {
        const Spare sp = h.spare();
        if (odd) {
            const int i = REL ? at(sp.own, own) : 0;
            // (every event before the bucket is older)
            int q = L, z = at(h.tab, bucket(y, h.t0, h.sh, h.nb) + 1);
            while (q < z) {
                const int mid = (q + z) >> 1;
                const bool older = REL ? at(sp.ei, mid) < i : at(h.et, mid + 1) <= y;
                q = older ? mid + 1 : q;
                z = older ? z : mid;
            }
            f = at(h.et, q);
            arrived(f);
            if (POS) p = q - 1;
        }
    }
    return f;
}
// The position of that event for an event in range of it (lanes on; the
// others' own is a position too).
template <bool REL>
__device__ __forceinline__ int first_of(const ChainIdx &ix, const NodeRow &row, bool on, int own)
{
    const Back h(ix, row);
    const int t = at(ix.et + rdl(row.start, 1), own);
    const int L = table_at<REL>(h, t);
    int p;
    newest_before<REL, true>(h, on, t, own, L, at4(h.et, L), p);
    return p;
}

// Whether a row's walk starts at node 1's list, pulling.  2048 rows over lists
// of about 2e5, ms a call from node 0's / pulling, by the lists' ratio.
// Relaxed, two nodes: 2.4 / 0.7 at 1/4, 3.0 / 2.9 at 1, 1.4 / 2.9 at 2 (both
// hops are one search; the shorter list wins).  Three nodes: 2.6 / 1.4 at 1/4,
// 8.8 / 7.0 at 1, 4.7 / 2.7 at 8, 2.6 / 1.4 at 24; four: 4.5 / 3.5 at 24 (from
// node 0's the same entries of node 1 are laid out and read again).
__device__ __forceinline__ bool pulls(const NodeRow &row, int N)
{
    return N >= 2 && rdl(row.count, 1) / (N == 2 ? 1 : 32) <= rdl(row.count, 0);
}

// One wave's rings in LDS: ring q's entries as their positions in node q's
// list and their chains' first positions in the source.
constexpr int RING_INTS = 2 * QCAP;

// Entries of node 1, kept in memory for every pair (mining): their ticks
// (FAR_TICK behind the last), chains' first positions and own positions.
struct Seeds {
    const int *t, *a, *p;
};

// The source of a walk: events of node 0's list, of node 1's, pulled, or a
// pair's entries of node 1.
enum Source { FROM_FIRST, FROM_SECOND, FROM_PAIR };

// Entries of node E, in order, from the source [a, aend) (aend is either the
// source's end or past every tick that an entry wanted from [a, ...) can
// reach).  sink(n, on, t, src, own, L, v): the next n <= 64 entries, one per
// lane (on; the other lanes' values are in range too): tick, position of the
// chain's first event in the source, own position; L, v: straight from the
// source to a sink that SEARCHES node E + 1's list, that list's table at their
// buckets and four entries from there on, else L = -1.
//   FROM_SECOND with E = 0: sink.direct(pass, its lanes, position, its node 0
// event's) for every event of the source instead.  With E = 1, a sink with
// FIRSTS gets that position as src, as does sink.search(on, t, src, own, L, v)
// of one that SEARCHES.
//   E <= EMAX.  FROM_PAIR: E = EMAX where that is 1 or 2, with sink.read(on,
// src, own, in) and sink.take(n, on, in) for a batch whose ticks are in.t, and
// E > 2 else.
template <bool REL, Source SRC, int EMAX, class Sink>
__device__ __forceinline__ void walk(const ChainIdx &ix, const NodeRow &row, int E, int a,
                                     int aend, int *lds, Sink &sink, const Seeds &seed = Seeds())
{
    constexpr int S = SRC == FROM_PAIR ? 1 : 0;  // the source's node (pulled: one less)
    constexpr bool PULL = SRC == FROM_SECOND;
    if (a >= aend) return;
    const int lane = __lane_id();
    const int *src_t = SRC == FROM_PAIR ? seed.t : ix.et + rdl(row.start, PULL ? 1 : 0);
    auto place = [&](int from) { return from + lane < aend ? from + lane : aend - 1; };
    // (the source's batches in flight, each a read behind the one before:
    // while one is worked on, the next one's four entries, the table of the
    // one after it and the ticks of the third are read)
    const Hop h(ix, row, S);
    const Back bk(ix, row);
    int t0 = 0, t1 = 0, t2 = 0, L0 = -1, L1 = -1;
    v4i v0 = {0, 0, 0, 0};
    auto ticks = [&](int from) { return at(src_t, place(from < aend ? from : aend - 1)); };
    const int t_end = PULL ? 0 : at(src_t, aend);
    // the next source event's tick: the next lane's, or the next batch's first
    auto next_tick = [&](int from, int t, int t_after) {
        const int tn = __builtin_amdgcn_update_dpp(rdl(t_after, 0), t, 0x130, 0xf, 0xf, false);
        return from + lane == aend - 1 ? t_end : tn;  // (wave_shl:1)
    };
    auto look = [&](int t) {
        if constexpr (PULL) return table_at<REL>(bk, t);
        else return table_at<REL>(h, t);
    };
    const int *to_et = PULL ? bk.et : h.et;
    auto fill = [&](bool search) {
        t0 = ticks(a);
        t1 = ticks(a + WAVE);
        t2 = ticks(a + 2 * WAVE);
        if (!search) return;
        L0 = look(t0);
        L1 = look(t1);
        v0 = at4(to_et, L0);
    };
    auto next_batch = [&](bool search) {
        if (search) {
            v0 = at4(to_et, L1);
            L0 = L1;
            L1 = look(t2);
        }
        t0 = t1;
        t1 = t2;
        t2 = ticks(a + 3 * WAVE);
    };
    // whether a pulled event has a predecessor in range
    // (m: the lanes')
    auto has_first = [&](bool on, int t, int pos, int L, v4i v, int &p, unsigned long long &m) {
        const int f = newest_before<REL, true>(bk, on, t, pos, L, v, p);
        m = bal(f >= t - bk.hi) & bal(on);
        return on & (f >= t - bk.hi);
    };
    if constexpr (SRC == FROM_PAIR && EMAX == S) {
        // (what the sink reads for a batch is in flight while it takes the
        // one before, its places a batch earlier)
        typename Sink::In now, next;
        auto on_at = [&](int from) { return from + lane < aend; };
        int own = at(seed.p, place(a));
        now.t = at(src_t, place(a));
        sink.read(on_at(a), place(a), own, now);
        own = at(seed.p, place(a + WAVE < aend ? a + WAVE : aend - 1));
        for (;;) {
            const int an = a + WAVE < aend ? a + WAVE : aend - 1;
            const int a2 = a + 2 * WAVE < aend ? a + 2 * WAVE : aend - 1;
            next.t = at(src_t, place(an));
            sink.read(on_at(an), place(an), own, next);
            own = at(seed.p, place(a2));
            sink.take(aend - a < WAVE ? aend - a : WAVE, on_at(a), now);
            a += WAVE;
            if (a >= aend) return;
            now = next;
        }
    }
    if (SRC != FROM_PAIR && E == S) {
        fill(Sink::SEARCHES);
        for (;;) {
            const int pos = place(a), n = aend - a < WAVE ? aend - a : WAVE;
            const int t = t0, L = L0;
            const v4i v = v0;
            next_batch(Sink::SEARCHES);
            if constexpr (PULL) {
                int first;
                unsigned long long m;
                const bool pass = has_first(lane < n, t, pos, L, v, first, m);
                sink.direct(pass, m, pos, first);
            } else {
                sink(n, lane < n, t, pos, pos, L, v);
            }
            a += WAVE;
            if (a >= aend) return;
        }
    }
    if constexpr (EMAX == S) return;
    if constexpr (PULL && Sink::SEARCHES) {
        // (three nodes: the second hop's reads are in flight too, its table
        // beside one of the source's batches and its entries beside the next;
        // what waits for it keeps its tick and first event's position.  A
        // round is two of the source's batches: without flags for the steps,
        // 1e5 rows of two passes take 11.3 ms instead of 11.7)
        if (E == S + 1) {
            const Hop hn(ix, row, S + 1);
            int *own_q = lds, *t_q = lds + QCAP, *first_q = lds + 2 * QCAP;
            int head = 0, n1 = 0;
            int np = 0, own = 0, t = 0, first = 0, L = 0;  // the batch in flight
            v4i v = {0, 0, 0, 0};                          // (its four entries)
            auto source = [&]() {
                if (a >= aend || n1 > QCAP - WAVE) return;
                const int pos = place(a), n = aend - a < WAVE ? aend - a : WAVE;
                const int tk = t0, Lk = L0;
                const v4i vk = v0;
                next_batch(true);
                int f;
                unsigned long long m;
                const bool pass = has_first(lane < n, tk, pos, Lk, vk, f, m);
                if (pass) {
                    const int to = (head + n1 + below(m)) & (QCAP - 1);
                    own_q[to] = pos;
                    t_q[to] = tk;
                    first_q[to] = f;
                }
                __builtin_amdgcn_wave_barrier();
                n1 += __builtin_popcountll(m);
                a += WAVE;
            };
            fill(true);
            for (;;) {
                source();
                if (np) sink.search(lane < np, t, first, own, L, v);
                np = 0;
                if (n1 >= WAVE || (a >= aend && n1 > 0)) {
                    np = n1 < WAVE ? n1 : WAVE;
                    const int q = (head + (lane < np ? lane : np - 1)) & (QCAP - 1);
                    own = own_q[q];
                    t = t_q[q];
                    first = first_q[q];
                    L = table_at<REL>(hn, t);
                    head = (head + np) & (QCAP - 1);
                    n1 -= np;
                } else if (a >= aend) {
                    return;
                }
                source();
                if (np) v = at4(hn.et, L);
            }
        }
    }
    // c events from p on of each lane's entry to the ring at slot `tail`, in
    // entry order; n: entries given, nc: taken whole, tot: events put out,
    // part: events of the next entry put out in total
    auto put = [&](int *q, int tail, int n, int p, int c, int src, int skip, int &nc, int &tot,
                   int &part) {
        nc = n;
        part = 0;
        int excl;
        const unsigned long long one = bal(c == 1), many = bal(c > 1);
        if (many == 0) {
            excl = below(one);
            tot = __builtin_popcountll(one);
        } else if (bal(c > 3) == 0) {
            const unsigned long long b0 = bal((c & 1) != 0), b1 = bal((c & 2) != 0);
            excl = below(b0) + 2 * below(b1);
            tot = __builtin_popcountll(b0) + 2 * __builtin_popcountll(b1);
        } else {
            excl = 0;
            tot = WAVE + 1;
        }
        if (__builtin_expect(tot > WAVE, 0)) {
            int inc = c;
#pragma unroll
            for (int off = 1; off < WAVE; off <<= 1) {
                const int y = __shfl_up(inc, off);
                inc += lane >= off ? y : 0;
            }
            excl = inc - c;
            tot = rdl(inc, WAVE - 1);
            // entries taken whole: the first ones whose events fit a batch
            const unsigned long long cut = bal((inc > WAVE) | (c >= WAVE));
            if (cut) {
                nc = (int)__builtin_ctzll(cut);
                if (nc == 0) {
                    // (the first alone fills it: its next WAVE events, and on)
                    part = skip + WAVE;
                    tot = WAVE;
                    c = lane == 0 ? WAVE : 0;
                } else {
                    tot = rdl(inc, nc - 1);
                    c = lane < nc ? c : 0;
                }
            }
        }
        if (tot == 0) return;
        tot = __builtin_amdgcn_readfirstlane(tot);
        tail += excl;
        if (c > 0) {
            const int s = tail & (QCAP - 1);
            q[s] = p;
            q[QCAP + s] = src;
        }
        if (many)
            for (int j = 1; bal(c > j) != 0; ++j) {
                if (c > j) {
                    const int s = (tail + j) & (QCAP - 1);
                    q[s] = p + j;
                    q[QCAP + s] = src;
                }
            }
        __builtin_amdgcn_wave_barrier();
    };
    if constexpr (SRC == FROM_PAIR && EMAX == S + 1) {
        // (the same for the next node's entries, beside the source's batches)
        const int *list = ix.et + rdl(row.start, S + 1);
        int *own_q = lds, *src_q = lds + QCAP;
        int head = 0, n1 = 0, np = 0, skip = 0;
        typename Sink::In in;
        fill(true);
        for (;;) {
            if (a < aend && n1 <= QCAP - WAVE) {
                const int pos = place(a), n = aend - a < WAVE ? aend - a : WAVE;
                const int a_next = a + WAVE, Lk = L0, tk = t0, tnk = next_tick(a, t0, t1);
                const v4i vk = v0;
                next_batch(true);
                int p, c, nc, tot;
                events_of<REL>(h, lane < n, tk, tnk, pos, pos + 1, Lk, vk, skip, p, c, seed.p);
                put(own_q, head + n1, n, p, c, pos, skip, nc, tot, skip);
                n1 += tot;
                a += nc;
                if (__builtin_expect((a != a_next) & (a < aend), 0)) fill(true);
            }
            if (np) {
                sink.take(np, lane < np, in);
                np = 0;
            }
            if (n1 >= WAVE || (a >= aend && n1 > 0)) {
                np = n1 < WAVE ? n1 : WAVE;
                const int q = (head + (lane < np ? lane : np - 1)) & (QCAP - 1);
                const int own = own_q[q];
                in.t = at(list, own);
                sink.read(lane < np, src_q[q], own, in);
                head = (head + np) & (QCAP - 1);
                n1 -= np;
            } else if (a >= aend) {
                return;
            }
        }
    }
    // lane q: ring q's first slot, its entries, and how many events of its
    // first entry's range have been put out already (an entry with more than
    // a batch's worth is put out in parts); ring S+1's in scalars
    int qh = 0, qn = 0, sk = 0;
    int h1 = 0, n1 = 0, sk0 = 0;
    auto ring = [&](int q) { return lds + (q - 1 - S) * RING_INTS; };
    // a batch of ring k's entries (flush: no more will come; k == S + 1 is the
    // ring whose counters are scalars)
    auto deeper = [&](int k, bool flush) {
        const int *q = ring(k);
        const int hk = k == S + 1 ? h1 : rdl(qh, k), ck = k == S + 1 ? n1 : rdl(qn, k);
        int n = (flush || k == E) ? ck : ck - 1;
        n = n < WAVE ? n : WAVE;
        const int i0 = lane < ck ? lane : ck - 1, i1 = lane + 1 < ck ? lane + 1 : ck - 1;
        const int s0 = (hk + i0) & (QCAP - 1), s1 = (hk + i1) & (QCAP - 1);
        // (a pulled source's entries keep their ticks, if not their firsts)
        const bool kept = PULL && !Sink::FIRSTS && k == S + 1;
        const int own = q[s0], q0 = q[QCAP + s0];
        const int *list = ix.et + rdl(row.start, k);
        const int src = kept ? own : q0;
        const int t = kept ? q0 : at(list, own);
        const bool on = lane < n;
        int nc = n;
        if (EMAX == S + 1 || k == E) {
            sink(n, on, t, src, own, -1, v4i{0, 0, 0, 0});
        } else {
            const Hop h(ix, row, k);
            const int next = q[s1];
            const int tn = lane + 1 >= ck ? FAR_TICK : kept ? q[QCAP + s1] : at(list, next);
            const int skip = rdl(sk, k);
            const int L = table_at<REL>(h, t);
            int p, c, tot, part;
            events_of<REL>(h, on, t, tn, own, next, L, at4(h.et, L), skip, p, c);
            put(ring(k + 1), rdl(qh, k + 1) + rdl(qn, k + 1), n, p, c, src, skip, nc, tot, part);
            qn = lane == k + 1 ? qn + tot : qn;
            sk = lane == k ? part : sk;
        }
        if (k == S + 1) {
            h1 = (h1 + nc) & (QCAP - 1);
            n1 -= nc;
        } else {
            qh = lane == k ? (qh + nc) & (QCAP - 1) : qh;
            qn = lane == k ? qn - nc : qn;
        }
    };
    const int full1 = E == S + 1 ? WAVE : WAVE + 1;
    fill(true);
    // (each stage's code once: the source, then every full batch, the deepest
    // first, and after the source's end what is left, from the source on -- a
    // stage's entries are its last when every stage before it is done)
    for (;;) {
        const bool more = a < aend;
        if (more) {
            const int pos = place(a), n = aend - a < WAVE ? aend - a : WAVE;
            const int a_next = a + WAVE, L_now = L0, t_now = t0;
            const int tn_now = PULL ? 0 : next_tick(a, t0, t1);
            const v4i v_now = v0;
            next_batch(true);
            int nc, tot, part;
            if constexpr (PULL) {
                int first;
                unsigned long long m;
                const bool pass = has_first(lane < n, t_now, pos, L_now, v_now, first, m);
                if (pass) {
                    int *q = ring(S + 1);
                    const int to = (h1 + n1 + below(m)) & (QCAP - 1);
                    q[to] = pos;
                    q[QCAP + to] = Sink::FIRSTS ? first : t_now;
                }
                __builtin_amdgcn_wave_barrier();
                nc = n;
                tot = __builtin_popcountll(m);
                part = 0;
            } else {
                int p, c;
                events_of<REL>(h, lane < n, t_now, tn_now, pos, pos + 1, L_now, v_now, sk0, p, c,
                               seed.p);
                put(ring(S + 1), h1 + n1, n, p, c, pos, sk0, nc, tot, part);
            }
            n1 += tot;
            sk0 = part;
            a += nc;
            if (__builtin_expect((a != a_next) & (a < aend), 0)) fill(true);
            if (n1 < full1 && a < aend) continue;
        }
        for (;;) {
            const bool end = a >= aend;
            const unsigned long long ready =
                EMAX == S + 1 ? 0 : bal(qn >= (lane == E ? WAVE : WAVE + 1));
            int k;
            bool flush = false;
            if (ready) {
                k = 63 - __builtin_clzll(ready);
            } else if (n1 >= full1) {
                k = S + 1;
            } else if (!end) {
                break;
            } else if (n1 > 0) {
                k = S + 1;
                flush = true;
            } else {
                const unsigned long long some = EMAX == S + 1 ? 0 : bal(qn > 0);
                if (!some) return;
                k = (int)__builtin_ctzll(some);
                flush = true;
            }
            deeper(k, flush);
        }
    }
}

}  // namespace fe
