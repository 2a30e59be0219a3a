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

typedef int v4i __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ int rdl(int v, int k) { return __builtin_amdgcn_readlane(v, k); }
__device__ __forceinline__ unsigned long long bal(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ int below(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

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

// bucket of tick x >= t0 in a list's table
__device__ __forceinline__ int bucket(int x, int t0, int sh, int nb)
{
    const int b = (x - t0) >> sh;
    return b < nb ? b : nb;
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

// A hop (wave-uniform): from node k's list to the next node's.
struct Hop {
    const int *et, *ei;    // the next list
    const int *tab;        // its bucket table
    const int *own;        // stream indices of node k's list
    int lo, hi, count, nb, sh, t0;
};
__device__ __forceinline__ Hop hop_of(const ChainIdx &ix, const NodeRow &row, int k)
{
    Hop h;
    const int start = rdl(row.start, k + 1);
    h.et = ix.et + start;
    h.ei = ix.ei + start;
    h.tab = ix.tab + rdl(row.boff, k + 1);
    h.own = ix.ei + rdl(row.start, k);
    h.lo = rdl(row.lo, k);
    h.hi = rdl(row.hi, k);
    h.count = rdl(row.count, k + 1);
    h.nb = rdl(row.nb, k + 1);
    h.sh = rdl(row.sh, k + 1);
    h.t0 = row.t0;
    return h;
}
// the tick a hop's events start at, and its place in the table
template <bool REL> __device__ __forceinline__ int from_tick(const Hop &h, int t)
{
    return REL ? t : t + h.lo + 1;
}
template <bool REL> __device__ __forceinline__ int table_at(const Hop &h, int t)
{
    return at(h.tab, bucket(from_tick<REL>(h, t), h.t0, h.sh, h.nb));
}

// The events of the next list chained to an entry: positions [p, p + c).
// Exact: ticks in (t + lo, min(t + hi, tn + lo)]; relaxed: events after the
// entry's (own: its position), up to tick t + hi and up to the next entry's
// event (tick tn, position next).  FIRST: the next entry is left out of it and
// c only tells whether there is an event.  L: the table at the first tick's
// bucket; v: four entries from there on (L <= count, and LIST_PAD guards of
// INT_MAX, which stop every search, follow a list); relaxed, indices are only
// read where ticks are equal.  skip: events of lane 0's entry that have been
// put out already.
template <bool REL, bool FIRST>
__device__ __forceinline__ void events_of(const Hop &h, bool on, int t, int tn, int own, int next,
                                          int L, v4i v, int skip, int &p, int &c)
{
    const int x = from_tick<REL>(h, t);
    int lim = t + h.hi;
    if constexpr (!FIRST) {
        const int tl = REL ? tn : __builtin_elementwise_add_sat(tn, h.lo);
        lim = tl < lim ? tl : lim;
    }
    const int k = (v[0] < x) + (v[1] < x) + (v[2] < x) + (v[3] < x);
    const int m = (v[0] <= lim) + (v[1] <= lim) + (v[2] <= lim) + (v[3] <= lim);
    p = L + k;
    c = m > k ? m - k : 0;
    bool odd = v[3] < x;
    if constexpr (!FIRST) odd |= v[3] <= lim;
    if constexpr (REL) {
        odd |= (v[0] == t) | (v[1] == t) | (v[2] == t) | (v[3] == t);
        if constexpr (!FIRST) odd |= (v[0] == tn) | (v[1] == tn) | (v[2] == tn) | (v[3] == tn);
    }
    c = on ? c : 0;
    odd &= on;
    if (skip) odd |= __lane_id() == 0;
    if (__builtin_expect(bal(odd) != 0, 0)) {
        if (odd) {
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
                    const int i = at(h.own, own);
                    int z = end;
                    while (q < z) {
                        const int mid = (q + z) >> 1;
                        const bool before = at(h.ei, mid) <= i;
                        q = before ? mid + 1 : q;
                        z = before ? z : mid;
                    }
                }
            }
            if constexpr (FIRST) {
                p = q;
                c = at(h.et, q) <= lim ? 1 : 0;
            } else {
                // (those entries were in range: the place exists)
                p = q = q + (__lane_id() == 0 ? skip : 0);
                const int in = REL && tn != FAR_TICK ? at(h.own, next) : FAR_TICK;
                auto in_range = [&](int e) {
                    const int te = at(h.et, e);
                    if constexpr (REL) return (te <= lim) & ((te != tn) || at(h.ei, e) <= in);
                    else return te <= lim;
                };
                // (a guard ends every range; at most a batch is put out at once)
                int step = 4;  // entries before q are in range
                while (q + step <= h.count && q < p + WAVE && in_range(q + step - 1)) {
                    q += step;
                    step *= 2;
                }
                int z = q + step <= h.count ? q + step - 1 : h.count;  // z is not (or the end)
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
}

// One wave's rings in LDS: ring q's entries as their positions in node q's
// list and their chains' first positions in the source.
constexpr int RING_INTS = 2 * QCAP;

// Entries of node 1, kept in memory for every pair (mining): their ticks
// (FAR_TICK behind the last), chains' first positions and own positions.
struct Seeds {
    const int *t, *a, *p;
};

// Entries of node E, in order, from the source [a, aend): node 0's events of
// the row's first list (aend is either the list's end or past every tick that
// an entry wanted from [a, ...) can reach), or, SEED, all of a pair's entries
// of node 1.  sink(n, on, t, src, own, L, v): the next n <= 64 entries, one per
// lane (on; the other lanes' values are in range too): tick, position of the
// chain's first event in the source, own position; L, v: straight from the
// source to a sink that SEARCHES node E + 1's list, that list's table at their
// buckets and four entries from there on, else L = -1.
template <bool REL, bool SEED, class Sink>
__device__ __forceinline__ void walk(const ChainIdx &ix, const NodeRow &row, int E, int a,
                                     int aend, int *lds, Sink &sink, const Seeds &seed = Seeds())
{
    constexpr int S = SEED ? 1 : 0;  // the source's node
    if (a >= aend) return;
    const int lane = __lane_id();
    const int *src_t = SEED ? seed.t : ix.et + rdl(row.start, 0);
    auto place = [&](int from) { return from + lane < aend ? from + lane : aend - 1; };
    // (the source's batches in flight, each a read behind the one before:
    // while one is worked on, the next one's four entries, the table of the
    // one after it and the ticks of the third are read)
    const Hop h = hop_of(ix, row, S);
    int t0 = 0, tn0 = 0, t1 = 0, tn1 = 0, t2 = 0, tn2 = 0, L0 = -1, L1 = -1;
    v4i v0 = {0, 0, 0, 0};
    auto ticks = [&](int from, int &t, int &tn) {
        const int np = place(from < aend ? from : aend - 1);
        t = at(src_t, np);
        tn = at(src_t, np + 1);
    };
    auto fill = [&](bool look) {
        ticks(a, t0, tn0);
        ticks(a + WAVE, t1, tn1);
        ticks(a + 2 * WAVE, t2, tn2);
        if (!look) return;
        L0 = table_at<REL>(h, t0);
        L1 = table_at<REL>(h, t1);
        v0 = at4(h.et, L0);
    };
    auto next_batch = [&](bool look) {
        if (look) {
            v0 = at4(h.et, L1);
            L0 = L1;
            L1 = table_at<REL>(h, t2);
        }
        t0 = t1;
        tn0 = tn1;
        t1 = t2;
        tn1 = tn2;
        ticks(a + 3 * WAVE, t2, tn2);
    };
    if (E == S) {
        fill(Sink::SEARCHES);
        for (;;) {
            const int pos = place(a), n = aend - a < WAVE ? aend - a : WAVE;
            const int t = t0, L = L0;
            const v4i v = v0;
            next_batch(Sink::SEARCHES);
            sink(n, lane < n, t, pos, SEED ? at(seed.p, pos) : pos, L, v);
            a += WAVE;
            if (a >= aend) return;
        }
    }
    // lane q: ring q's first slot, its entries, and how many events of its
    // first entry's range have been put out already (an entry with more than
    // a batch's worth is put out in parts); ring S+1's in scalars
    int qh = 0, qn = 0, sk = 0;
    int h1 = 0, n1 = 0, sk0 = 0;
    auto ring = [&](int q) { return lds + (q - 1 - S) * RING_INTS; };
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
    // a batch of ring k's entries (flush: no more will come; k == S + 1 is the
    // ring whose counters are scalars)
    auto deeper = [&](int k, bool flush) {
        const int *q = ring(k);
        const int hk = k == S + 1 ? h1 : rdl(qh, k), ck = k == S + 1 ? n1 : rdl(qn, k);
        int n = (flush || k == E) ? ck : ck - 1;
        n = n < WAVE ? n : WAVE;
        const int i0 = lane < ck ? lane : ck - 1, i1 = lane + 1 < ck ? lane + 1 : ck - 1;
        const int s0 = (hk + i0) & (QCAP - 1), s1 = (hk + i1) & (QCAP - 1);
        const int own = q[s0], src = q[QCAP + s0];
        const int *list = ix.et + rdl(row.start, k);
        const int t = at(list, own);
        const bool on = lane < n;
        int nc = n;
        if (k == E) {
            sink(n, on, t, src, own, -1, v4i{0, 0, 0, 0});
        } else {
            const Hop h = hop_of(ix, row, k);
            const int next = q[s1];
            const int tn = lane + 1 < ck ? at(list, next) : FAR_TICK;
            const int skip = rdl(sk, k);
            const int L = table_at<REL>(h, t);
            int p, c, tot, part;
            events_of<REL, false>(h, on, t, tn, own, next, L, at4(h.et, L), skip, p, c);
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
            const int a_next = a + WAVE, L_now = L0, t_now = t0, tn_now = tn0;
            const v4i v_now = v0;
            next_batch(true);
            int own = pos, next = pos + 1;
            if constexpr (SEED && REL) {
                own = at(seed.p, pos);
                next = at(seed.p, pos + 1);  // (behind the last: not used)
            }
            int p, c, nc, tot, part;
            events_of<REL, false>(h, lane < n, t_now, tn_now, own, next, L_now, v_now, sk0, p, c);
            put(ring(S + 1), h1 + n1, n, p, c, pos, sk0, nc, tot, part);
            n1 += tot;
            sk0 = part;
            a += nc;
            if (__builtin_expect((a != a_next) & (a < aend), 0)) fill(true);
            if (n1 < full1 && a < aend) continue;
        }
        for (;;) {
            const bool end = a >= aend;
            const unsigned long long ready = bal(qn >= (lane == E ? WAVE : WAVE + 1));
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
                const unsigned long long some = bal(qn > 0);
                if (!some) return;
                k = (int)__builtin_ctzll(some);
                flush = true;
            }
            deeper(k, flush);
        }
    }
}

}  // namespace fe
