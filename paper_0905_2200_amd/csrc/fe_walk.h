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
// every batch but the last few has 64 entries and no ring overflows.
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

// A lane's place in a list: entries L..L+3, of which the first k come before
// the wanted one at p = L + k.
struct Place {
    int L, k;
    v4i v;  // ticks
    __device__ __forceinline__ int p() const { return L + k; }
    __device__ __forceinline__ int tick() const
    {
        return k == 0 ? v[0] : k == 1 ? v[1] : k == 2 ? v[2] : v[3];
    }
};

// bucket of tick x >= t0 in a list's table
__device__ __forceinline__ int bucket(int x, int t0, int sh, int nb)
{
    const int b = (x - t0) >> sh;
    return b < nb ? b : nb;
}

// First entry of the list with tick >= x.  L0: the list's table at x's
// bucket b.  Bounds: L0 <= count and LIST_PAD guards follow the list, so the
// four entries read always exist; the guards (INT_MAX) stop every search.
//   REL: the first entry after the event at ei[self], whose tick is x; only
// entries of the same tick can come before it, so indices are read there
// alone (the stream's indices are half of its lists' bytes).
template <bool REL>
__device__ __forceinline__ void find(const ChainIdx &ix, int start, int boff, int b, int L0,
                                     bool on, int x, int self, Place &pl)
{
    pl.L = L0;
    pl.v = *(const v4i *)(ix.et + start + L0);
    pl.k = (pl.v[0] < x) + (pl.v[1] < x) + (pl.v[2] < x) + (pl.v[3] < x);
    const bool slow = on & (pl.k == 4);
    if (__builtin_expect(bal(slow) != 0, 0)) {
        // a crowded bucket: binary search in the rest of it
        if (slow) {
            int lo = L0 + 4, hi = ix.tab[boff + b + 1];
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                const bool before = ix.et[start + mid] < x;
                lo = before ? mid + 1 : lo;
                hi = before ? hi : mid;
            }
            pl.L = lo;
            pl.k = 0;
            pl.v = *(const v4i *)(ix.et + start + lo);
        }
    }
    pl.k = pl.k < 4 ? pl.k : 3;  // (lanes off)
    if constexpr (REL) {
        const bool tie = on & (pl.tick() == x);
        if (__builtin_expect(bal(tie) != 0, 0)) {
            // (the entries of tick x end by the bucket's end)
            if (tie) {
                const int i = ix.ei[self];
                int lo = pl.p(), hi = ix.tab[boff + b + 1];
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    const bool before = ix.ei[start + mid] <= i;
                    lo = before ? mid + 1 : lo;
                    hi = before ? hi : mid;
                }
                pl.L = lo;
                pl.k = 0;
                pl.v = *(const v4i *)(ix.et + start + lo);
            }
        }
    }
}

// One wave's rings in LDS: ring q (1..) at base + (q-1)*ring_ints: ticks,
// positions of the chains' first events in node 0's list and, where something
// asks for it (the relaxed counter's ties, the siblings' masks), the entries'
// positions in their own list.
__host__ __device__ constexpr int ring_ints(bool third) { return QCAP * (third ? 3 : 2); }

// Entries of node 1, kept in memory for every pair (mining): their ticks,
// chains' first positions and own positions.
struct Seeds {
    const int *t, *a, *p;
};

// Entries of node E, in order, from the source [a, aend): node 0's events of
// the row's first list (aend is either the list's end or past every tick that
// an entry wanted from [a, ...) can reach), or, SEED, all of a pair's entries
// of node 1.  sink(n, on, t, apos, own, first, L0): the next n <= 64 entries,
// one per lane (on): tick, position of the chain's first event in node 0's
// list, own position (POS); first: straight from the source, L0 then being
// the next list's table at their buckets.
template <bool REL, bool POS, bool SEED, class Sink>
__device__ __forceinline__ void walk(const ChainIdx &ix, const NodeRow &row, int E, int a,
                                     int aend, int *lds, Sink &sink, const Seeds &seed = Seeds())
{
    static_assert(POS || !REL, "the relaxed counter's ties need the positions");
    constexpr int S = SEED ? 1 : 0;  // the source's node
    const int lane = __lane_id();
    const int start0 = rdl(row.start, 0);
    auto ring = [&](int q) { return lds + (q - 1 - S) * ring_ints(POS); };
    // lane q: ring q's first slot, its entries, and how many events of its
    // first entry's range have been put out already (an entry with more than
    // a batch's worth is put out in parts)
    int qh = 0, qn = 0, sk = 0;
    // the next batch of node 0's events, loaded while this one is worked on
    int pa = -1, pt = 0, ptn = 0, pL = 0;
    const int x0 = REL ? 0 : rdl(row.lo, S) + 1;
    const int boff1 = rdl(row.boff, S + 1), nb1 = rdl(row.nb, S + 1), sh1 = rdl(row.sh, S + 1);
    auto load_t = [&](int at) {
        const int pos = at + lane < aend ? at + lane : aend - 1;
        if constexpr (SEED) {
            pt = seed.t[pos];
            ptn = pos + 1 < aend ? seed.t[pos + 1] : FAR_TICK;
        } else {
            pt = ix.et[start0 + pos];
            ptn = ix.et[start0 + pos + 1];
        }
    };
    auto load_L = [&] { pL = ix.tab[boff1 + bucket(pt + x0, row.t0, sh1, nb1)]; };
    for (;;) {
        int k;
        bool flush = false;
        const unsigned long long ready = bal(qn >= (lane == E ? WAVE : WAVE + 1));
        if (ready) {
            k = 63 - __builtin_clzll(ready);
        } else if (a < aend) {
            k = S;
        } else {
            const unsigned long long some = bal(qn > 0);
            if (!some) break;
            // (every stage before it is done: its entries are the last ones)
            k = (int)__builtin_ctzll(some);
            flush = true;
        }
        int t, tn = FAR_TICK, apos, own = 0, next = 0, n, L0 = 0;
        if (k == S) {
            n = aend - a < WAVE ? aend - a : WAVE;
            if (pa != a) {
                load_t(a);
                if (!SEED || E > S) load_L();
            }
            t = pt;
            tn = ptn;
            L0 = pL;
            apos = a + lane < aend ? a + lane : aend - 1;
            if constexpr (SEED) {
                if (E == S) own = seed.p[apos];
                apos = seed.a[apos];
            } else {
                own = apos;
                next = apos + 1;
            }
            pa = a + WAVE;
            if (pa < aend) load_t(pa);
        } else {
            const int h = rdl(qh, k), c = rdl(qn, k);
            const int *q = ring(k);
            n = (flush || k == E) ? c : c - 1;
            n = n < WAVE ? n : WAVE;
            const int s0 = (h + lane) & (QCAP - 1), s1 = (h + lane + 1) & (QCAP - 1);
            t = q[s0];
            apos = q[QCAP + s0];
            if (lane + 1 < c) tn = q[s1];
            if constexpr (POS) own = q[2 * QCAP + s0];
            if constexpr (REL) next = q[2 * QCAP + s1];
        }
        bool on = lane < n;
        if (k == E) {
            sink(n, on, t, apos, own, k == S, L0);
            if (k == S) {
                a += n;
            } else {
                qh = lane == k ? (qh + n) & (QCAP - 1) : qh;
                qn = lane == k ? qn - n : qn;
            }
            if (!SEED && k == S && pa < aend) load_L();
            continue;
        }
        const int lo = rdl(row.lo, k), hi = rdl(row.hi, k);
        const int start = rdl(row.start, k + 1), boff = rdl(row.boff, k + 1);
        t = on ? t : row.t0;
        const int x = REL ? t : t + lo + 1;
        int lim = t + hi;
        const int tl = REL || tn == FAR_TICK ? tn : tn + lo;
        lim = tl < lim ? tl : lim;
        const int b = bucket(x, row.t0, rdl(row.sh, k + 1), rdl(row.nb, k + 1));
        if (k != S) L0 = ix.tab[boff + b];
        else if (!on) L0 = 0;
        Place pl;
        find<REL>(ix, start, boff, b, L0, on, x, rdl(row.start, k) + own, pl);
        const int skip = rdl(sk, k);
        if (__builtin_expect(skip != 0, 0)) {
            if (lane == 0) {
                // (those entries were in range: the place exists)
                pl.L = pl.p() + skip;
                pl.k = 0;
                pl.v = *(const v4i *)(ix.et + start + pl.L);
            }
        }
        // events of the range among the four at hand; more: the last is one,
        // or (relaxed) one shares the next entry's tick and is in this range
        // only if it comes before that entry's event
        int c = 0;
        bool tie = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c += ((j >= pl.k) & (pl.v[j] <= lim)) ? 1 : 0;
            if constexpr (REL) tie |= (j >= pl.k) & (pl.v[j] == tn) & (pl.v[j] <= lim);
        }
        const bool more = on & ((pl.v[3] <= lim) | tie);
        c = on ? c : 0;
        if (__builtin_expect(bal(more) != 0, 0)) {
            if (more) {
                // (a guard ends every range; at most a batch is put out at once)
                const int in = REL && tn != FAR_TICK ? ix.ei[rdl(row.start, k) + next] : FAR_TICK;
                auto in_range = [&](int p) {
                    const int te = ix.et[start + p];
                    if constexpr (REL)
                        return (te <= lim) & ((te != tn) || ix.ei[start + p] <= in);
                    else return te <= lim;
                };
                const int cnt = rdl(row.count, k + 1), top = pl.p() + WAVE;
                int e = pl.p(), step = 4;  // entries before e are in range
                while (e + step <= cnt && e < top && in_range(e + step - 1)) {
                    e += step;
                    step *= 2;
                }
                int f = e + step <= cnt ? e + step - 1 : cnt;  // entry f is not (or the end)
                if (e >= top) f = e;
                while (e < f) {
                    const int mid = (e + f) >> 1;
                    const bool r = in_range(mid);
                    e = r ? mid + 1 : e;
                    f = r ? f : mid;
                }
                c = e - pl.p();
                c = c < WAVE ? c : WAVE;
            }
        }
        // the events go to ring k+1 in entry order
        int excl, tot, nc = n, put_skip = 0;
        if (bal(c > 1) == 0) {
            const unsigned long long m = bal(c != 0);
            excl = below(m);
            tot = __builtin_popcountll(m);
        } else {
            int inc = c;
#pragma unroll
            for (int off = 1; off < WAVE; off <<= 1) {
                const int y = __shfl_up(inc, off);
                inc += lane >= off ? y : 0;
            }
            excl = inc - c;
            // entries taken whole: the first ones whose events fit a batch
            const unsigned long long cut = bal(on & ((inc > WAVE) | (c >= WAVE)));
            if (cut) {
                nc = (int)__builtin_ctzll(cut);
                if (nc == 0) {
                    // (the first alone fills it: its next WAVE events, and on)
                    put_skip = skip + WAVE;
                    tot = WAVE;
                    c = lane == 0 ? WAVE : 0;
                } else {
                    tot = rdl(inc, nc - 1);
                    c = lane < nc ? c : 0;
                }
            } else {
                tot = rdl(inc, WAVE - 1);
            }
        }
        if (tot) {
            int *q = ring(k + 1);
            const int tail = rdl(qh, k + 1) + rdl(qn, k + 1) + excl;
            if (c > 0) {
                const int s0 = tail & (QCAP - 1);
                q[s0] = pl.tick();
                q[QCAP + s0] = apos;
                if constexpr (POS) q[2 * QCAP + s0] = pl.p();
            }
            for (int j = 1; bal(c > j) != 0; ++j) {
                if (c > j) {
                    const int s0 = (tail + j) & (QCAP - 1);
                    q[s0] = ix.et[start + pl.p() + j];
                    q[QCAP + s0] = apos;
                    if constexpr (POS) q[2 * QCAP + s0] = pl.p() + j;
                }
            }
            qn = lane == k + 1 ? qn + tot : qn;
            __builtin_amdgcn_wave_barrier();
        }
        sk = lane == k ? put_skip : sk;
        if (k == S) {
            a += nc;
        } else {
            qh = lane == k ? (qh + nc) & (QCAP - 1) : qh;
            qn = lane == k ? qn - nc : qn;
        }
        if (k == S && pa < aend) load_L();
    }
}

}  // namespace fe
