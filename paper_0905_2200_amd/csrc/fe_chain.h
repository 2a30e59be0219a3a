// fe_chain.h -- counting by chains over per-type event lists: the stream
// index, its descriptors and the launchers (fe_chain.hip).  Not public.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fe_const.h"

namespace fe {

// Types an index may hold: the sort keeps three words of LDS per type in
// each wave (48 KiB at this limit).  Streams with more take the Map kernels.
constexpr int CHAIN_TYPES = 4096;
// Guard entries around every type's list, as a search reads four entries at
// once: one of INT_MIN before it, four of INT_MAX behind it.
constexpr int LIST_PAD = 4;
constexpr int LIST_EXTRA = LIST_PAD + 1;

// One type's events in the index.
struct TypeIdx {
    int start;  // first entry of its list in et / ei
    int count;  // events
    int boff;   // its bucket table in tab: nb + 2 entries
    int nb;     // buckets
    int sh;     // bucket of tick t: (t - t0) >> sh
    int t0;     // the stream's first tick
    int pad[2];
};

// Per-type event lists of a stream (in stream order) and, per type, the
// position of the first event of each power-of-two stretch of ticks.
struct ChainIdx {
    const int *et;       // ticks, with guards around each list
    const int *ei;       // stream indices, same layout
    const int *tab;      // bucket tables
    const TypeIdx *ty;   // [num_types]
};

// Device layout of an index over n events of T types, in ints.
struct IndexPlan {
    int n = 0, T = 0, nch = 0, chunk = 0;
    int64_t o_et = 0, o_ei = 0, o_tab = 0, o_ty = 0, o_hist = 0, o_off = 0, o_scan = 0, ints = 0;
};
// alone: one stream a call (the counts of a large one are scanned by many
// blocks); else one of several indexed together, each scanned by one block.
IndexPlan index_plan(int64_t n, int T, bool alone);
ChainIdx index_view(const IndexPlan &p, int *base);

// One stream to index; base_index is added to the stored indices.
struct IndexJob {
    const int *ids, *ticks;
    int n, T, chunk, nch, base_index;
    int *et, *ei, *tab, *hist, *off;
    TypeIdx *ty;
    int first_chunk, first_type;  // over the jobs before it
};
IndexJob index_job(const IndexPlan &p, const int *ids, const int *ticks, int *base, int base_index);

// Streams indexed by one launch each step: `one`, or jobs[0..njobs).
struct IndexSet {
    IndexJob one;
    const IndexJob *jobs = nullptr;  // device
    int njobs = 1;
    int chunks = 0, types = 0;  // of all jobs
    int most_types = 0, parts = 1;
    bool alone = true;
    int64_t scan = 0;           // counts of a stream indexed alone
    int *scan_scratch = nullptr;
};
// blocks a type that fill the bucket tables of a stream of T types (types: of all
// that are indexed together)
int index_parts(int n, int T, int types);
IndexSet index_set(const IndexPlan &p, const IndexJob &j, int *base);

// Candidate rows with strides: node k of candidate m has type
// ty[m*ts + k*tk], hop k (lo, hi] = lo[m*hs + k*hk], hi[m*hs + k*hk]; its
// size is len[m], or N when len is null.
struct Rows {
    const int *ty, *lo, *hi, *len;
    int ts, tk, hs, hk, N;
    int M;
};

// One stream's table to count; the two-pass form writes both outputs.
struct ChainJob {
    ChainIdx ix;
    Rows rows;
    int theta;
    int *upper;  // relaxed counts
    int *exact;  // exact counts
    int P;       // segments per candidate
    unsigned share;  // seg_share(P) (launch_chain sets it)
    int4 *seg;   // [M][P] segment results (P > 1): completions, last one's index, first
                 // event of the first chain, count of a second run (-1: none)
    // incremental form (count_io set): the events before `from`, whose tick
    // is *t_from, are counted; adds the rest to the carry
    int *count_io, *last_io;
    const int *t_from;
    int from;
};

inline unsigned seg_share(int P) { return 0xffffffffu / (unsigned)P; }

// (CHAIN_SURVIVORS: exact counts where upper, which is there already, is at least
// theta; -1 elsewhere)
enum ChainMode { CHAIN_EXACT = 0, CHAIN_RELAXED = 1, CHAIN_TWO_PASS = 2, CHAIN_SURVIVORS = 3 };

// Validates the streams and (rows.M > 0) the candidate rows into *status, and
// starts the index with the per-chunk type histograms (T = 0 in the plan:
// the checks alone); *wmax: the largest sum of hi among the candidates (may
// be null).
void launch_index_check(const IndexSet &x, const Rows &rows, int nmax, int num_types, int *status,
                        int *wmax, hipStream_t s);
// The rest of the index; the first kernel also copies *status to hstat (may be
// null), the last one zeroes *clear (not status; may be null).
void launch_index_types(const IndexSet &x, const int *status, int *hstat, hipStream_t s);
void launch_index_lists(const IndexSet &x, const int *status, int *clear, hipStream_t s);
// lam[0] = first index with tick >= ticks[from] - *wmax, lam[1] = *status
// (lam: pinned host words).
void launch_look_back(const int *ticks, int from, const int *wmax, const int *status, int *lam,
                      hipStream_t s);
// Counts every row of one job (status non-zero: nothing is written).
void launch_chain(const ChainJob &job, ChainMode mode, int nmax, const int *status,
                  hipStream_t s);
// Both counts of every row of several jobs (device array), whose rows are
// numbered first_row[0..njobs] and segments first_item[0..njobs]: job q has rows
// first_row[q] to first_row[q + 1] and P times as many segments.  (items == rows:
// P = 1 throughout.  status non-zero: every count is -1)
void launch_chains(const ChainJob *jobs, const int64_t *first_row, const int64_t *first_item,
                   int njobs, int64_t rows, int64_t items, int nmax, const int *status,
                   hipStream_t s);
// *out = the number of v[0..M) that are at least theta (status non-zero: not
// written).
void launch_count_ge(const int *v, int M, int theta, int *out, const int *status, hipStream_t s);

// ---- mining: every candidate is a frequent episode and one more node and
// hop (a join sibling), and every entry of its last shared node is met with
// all types at once

// 64-bit words of a place's masks: 64 types and a hop each
constexpr int mask_words(int T, int n_iv) { return (T + 63) / 64 * n_iv; }

// Node 1's entries of every pair (a pair's share: (first type's rank * n_iv +
// hop) * stride + the second type's place in the lists; see Seeds).
struct PairLists {
    int *t, *a, *p;
    int *n;  // [pairs] entries
    int64_t stride;
};

// Level 2: the entries and the counts of every pair of frequent types.
struct PairJob {
    ChainIdx ix;
    const int *F1;  // [nF] frequent types
    int nF;
    const int *ivlo, *ivhi;  // the interval set (device)
    int n_iv;
    PairLists sd;
    int *out;          // counts in the level's order, (a * nF + b) * n_iv + k; may be null
    const int *upper;  // set: -1 for candidates with upper < theta
    int theta;
};

// Level m + 1 from its frequent episodes of m >= 2 nodes.
struct SibJob {
    ChainIdx ix;
    const int *F;                // frequent episodes' keys, sorted, w ints each
    int w, m;                    // m nodes
    const int *order;            // the order to take them in (launch_order)
    const int64_t *first, *off;  // episode a's siblings end like F[first[a] + c]; outputs off[a] + c
    int *out;                    // counts
    const int *upper;            // set: -1 for candidates with upper < theta
    int theta;
    const uint2 *mask;  // [place][Q]
    int Q;
    const int *ivlo, *ivhi;  // the interval set (device)
    int n_iv;
    PairLists sd;
    const int *rank;  // [num_types] rank among the frequent types
    int nF;
    int words;   // (set by the launcher: mask words a wave counts)
};

void launch_masks(bool rel, const IndexPlan &p, const int *base, const int *ivlo, const int *ivhi,
                  int n_iv, uint2 *mask, hipStream_t s);
void launch_pairs(bool rel, const PairJob &j, hipStream_t s);
// The cnt episodes ordered by their last type (order: order_ints ints).
int64_t order_ints(int64_t cnt, int T);
void launch_order(const int *F, int w, int64_t cnt, int T, int *order, hipStream_t s);
// cnt episodes.
void launch_siblings(bool rel, const SibJob &j, int64_t cnt, hipStream_t s);

}  // namespace fe
