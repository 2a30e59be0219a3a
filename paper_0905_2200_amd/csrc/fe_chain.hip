// fe_chain.hip -- the stream index (per-type event lists) and the counting
// kernels that walk it (fe_walk.h).
#include <cmath>

#include "fe_chain.h"
#include "fe_internal.h"
#include "fe_walk.h"

namespace fe {

// A pointer read from memory as one to global memory (the compiler would
// otherwise go through flat accesses).
template <class T> __device__ __forceinline__ T *global_ptr(T *p)
{
    return (T *)(__attribute__((address_space(1))) T *)(unsigned long long)p;
}

// ------------------------------------------------------------------ index
// A stable counting sort by type: one wave per chunk of consecutive events
// counts its types, the counts are scanned type by type, and the wave then
// places its events; a last kernel fills each type's bucket table.
namespace {

constexpr int MAX_CHUNKS = 4096;
constexpr int SMALL_SCAN = 16384;  // counts scanned by one block
constexpr unsigned FOLD = 1u << 20;  // blocks in one dimension of a grid of lists or jobs

int64_t align64(int64_t x) { return (x + 63) & ~(int64_t)63; }

// buckets of a type with c events: at most 2c + 2 (see k_ix_types)
__host__ __device__ __forceinline__ int64_t tab_room(int64_t n, int64_t T) { return 2 * n + 4 * T; }

}  // namespace

IndexPlan index_plan(int64_t n, int T, bool alone)
{
    IndexPlan p;
    p.n = (int)n;
    p.T = T;
    int64_t chunk = (n + MAX_CHUNKS - 1) / MAX_CHUNKS;
    if (!alone) {
        // (several together: one block scans a stream's counts, 32 a thread, and
        // goes on where a chunk, which a wave walks in steps of 64, would be longer
        // than the scan.  A batch of 1e6 events a stream, us by chunks of n T / 32768
        // / these: one stream of 4096 types 1328 / 389, 32 streams 3489 / 1881; 1000
        // types 429 / 221 and 1456 / 1340; 3e5 events of 4096 types 487 / 231 and 865 /
        // 816.  Up to 4096 events longer chunks are as good: 3e5 of 200 types, 1831 /
        // 1024 events, 117 / 119 and 387 / 420)
        chunk = n * T / (32 * 1024);
        const int64_t even = (int64_t)std::sqrt((double)n * T / 64);
        if (chunk > 4096) chunk = std::max<int64_t>(4096, std::min(chunk, even));
    }
    if (chunk < 512) chunk = 512;
    p.chunk = (int)((chunk + WAVE - 1) / WAVE * WAVE);
    p.nch = (int)((n + p.chunk - 1) / p.chunk);
    int64_t o = 0;
    auto take = [&](int64_t ints) {
        const int64_t at = o;
        o += align64(ints);
        return at;
    };
    const int64_t H = (int64_t)T * p.nch;
    p.o_et = take(n + (int64_t)LIST_EXTRA * T);
    p.o_ei = take(n + (int64_t)LIST_EXTRA * T);
    p.o_tab = take(tab_room(n, T));
    p.o_ty = take((int64_t)T * (sizeof(TypeIdx) / sizeof(int)));
    p.o_hist = take(H);
    p.o_off = take(H);
    p.o_scan = take(alone && H > SMALL_SCAN ? scan_scratch_ints(H) + 1 : 0);
    p.ints = o;
    return p;
}

IndexJob index_job(const IndexPlan &p, const int *ids, const int *ticks, int *base, int base_index)
{
    IndexJob j{};
    j.ids = ids;
    j.ticks = ticks;
    j.n = p.n;
    j.T = p.T;
    j.chunk = p.chunk;
    j.nch = p.nch;
    j.base_index = base_index;
    j.et = base + p.o_et;
    j.ei = base + p.o_ei;
    j.tab = base + p.o_tab;
    j.hist = base + p.o_hist;
    j.off = base + p.o_off;
    j.ty = (TypeIdx *)(base + p.o_ty);
    return j;
}

int index_parts(int n, int T, int types)
{
    // 1024 events of a list of average length, and if blocks are to spare also
    // 16384 of one that holds the whole stream: 1e6 events of 1000 types, nine
    // tenths of them in two, 1330 -> 130 us, where one block took such a list.
    const int64_t even = T ? (int64_t)n / T / 1024 + 1 : 1;
    const int64_t one = std::min((int64_t)n / 16384 + 1, (int64_t)16384 / std::max(types, 1));
    return (int)std::min<int64_t>(std::max(even, one), 256);
}

IndexSet index_set(const IndexPlan &p, const IndexJob &j, int *base)
{
    IndexSet x;
    x.one = j;
    x.chunks = j.nch;
    x.types = x.most_types = j.T;
    x.parts = index_parts(j.n, j.T, j.T);
    x.scan = (int64_t)j.T * j.nch;
    x.scan_scratch = base + p.o_scan;
    return x;
}

ChainIdx index_view(const IndexPlan &p, int *base)
{
    ChainIdx v;
    v.et = base + p.o_et;
    v.ei = base + p.o_ei;
    v.tab = base + p.o_tab;
    v.ty = (const TypeIdx *)(base + p.o_ty);
    return v;
}

namespace {

__device__ __forceinline__ IndexJob global_job(IndexJob j)
{
    j.ids = global_ptr(j.ids);
    j.ticks = global_ptr(j.ticks);
    j.et = global_ptr(j.et);
    j.ei = global_ptr(j.ei);
    j.tab = global_ptr(j.tab);
    j.hist = global_ptr(j.hist);
    j.off = global_ptr(j.off);
    j.ty = global_ptr(j.ty);
    return j;
}

// The job of a block, by its number among all jobs' chunks or types (FIRST
// reads a job's first).
template <class First>
__device__ __forceinline__ IndexJob job_of(const IndexSet &x, int block, First first)
{
    if (!x.jobs) return global_job(x.one);
    int lo = 0, hi = x.njobs;  // the last job that starts by block
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first(x.jobs[mid]) <= block) lo = mid;
        else hi = mid;
    }
    return global_job(x.jobs[lo]);
}

// Blocks [0, chunks): stream checks (ticks non-decreasing and in range, ids
// in range) and the chunk's type counts, hist[type*nch + chunk].  Blocks
// after them: candidate checks, 64 rows each.  A read of the stream: 54 us for
// 9.7e6 events and 1e5 rows (1.5 TB/s, a chunk's 8 to 38 reads in a row).
__global__ __launch_bounds__(WAVE) void k_ix_check(IndexSet x, Rows rows, int nmax, int num_types,
                                                   int *status, int *wmax)
{
    extern __shared__ int sh[];
    const int lane = threadIdx.x;
    int bits = 0;
    if ((int)blockIdx.x < x.chunks) {
        const IndexJob j = job_of(x, blockIdx.x, [](const IndexJob &q) { return q.first_chunk; });
        const int c = (int)blockIdx.x - j.first_chunk;
        const int T = j.T, types = T ? T : num_types;
        for (int e = lane; e < T; e += WAVE) sh[e] = 0;
        __syncthreads();
        const int b = c * j.chunk, e = b + j.chunk < j.n ? b + j.chunk : j.n;
        for (int i = b + lane; i < e; i += WAVE) {
            const int id = j.ids[i], t = j.ticks[i];
            if (id < 0 || id >= types || t < 0 || t >= TICK_LIMIT) bits |= ST_RANGE;
            else if (T) atomicAdd(&sh[id], 1);
            if (i > 0 && j.ticks[i - 1] > t) bits |= ST_UNSORTED;
        }
        __syncthreads();
        for (int e2 = lane; e2 < T; e2 += WAVE) j.hist[(int64_t)e2 * j.nch + c] = sh[e2];
    } else {
        const int m = ((int)blockIdx.x - x.chunks) * WAVE + lane;
        int W = 0;
        if (m < rows.M) {
            const int N = rows.len ? rows.len[m] : rows.N;
            bool ok = N >= 1 && N <= nmax;
            int64_t w = 0;
            for (int k = 0; ok && k < N; ++k) {
                const int t = rows.ty[(int64_t)m * rows.ts + k * rows.tk];
                ok = t >= 0 && t < num_types;
                if (ok && k < N - 1) {
                    const int l = rows.lo[(int64_t)m * rows.hs + k * rows.hk];
                    const int h = rows.hi[(int64_t)m * rows.hs + k * rows.hk];
                    ok = l >= 0 && l < h && h < TICK_LIMIT;
                    w += h;
                }
            }
            if (!ok || w >= TICK_LIMIT) bits |= ST_BADCAND;
            else W = (int)w;
        }
        if (wmax) {
            for (int off = 32; off >= 1; off >>= 1) {
                const int o = __shfl_xor(W, off);
                W = o > W ? o : W;
            }
            if (lane == 0) atomicMax(wmax, W);
        }
    }
    for (int off = 32; off >= 1; off >>= 1) bits |= __shfl_xor(bits, off);
    if (bits && lane == 0) atomicOr(status, bits);
}

constexpr int TYB = 1024;  // threads of the type kernel
constexpr int TYS = 16;    // counts a thread scans at a time

// exclusive prefix of v over the block, and the block's total
__device__ __forceinline__ int64_t block_prefix(int64_t v, int64_t *sh, int64_t &tot)
{
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x >> 6;
    int64_t x = v;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const int64_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == WAVE - 1) sh[wv] = x;
    __syncthreads();
    int64_t base = 0, all = 0;
    for (int k = 0; k < TYB / WAVE; ++k) {
        base += k < wv ? sh[k] : 0;
        all += sh[k];
    }
    __syncthreads();
    tot = all;
    return base + x - v;
}

// One block a stream.  Scans the counts (hist to off) unless many blocks
// have.  Then, per type: its list's place, the buckets of its table (a power
// of two of ticks wide, so many that a bucket holds half an event to one on
// average) and the list's guards.  Bound by the latency of the scan's reads:
// for 32 streams of up to 32768 counts, 61 -> 14 us with 16 in one go.
__global__ __launch_bounds__(TYB) void k_ix_types(IndexSet x, int scan_here, const int *status,
                                                  int *hstat)
{
    __shared__ int64_t sh[TYB / WAVE];
    const int st = *status;
    if (threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0 && hstat) *hstat = st;
    if (st) return;
    const unsigned job = blockIdx.y * FOLD + blockIdx.x;
    if (job >= (unsigned)x.njobs) return;
    const IndexJob j = global_job(x.jobs ? x.jobs[job] : x.one);
    const int n = j.n, T = j.T, nch = j.nch;
    const int *hist = j.hist;
    int *off = j.off, *et = j.et, *ei = j.ei;
    TypeIdx *ty = j.ty;
    const int64_t H = (int64_t)T * nch;
    int64_t tot;
    if (scan_here) {
        // (TYS counts a thread at a time, all read at once; the room behind
        // the counts is a multiple of four)
        int64_t base = 0;
        for (int64_t b0 = 0; b0 < H; b0 += TYB * TYS) {
            const int64_t b = b0 + threadIdx.x * TYS;
            v4i v[TYS / 4];
            int s = 0;
#pragma unroll
            for (int q = 0; q < TYS / 4; ++q)
                v[q] = b + 4 * q < H ? *(const v4i *)(hist + b + 4 * q) : v4i{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < TYS; ++q) {
                const int c = b + q < H ? v[q / 4][q % 4] : 0;
                v[q / 4][q % 4] = s;
                s += c;
            }
            const int run = (int)(base + block_prefix(s, sh, tot));
            base += tot;
#pragma unroll
            for (int q = 0; q < TYS / 4; ++q)
                if (b + 4 * q < H) *(v4i *)(off + b + 4 * q) = v[q] + run;
        }
        __syncthreads();
    }
    const int t0 = n ? j.ticks[0] : 0;
    const int span = n ? j.ticks[n - 1] - t0 : 0;
    int64_t boff = 0;
    for (int e0 = 0; e0 < T; e0 += TYB) {
        const int e = e0 + threadIdx.x;
        TypeIdx x{};
        if (e < T) {
            const int a = n ? off[(int64_t)e * nch] : 0;
            const int b = n && e + 1 < T ? off[(int64_t)(e + 1) * nch] : n;
            x.start = a + LIST_EXTRA * e + 1;
            x.count = b - a;
            x.t0 = t0;
            const int64_t most = 2 * (int64_t)x.count;
            while (((int64_t)span >> x.sh) + 1 > (most > 1 ? most : 1)) ++x.sh;
            x.nb = (span >> x.sh) + 1;
            et[x.start - 1] = ei[x.start - 1] = BEFORE;
            for (int j = 0; j < LIST_PAD; ++j) {
                et[x.start + x.count + j] = FAR_TICK;
                ei[x.start + x.count + j] = FAR_TICK;
            }
        }
        const int64_t room = e < T ? (int64_t)x.nb + 2 : 0;
        const int64_t at = boff + block_prefix(room, sh, tot);
        boff += tot;
        if (e < T) {
            x.boff = (int)at;
            ty[e] = x;
        }
    }
}

// One wave per chunk: 64 events at a time, each lane's rank among the
// events of its type from a bit mask per type.  Bound by the scattered stores
// (two of 4 bytes an event, each to its own line): 280 us for 9.7e6 events of
// 256 types, the same with the next events read ahead, without the barriers'
// waits for the stores, and with neighbouring chunks on one XCD.
__global__ __launch_bounds__(WAVE) void k_ix_lists(IndexSet x, const int *status)
{
    extern __shared__ unsigned long long sm[];
    if (*status) return;
    const IndexJob j = job_of(x, blockIdx.x, [](const IndexJob &q) { return q.first_chunk; });
    const int T = j.T, n = j.n, chunk = j.chunk, nch = j.nch;
    unsigned long long *mask = sm;
    int *cur = (int *)(sm + T);
    const int lane = threadIdx.x, c = (int)blockIdx.x - j.first_chunk;
    for (int e = lane; e < T; e += WAVE) {
        mask[e] = 0;
        cur[e] = j.off[(int64_t)e * nch + c] + LIST_EXTRA * e + 1;
    }
    __syncthreads();
    const int b = c * chunk, e = b + chunk < n ? b + chunk : n;
    for (int i0 = b; i0 < e; i0 += WAVE) {
        const int i = i0 + lane;
        const bool in = i < e;
        const int id = in ? j.ids[i] : 0, t = in ? j.ticks[i] : 0;
        if (in) atomicOr(&mask[id], 1ull << lane);
        __syncthreads();
        const unsigned long long m = mask[id];
        const int rank = below(m);
        const int at = cur[id] + rank;
        __syncthreads();
        if (in) {
            j.et[at] = t;
            j.ei[at] = j.base_index + i;
            if (rank == 0) {
                cur[id] += __builtin_popcountll(m);
                mask[id] = 0;
            }
        }
        __syncthreads();
    }
}

// tab[boff + b] = events of the type before bucket b.  Each position fills
// the buckets after its predecessor's, up to its own; the end of the list
// fills the rest.  Long stretches are filled by the whole wave.  (54 us for
// 9.7e6 events of 256 types, 78 MB of tables.)
// clear (may be null): a word to zero.
__global__ __launch_bounds__(256) void k_ix_tab(IndexSet s, const int *status, int *clear)
{
    // (at the end: a store before them would take the jobs' reads off the scalar cache)
    const bool clears = clear && blockIdx.x + blockIdx.y + blockIdx.z + threadIdx.x == 0;
    if (*status) {
        if (clears) *clear = 0;
        return;
    }
    const unsigned type = blockIdx.z * FOLD + blockIdx.x;
    if (type >= (unsigned)s.types) return;
    const IndexJob j = job_of(s, (int)type, [](const IndexJob &q) { return q.first_type; });
    const TypeIdx x = j.ty[(int)type - j.first_type];
    const int *et = j.et;
    int *tab = j.tab;
    const int lane = __lane_id();
    const int w0 = (int)(blockIdx.y * (blockDim.x / WAVE) + (threadIdx.x >> 6));
    const int64_t step = (int64_t)gridDim.y * blockDim.x;
    for (int64_t p0 = (int64_t)w0 * WAVE; p0 <= x.count; p0 += step) {
        const int64_t p = p0 + lane;
        int b0 = 0, b1 = -1;  // buckets b0..b1 are this position's
        if (p <= x.count) {
            b0 = p ? ((et[x.start + p - 1] - x.t0) >> x.sh) + 1 : 0;
            b1 = p < x.count ? (et[x.start + p] - x.t0) >> x.sh : x.nb + 1;
        }
        const bool wide = b1 - b0 >= 16;
        if (!wide)
            for (int b = b0; b <= b1; ++b) tab[x.boff + b] = (int)p;
        unsigned long long m = bal(wide);
        while (m) {
            const int q = (int)__builtin_ctzll(m);
            m &= m - 1;
            const int c0 = rdl(b0, q), c1 = rdl(b1, q);
            for (int b = c0 + lane; b <= c1; b += WAVE) tab[x.boff + b] = (int)(p0 + q);
        }
    }
    if (clears) *clear = 0;
}

}  // namespace

void launch_index_check(const IndexSet &x, const Rows &rows, int nmax, int num_types, int *status,
                        int *wmax, hipStream_t s)
{
    const int cb = (rows.M + WAVE - 1) / WAVE;
    if (x.chunks + cb == 0) return;
    hipLaunchKernelGGL(k_ix_check, dim3((unsigned)(x.chunks + cb)), dim3(WAVE),
                       (size_t)x.most_types * sizeof(int), s, x, rows, nmax, num_types, status,
                       wmax);
}

void launch_index_types(const IndexSet &x, const int *status, int *hstat, hipStream_t s)
{
    const bool here = !x.alone || x.scan <= SMALL_SCAN;
    if (!here) launch_scan_excl(x.one.hist, x.scan, x.one.off, x.scan_scratch, s);
    const unsigned R = (unsigned)x.njobs;
    hipLaunchKernelGGL(k_ix_types, dim3(std::min(R, FOLD), (R - 1) / FOLD + 1), dim3(TYB), 0, s, x,
                       here ? 1 : 0, status, hstat);
}

void launch_index_lists(const IndexSet &x, const int *status, int *clear, hipStream_t s)
{
    if (x.chunks > 0)
        hipLaunchKernelGGL(k_ix_lists, dim3((unsigned)x.chunks), dim3(WAVE),
                           (size_t)x.most_types * (sizeof(unsigned long long) + sizeof(int)), s,
                           x, status);
    if (x.types == 0) return;
    // (a grid's dimension holds fewer than 2^32 threads)
    const unsigned T = (unsigned)x.types;
    const dim3 grid(std::min(T, FOLD), (unsigned)x.parts, (T - 1) / FOLD + 1);
    hipLaunchKernelGGL(k_ix_tab, grid, dim3(256), 0, s, x, status, clear);
}

namespace {
__global__ void k_look_back(const int *ticks, int from, const int *wmax, const int *status,
                            int *lam)
{
    const int st = *status;
    int a = 0, b = from;
    if (!st) {
        const int x = ticks[from] - *wmax;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if (ticks[mid] < x) a = mid + 1;
            else b = mid;
        }
    }
    lam[0] = a;
    lam[1] = st;
}
}  // namespace

void launch_look_back(const int *ticks, int from, const int *wmax, const int *status, int *lam,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_look_back, dim3(1), dim3(1), 0, s, ticks, from, wmax, status, lam);
}

// ------------------------------------------------------------------ counting
namespace {

// One block per item in a grid of two dimensions (a dimension holds fewer
// than 2^32 threads).
constexpr int64_t GRID_X = 1 << 24;
dim3 grid_of(int64_t items, int64_t z = 1)
{
    const int64_t x = items < GRID_X ? items : GRID_X;
    return dim3((unsigned)x, (unsigned)((items + x - 1) / x), (unsigned)z);
}
__device__ __forceinline__ int64_t grid_item()
{
    return (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
}

constexpr int XCDS = 8;
constexpr int FCAP = 2 * WAVE;  // completions waiting (64 and one batch's)

// Takes node N-2's entries, finds each one's first event of the last type
// and counts the completions (s, i) greedily.  Only the first event matters:
// a later one of the same entry has the same s and comes after it.
//   PULL: the source is node 1's list; node 0's events are found at the end.
//   DUAL: the same also from rf, the state the segment's own run began in;
// both runs are the same from their first common completion on.
template <bool REL, bool DUAL, bool PULL> struct Count {
    const ChainIdx &ix;
    const NodeRow &row;
    int N, a1;       // completions of chains from [.., a1) of the source count
    const Hop h;     // the last hop
    int *fq;         // FCAP (chain start, completing event) positions
    int fh = 0, fn = 0;
    int r, cnt = 0;
    int rf = -1, cntf = 0;
    int s1 = FAR_TICK;  // first event of the first completion's chain

    __device__ __forceinline__ Count(const ChainIdx &x, const NodeRow &w, int N_, int a1_, int *q,
                                     int r0)
        : ix(x), row(w), N(N_), a1(a1_), h(x, w, N_ - 2), fq(q), r(r0)
    {
    }

    // The greedy choice among 64 completions in order (valid: their lanes),
    // after one at rr: one is taken if its chain starts after the last one
    // taken.  If that is after its neighbour's completion it always is; its
    // neighbour taken, it is not, and two lanes on the same with the one
    // before; what is left goes one stretch at a time.  (A later completion of
    // a chain is not taken by the same rules.)
    __device__ __forceinline__ void choose(unsigned long long valid, int s, int i, int &rr,
                                           int &c) const
    {
        const int i1 = before(i, rr);
        unsigned long long sel = bal(s > i1) & valid;
        unsigned long long rem = valid & ~sel, no = rem & (sel << 1 | 1ull);
        rem &= ~no;
        if (rem) {
            const unsigned long long free2 = bal(s > before(i1, rr));
            for (;;) {
                const unsigned long long next = rem & (no << 1), yes = next & free2;
                rem &= ~next;
                if (yes == 0) break;
                sel |= yes;
                no = rem & (yes << 1);
                rem &= ~no;
            }
            while (rem) {
                const unsigned long long from = rem & -rem, lower = sel & (from - 1ull);
                const int last = lower ? rdl(i, 63 - __builtin_clzll(lower)) : rr;
                const unsigned long long free = bal(s > last) & valid & ~(from - 1ull);
                const unsigned long long take = free & -free;
                sel |= take;
                rem &= take ? ~(take | (take - 1ull)) : 0;
            }
        }
        c += __builtin_popcountll(sel);
        if (sel) rr = rdl(i, 63 - __builtin_clzll(sel));
    }
    // the lane's before, lane 0's: first
    static __device__ __forceinline__ int before(int v, int first)
    {
        return __builtin_amdgcn_update_dpp(first, v, 0x138, 0xf, 0xf, false);  // wave_shr:1
    }
    __device__ __forceinline__ void drain(int n)
    {
        const int lane = __lane_id();
        const bool on = lane < n;
        const int q = (fh + (on ? lane : 0)) & (FCAP - 1);
        int ap = fq[q];
        const int dp = fq[FCAP + q];
        if (PULL && N > 3) ap = first_of<REL>(ix, row, on, ap);
        const int s = at(ix.ei + rdl(row.start, 0), ap);
        const int i = at(ix.ei + rdl(row.start, N - 1), dp);
        const unsigned long long valid = bal(on);
        if (s1 == FAR_TICK) s1 = rdl(s, 0);
        choose(valid, s, i, r, cnt);
        if (DUAL) choose(valid, s, i, rf, cntf);
        fh = (fh + n) & (FCAP - 1);
        fn -= n;
    }
    __device__ __forceinline__ void finish()
    {
        if (fn) drain(fn);
    }
    static constexpr bool SEARCHES = true, FIRSTS = false;
    __device__ __forceinline__ void operator()(int, bool on, int t, int src, int own, int L, v4i v)
    {
        if (N > 2) {
            L = table_at<REL>(h, t);
            v = at4(h.et, L);
        }
        search(on, t, src, own, L, v);
    }
    __device__ __forceinline__ void search(bool on, int t, int src, int own, int L, v4i v)
    {
        int p;
        const int f = first_after<REL>(h, on, t, own, L, v, p);
        const int from = PULL && N == 3 ? own : src;
        const bool reached = f <= t + h.hi, counts = from < a1;
        take(on & reached & counts, bal(on) & bal(reached) & bal(counts), src, p);
    }
    // completions at positions p of the last list, of chains from src on
    // (m: the lanes that pass)
    __device__ __forceinline__ void take(bool pass, unsigned long long m, int src, int p)
    {
        if (m == 0) return;
        if (pass) {
            const int q = (fh + fn + below(m)) & (FCAP - 1);
            fq[q] = src;
            fq[FCAP + q] = p;
        }
        __builtin_amdgcn_wave_barrier();
        fn += __builtin_popcountll(m);
        if (fn >= WAVE) drain(WAVE);
    }
    // (two nodes, pulled: the source's own events complete; it ends at a1)
    __device__ __forceinline__ void direct(bool pass, unsigned long long m, int pos, int first)
    {
        take(pass, m, first, pos);
    }
};

// Sum of the row's hop widths (an occurrence spans at most this).
__device__ __forceinline__ int row_width(const NodeRow &row, int N)
{
    int W = 0;
    for (int k = 0; k < N - 1; ++k) W += rdl(row.hi, k);
    return W;
}

// Where the walk over chains from [.., a1) of the source (node sn's list) may
// end: past every event within W ticks of the last one (their entries bound
// those of the chains counted); a bucket's end, so possibly a few more.
__device__ __forceinline__ int look_ahead(const ChainIdx &ix, const NodeRow &row, int N, int sn,
                                          int a1)
{
    const int start = rdl(row.start, sn), count = rdl(row.count, sn);
    if (N - sn <= 2 || a1 >= count || a1 <= 0) return a1;
    const int x = ix.et[start + a1 - 1] + row_width(row, N);
    const int b = bucket(x, row.t0, rdl(row.sh, sn), rdl(row.nb, sn));
    const int e = __builtin_amdgcn_readfirstlane(ix.tab[rdl(row.boff, sn) + b + 1]);
    return e > a1 ? e : a1;
}

// Counts the chains from [a0, a1) of the source after a completion at index r
// (DUAL: and, into rf/cntf, after none).  s1: the first event of the
// first chain that completes (unless N = 1, where none can be cut off).
template <bool REL, bool DUAL, Source SRC, int EMAX>
__device__ __forceinline__ void count_from(const ChainIdx &ix, const NodeRow &row, int N, int a0,
                                           int a1, int *lds, int &r, int &cnt, int &rf, int &cntf,
                                           int &s1)
{
    constexpr int sn = SRC == FROM_SECOND ? 1 : 0;
    Count<REL, DUAL, SRC == FROM_SECOND> sink(ix, row, N, a1, lds, r);
    if (DUAL) sink.rf = rf;
    walk<REL, SRC, EMAX>(ix, row, N - 2, a0, look_ahead(ix, row, N, sn, a1), lds + 2 * FCAP, sink);
    sink.finish();
    s1 = sink.s1;
    r = sink.r;
    cnt += sink.cnt;
    if (DUAL) {
        rf = sink.rf;
        cntf += sink.cntf;
    }
}
template <bool REL, bool DUAL, int EMAX>
__device__ __forceinline__ void count_range(const ChainIdx &ix, const NodeRow &row, int N, bool pull,
                                            int a0, int a1, int *lds, int &r, int &cnt, int &rf,
                                            int &cntf, int &s1)
{
    if (a0 >= a1) return;
    if (N == 1) {
        // every event is a completion
        const int last =
            __builtin_amdgcn_readfirstlane(ix.ei[rdl(row.start, 0) + a1 - 1]);
        cnt += a1 - a0;
        r = last;
        if (DUAL) {
            cntf += a1 - a0;
            rf = last;
        }
        return;
    }
    if (pull) count_from<REL, DUAL, FROM_SECOND, EMAX>(ix, row, N, a0, a1, lds, r, cnt, rf, cntf, s1);
    else count_from<REL, DUAL, FROM_FIRST, EMAX>(ix, row, N, a0, a1, lds, r, cnt, rf, cntf, s1);
}

__host__ __device__ constexpr int chain_lds(int nmax)
{
    return 2 * FCAP + (nmax > 3 ? (nmax - 2) * RING_INTS : nmax == 3 ? 3 * QCAP : 0);
}

// Where segment p of a list of c events starts (j.share: 2^32 / P, less).
__device__ __forceinline__ int seg_at(const ChainJob &j, int c, int p)
{
    return p < j.P ? (int)__umulhi(j.share * (unsigned)p, (unsigned)c) : c;
}

// Waves a SIMD is given registers for.  Tables of up to three nodes (EMAX = 1)
// need 2.5 KB of LDS a wave, so their walks keep to eight waves' scalar
// registers, the rest of them in vector lanes: 14.5 -> 12.3 ms for the 1e5
// rows above (5.7 -> 7.6 waves resident).  Tables of four and five (EMAX = 3; 3
// and 4 KB) do so where the launch has the waves.  Eight waves' registers / the
// others', exact and relaxed ms by waves, 4 nodes: 3e5 events of 200 types, 12 000
// waves 0.175 / 0.163 and 0.194 / 0.188, 30 000 0.230 / 0.235 and 0.272 / 0.289; 1e6
// of 64 types, 24 000 waves 0.448 / 0.444 and 0.593 / 0.666, 36 000 0.577 / 0.595 and
// 0.787 / 0.866, 180 000 2.06 / 2.24 and 2.88 / 3.32; 3e6 of 128 types, 44 000 waves
// 0.453 / 0.480 and 0.555 / 0.595; 5 nodes the same.  Longer tables take the general
// kernel, whose scalar registers hold seven waves; of six nodes they have LDS for
// eight (5 KB a wave), of eight for five (7 KB).
constexpr int64_t EIGHT_WAVES = 1 << 15;
constexpr int chain_waves(int emax) { return emax <= 3 ? 8 : 1; }

// One wave per (segment, candidate).  P = 1 writes the counts; P > 1 the
// segment's own count (after no completion), its last completion's index
// and the first event of its first completed chain.
//   A batch of 64 source events is one coalesced read of their ticks and two
// of the other list (its bucket, four entries), so the kernel is bound by the
// latency of those reads at few waves and by its instructions at many (1e5
// rows of 3 nodes: 0.73 of the vector issue rate).  Why not the Map kernels'
// scan: a wave there reads every event of the stream for 64 candidates, here
// only its candidate's shorter list of the first two and the few entries that
// pass.  20011 episodes of 1-8 nodes over 3.0e5 events of 200 types: 22.6 ->
// 0.17 ms a call; 5000 relaxed of 5-8 nodes over 1.06e6 events of 128 types:
// 13.2 -> 0.30 ms; 1e5 of 3 nodes over 9.7e6 events, both passes: 81 -> 11
// ms (16.1 from node 0's list); 3000 with 9 to 19 live windows a list: 26 ->
// 0.08 ms.
template <int MODE, int EMAX>
__device__ __forceinline__ void chain_item(const ChainJob &j, int m, int p, int *lds)
{
    const int lane = __lane_id();
    NodeRow row;
    const int N = load_row(j.ix, j.rows, m, row);
    // (the incremental form starts at an event of node 0)
    const bool pull = (MODE == CHAIN_TWO_PASS || !j.count_io) && pulls(row, N);
    const int c = rdl(row.count, pull ? 1 : 0);
    int dr = -1, dc = 0, s1 = FAR_TICK;
    int a0 = 0, a1 = c, r = -1;
    if (MODE != CHAIN_TWO_PASS && j.P > 1) {
        a0 = seg_at(j, c, p);
        a1 = seg_at(j, c, p + 1);
    } else if (MODE != CHAIN_TWO_PASS && j.count_io) {
        // chains that start after the last completion, and no more than the
        // episode's width before the first new event: the others have been
        // counted or can complete at no new event
        int last = j.last_io[m];
        last = last < j.from ? last : j.from - 1;
        const int start = rdl(row.start, 0);
        const int x = j.t_from[0] - row_width(row, N);
        int hi = c;
        while (a0 < hi) {
            const int mid = (a0 + hi) >> 1;
            const bool before = (j.ix.ei[start + mid] <= last) | (j.ix.et[start + mid] < x);
            if (bal(before) != 0) a0 = mid + 1;
            else hi = mid;
        }
        r = last;
    }
    bool take = true;
    if (MODE == CHAIN_TWO_PASS) {
        int cnt = 0;
        count_range<true, false, EMAX>(j.ix, row, N, pull, a0, a1, lds, r, cnt, dr, dc, s1);
        if (lane == 0) j.upper[m] = cnt;
        take = cnt >= j.theta;
        r = -1;
    }
    int cnt = 0;
    if (take)
        count_range<MODE == CHAIN_RELAXED, false, EMAX>(j.ix, row, N, pull, a0, a1, lds, r, cnt, dr, dc, s1);
    if (lane != 0) return;
    if (MODE != CHAIN_TWO_PASS && j.P > 1) {
        j.seg[(int64_t)m * j.P + p] = make_int4(cnt, r, s1, -1);
    } else if (MODE != CHAIN_TWO_PASS && j.count_io) {
        if (cnt) {
            j.count_io[m] += cnt;
            j.last_io[m] = r;
        }
    } else {
        (MODE == CHAIN_RELAXED ? j.upper : j.exact)[m] = take ? cnt : -1;
    }
}

template <int MODE, int EMAX>
__global__ __launch_bounds__(WAVE, chain_waves(EMAX)) void k_chain(ChainJob j, const int *status,
                                                                   int log2_rows)
{
    extern __shared__ int lds[];
    if (*status) return;
    const int M = j.rows.M, b = (int)grid_item(), per_wave = 1 << log2_rows;
    const int blocks = (M + per_wave - 1) >> log2_rows;
    if (b >= blocks) return;
    // (blocks go round the XCDs: each XCD takes a stretch of the rows, whose
    // lines then come into one L2)
    const int per = blocks / XCDS;
    const int m = (b < per * XCDS ? b % XCDS * per + b / XCDS : b) << log2_rows;
    unsigned long long todo = 1;
    if (MODE == CHAIN_EXACT && j.upper) {
        // survivors only
        const int at = m + __lane_id();
        todo = bal((int)__lane_id() < per_wave && at < M && j.upper[at < M ? at : 0] >= j.theta);
    }
    for (; todo; todo &= todo - 1) {
        chain_item<MODE, EMAX>(j, m + (int)__builtin_ctzll(todo), (int)blockIdx.z, lds);
        if (MODE != CHAIN_EXACT) break;
    }
}

// Job and item of a wave among several jobs' (numbered first[0..njobs]).
__device__ __forceinline__ ChainJob job_at(const ChainJob *jobs, const int64_t *first, int njobs,
                                           int64_t item, int &at)
{
    int lo = 0, hi = njobs;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first[mid] <= item) lo = mid;
        else hi = mid;
    }
    at = (int)(item - first[lo]);
    ChainJob j = jobs[lo];
    j.ix.et = global_ptr(j.ix.et);
    j.ix.ei = global_ptr(j.ix.ei);
    j.ix.tab = global_ptr(j.ix.tab);
    j.ix.ty = global_ptr(j.ix.ty);
    j.rows.ty = global_ptr(j.rows.ty);
    j.rows.lo = global_ptr(j.rows.lo);
    j.rows.hi = global_ptr(j.rows.hi);
    j.rows.len = global_ptr(j.rows.len);
    j.upper = global_ptr(j.upper);
    j.exact = global_ptr(j.exact);
    j.seg = global_ptr(j.seg);
    j.count_io = nullptr;  // (not incremental)
    return j;
}

// The same for the rows of several jobs, each a wave.
template <int MODE, int EMAX>
__global__ __launch_bounds__(WAVE, chain_waves(EMAX)) void k_chains(const ChainJob *jobs, const int64_t *first,
                                                 int njobs, int64_t total, const int *status)
{
    extern __shared__ int lds[];
    const int64_t item = grid_item();
    if (item >= total) return;
    int m;
    if (__builtin_expect(*status != 0, 0)) {
        // (no caller waits for the checks of a batch's run)
        const ChainJob j = job_at(jobs, first, njobs, item, m);
        if (__lane_id() == 0) j.upper[m] = j.exact[m] = -1;
        return;
    }
    ChainJob j = job_at(jobs, first, njobs, item, m);
    j.seg = nullptr;
    j.P = 1;
    chain_item<MODE, EMAX>(j, m, 0, lds);
}

// One pass over the rows' segments, a wave each (a job's numbered segment by
// segment): where the jobs' rows leave the device idle, and one of them is long.
template <int MODE, int EMAX>
__global__ __launch_bounds__(WAVE, chain_waves(EMAX)) void k_chains_cut(const ChainJob *jobs,
                                                                        const int64_t *first, int njobs,
                                                                        int64_t total, const int *status)
{
    extern __shared__ int lds[];
    const int64_t item = grid_item();
    if (item >= total) return;
    int at;
    const ChainJob j = job_at(jobs, first, njobs, item, at);
    const int p = (int)((unsigned)at / (unsigned)j.rows.M), m = at - p * j.rows.M;
    int *out = MODE == CHAIN_RELAXED ? j.upper : j.exact;
    if (*status || (MODE == CHAIN_EXACT && j.upper[m] < j.theta)) {
        if (p == 0 && __lane_id() == 0) out[m] = -1;
        return;
    }
    chain_item<MODE, EMAX>(j, m, p, lds);
}

// A segment's own run, counted after no completion, stands when the first chain
// it completes starts after the last completion before it (the run would take
// it too).  Otherwise it is run again from there, a growing stretch at a time,
// until both runs take the same completion: from then on they are one.
// r: the last completion before the segment, and after it; the count returned.
// (own, own_r: the segment's own count and last completion)
template <bool REL>
__device__ __forceinline__ int run_again(const ChainJob &j, const NodeRow &row, int N, int p,
                                         int own, int own_r, int *lds, int &r)
{
    const bool pull = pulls(row, N);
    const int c = rdl(row.count, pull ? 1 : 0);
    const int a1 = seg_at(j, c, p + 1);
    int b = seg_at(j, c, p), len = WAVE;
    int cnt = 0, rf = -1, cntf = 0, s1 = 0;
    while (b < a1 && rf != r) {
        const int e = a1 - b < len ? a1 : b + len;
        count_range<REL, true, NMAX - 2>(j.ix, row, N, pull, b, e, lds, r, cnt, rf, cntf, s1);
        b = e;
        len *= 2;
    }
    if (rf != r) return cnt;
    r = own_r;
    return cnt + own - cntf;
}

// Segments' second runs, all at once: each from the last completion of the
// segments' own runs before it, which is the true one unless a run before it
// ends without having met its own.  A wave looks at 2^log2_items segments of the
// rows one after the other.  j.seg[].w: the count of a run that met its own.
//   Without it k_stitch makes them one after the other for each row, which is
// as good where the rows alone fill the device, and for few segments saves the
// launch (5000 rows, 3 segments: 0.302 / 0.299 ms with / without).  Dense
// streams have a second run at every other segment: 64 rows over 1e6 events,
// relaxed, 8 types and two nodes, 244 segments 0.15 ms, where one wave that took
// its 64 rows' second runs in order needed 1.5; 3 types at 1 kHz and five nodes,
// exact, 256 segments 28 ms against 854.
constexpr int SECOND_RUNS = 8192;  // waves that fill it
constexpr int FEW_SEGMENTS = 4;
// The second run that a segment's result (place `at` of j.seg, segment p) asks
// for; r: where it starts.
__device__ __forceinline__ bool asks_again(const ChainJob &j, int at, int p, int4 &g, int &r)
{
    g = j.seg[at];
    r = -1;
    // (behind a few segments without a completion there is hardly one that
    // matters; k_stitch takes those that do)
    for (int q = 1; g.x > 0 && q <= p && q <= FEW_SEGMENTS; ++q) {
        const int4 before = j.seg[at - q];
        if (before.x == 0) continue;
        r = before.y;
        break;
    }
    return g.x > 0 && r >= g.z;
}
template <bool REL>
__device__ __forceinline__ void again_item(const ChainJob &j, int m, int p, int x, int own_r, int r,
                                           int *lds)
{
    NodeRow row;
    const int N = load_row(j.ix, j.rows, m, row);
    const int cnt = run_again<REL>(j, row, N, p, x, own_r, lds, r);
    if (__lane_id() == 0 && r == own_r) j.seg[(int64_t)m * j.P + p].w = cnt;
}

template <bool REL>
__global__ __launch_bounds__(WAVE) void k_again(ChainJob j, const int *status, int log2_items)
{
    extern __shared__ int lds[];
    if (*status) return;
    const int lane = __lane_id(), items = j.rows.M * j.P;
    const int i = (int)blockIdx.x << log2_items;
    const int at = i + lane, m = (int)((unsigned)at / (unsigned)j.P), p = at - m * j.P;
    bool again = false;
    int4 g = make_int4(0, -1, FAR_TICK, 0);
    int r = -1;
    // (a row of the first pass alone has no segments)
    if (lane < 1 << log2_items && at < items && (REL || !j.upper || j.upper[m] >= j.theta))
        again = asks_again(j, at, p, g, r);
    for (unsigned long long todo = bal(again); todo; todo &= todo - 1) {
        const int q = (int)__builtin_ctzll(todo);
        again_item<REL>(j, rdl(m, q), rdl(p, q), rdl(g.x, q), rdl(g.y, q), rdl(r, q), lds);
    }
}
// The same for several jobs, a wave a segment.
template <bool REL>
__global__ __launch_bounds__(WAVE) void k_agains(const ChainJob *jobs, const int64_t *first,
                                                 int njobs, int64_t total, const int *status)
{
    extern __shared__ int lds[];
    const int64_t item = grid_item();
    if (item >= total || *status) return;
    int at;
    const ChainJob j = job_at(jobs, first, njobs, item, at);
    const int m = (int)((unsigned)at / (unsigned)j.P), p = at - m * j.P;
    if (j.P == 1 || (!REL && j.upper[m] < j.theta)) return;
    int4 g;
    int r;
    if (!asks_again(j, at, p, g, r)) return;
    again_item<REL>(j, m, p, g.x, g.y, r, lds);
}

// One wave per candidate: its segments' results in order, 64 at a time.  As
// long as the state is that of the last own run, the counts of those that
// stand and of the second runs that met them are only added up; a segment that
// has neither is run again here (regular gaps, whose runs need never meet: the
// row's second runs are then as long as its list).
template <bool REL> __device__ __forceinline__ void stitch_row(const ChainJob &j, int64_t m, int *lds)
{
    const int lane = __lane_id();
    int *out = REL ? j.upper : j.exact;
    if (!REL && j.upper && j.upper[m] < j.theta) {
        if (lane == 0) out[m] = -1;
        return;
    }
    NodeRow row;
    int N = 0;  // (the row is read when it is needed)
    int sum = 0, tot = 0, r = -1;
    bool same = true;  // r is the last own run's
    for (int p0 = 0; p0 < j.P; p0 += WAVE) {
        const int4 g = p0 + lane < j.P ? j.seg[m * j.P + p0 + lane] : make_int4(0, -1, FAR_TICK, 0);
        const unsigned long long some = bal(g.x > 0);
        for (int from = 0; from < WAVE;) {
            const unsigned long long on = some & (~0ull << from);
            if (!on) break;
            int b;  // the next segment that is run again
            if (same) {
                const unsigned long long lower = on & ((1ull << lane) - 1ull);
                const int before = __shfl(g.y, lower ? 63 - __builtin_clzll(lower) : 0);
                const bool stands = (lower ? before : r) < g.z;
                const unsigned long long bad = bal(!stands & (g.w < 0)) & on;
                b = bad ? (int)__builtin_ctzll(bad) : WAVE;
                sum += ((on >> lane) & 1) && lane < b ? (stands ? g.x : g.w) : 0;
                const unsigned long long done = bad ? on & ((1ull << b) - 1ull) : on;
                if (done) r = rdl(g.y, 63 - __builtin_clzll(done));
                if (!bad) break;
            } else {
                b = (int)__builtin_ctzll(on);
                if (r < rdl(g.z, b)) {
                    tot += rdl(g.x, b);
                    r = rdl(g.y, b);
                    same = true;
                    from = b + 1;
                    continue;
                }
            }
            if (N == 0) N = load_row(j.ix, j.rows, m, row);
            const int own_r = rdl(g.y, b);
            tot += run_again<REL>(j, row, N, p0 + b, rdl(g.x, b), own_r, lds, r);
            same = r == own_r;
            from = b + 1;
        }
    }
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) out[m] = tot + sum;
}

template <bool REL> __global__ __launch_bounds__(WAVE) void k_stitch(ChainJob j, const int *status)
{
    extern __shared__ int lds[];
    if (*status) return;
    const int64_t m = grid_item();
    if (m < j.rows.M) stitch_row<REL>(j, m, lds);
}
// (jobs' rows numbered first[0..njobs]; those in one segment are done)
template <bool REL>
__global__ __launch_bounds__(WAVE) void k_stitches(const ChainJob *jobs, const int64_t *first,
                                                   int njobs, int64_t total, const int *status)
{
    extern __shared__ int lds[];
    const int64_t item = grid_item();
    if (item >= total || *status) return;
    int m;
    const ChainJob j = job_at(jobs, first, njobs, item, m);
    if (j.P > 1) stitch_row<REL>(j, m, lds);
}

template <int MODE> void chain_mode(ChainJob j, int nmax, const int *status, hipStream_t s)
{
    j.share = seg_share(j.P);
    const size_t lds = (size_t)chain_lds(nmax) * sizeof(int);
    // (survivors of a first pass: a wave looks for them among several rows
    // where that leaves eight waves' worth for every place on the chip)
    int rows = 0;
    if (MODE == CHAIN_EXACT && j.P > 1 && j.upper)
        while (rows < 4 && (int64_t)j.P * j.rows.M >> (rows + 1) >= 65536) ++rows;
    const dim3 grid = grid_of((j.rows.M + (1 << rows) - 1) >> rows, j.P);
    if (nmax <= 3)
        hipLaunchKernelGGL((k_chain<MODE, 1>), grid, dim3(WAVE), lds, s, j, status, rows);
    else if (nmax <= 5 && (int64_t)j.P * j.rows.M >= EIGHT_WAVES)
        hipLaunchKernelGGL((k_chain<MODE, 3>), grid, dim3(WAVE), lds, s, j, status, rows);
    else
        hipLaunchKernelGGL((k_chain<MODE, NMAX - 2>), grid, dim3(WAVE), lds, s, j, status, rows);
    if (j.P == 1) return;
    constexpr bool REL = MODE == CHAIN_RELAXED;
    if (j.rows.M < SECOND_RUNS && j.P > FEW_SEGMENTS) {
        const int items = j.rows.M * j.P;
        int each = 0;
        while (each < 6 && items >> each > SECOND_RUNS) ++each;
        hipLaunchKernelGGL((k_again<REL>), dim3((unsigned)((items + (1 << each) - 1) >> each)),
                           dim3(WAVE), lds, s, j, status, each);
    }
    hipLaunchKernelGGL((k_stitch<REL>), grid_of(j.rows.M), dim3(WAVE), lds, s, j, status);
}

}  // namespace

namespace {
constexpr int GEB = 1024;
__global__ __launch_bounds__(GEB) void k_count_ge(const int *v, int M, int theta, int *out,
                                                  const int *status)
{
    __shared__ int part[GEB / WAVE];
    if (*status) return;
    int c = 0;
    for (int64_t i = blockIdx.x * GEB + threadIdx.x; i < M; i += gridDim.x * GEB)
        c += v[i] >= theta ? 1 : 0;
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
    if (__lane_id() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x) return;
    c = 0;
    for (int w = 0; w < GEB / WAVE; ++w) c += part[w];
    if (gridDim.x == 1) *out = c;
    else if (c) atomicAdd(out, c);
}
__global__ void k_clear(int *out, const int *status)
{
    if (*status == 0) *out = 0;
}
}  // namespace

void launch_count_ge(const int *v, int M, int theta, int *out, const int *status, hipStream_t s)
{
    // (one block needs no clearing)
    const int blocks = M <= 8 * GEB ? 1 : std::min((M + 4 * GEB - 1) / (4 * GEB), 256);
    if (blocks > 1) hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, s, out, status);
    hipLaunchKernelGGL(k_count_ge, dim3(blocks), dim3(GEB), 0, s, v, M, theta, out, status);
}

void launch_chain(const ChainJob &job, ChainMode mode, int nmax, const int *status, hipStream_t s)
{
    if (job.rows.M <= 0) return;
    if (mode == CHAIN_TWO_PASS && job.P == 1) return chain_mode<CHAIN_TWO_PASS>(job, nmax, status, s);
    ChainJob j = job;
    if (mode == CHAIN_SURVIVORS) {
        if (j.P == 1) launch_fill(j.exact, -1, j.rows.M, s);  // (else k_stitch does)
        return chain_mode<CHAIN_EXACT>(j, nmax, status, s);
    }
    if (mode != CHAIN_EXACT) chain_mode<CHAIN_RELAXED>(j, nmax, status, s);
    if (mode != CHAIN_RELAXED) {
        // (exact alone: every candidate is taken)
        if (mode == CHAIN_EXACT) j.upper = nullptr;
        chain_mode<CHAIN_EXACT>(j, nmax, status, s);
    }
}

namespace {
template <int MODE>
void chains_cut(const ChainJob *jobs, const int64_t *first_row, const int64_t *first_item,
                int njobs, int64_t rows, int64_t items, int nmax, size_t lds, const int *status,
                hipStream_t s)
{
    constexpr bool REL = MODE == CHAIN_RELAXED;
    if (nmax <= 3)
        hipLaunchKernelGGL((k_chains_cut<MODE, 1>), grid_of(items), dim3(WAVE), lds, s, jobs,
                           first_item, njobs, items, status);
    else
        hipLaunchKernelGGL((k_chains_cut<MODE, NMAX - 2>), grid_of(items), dim3(WAVE), lds, s, jobs,
                           first_item, njobs, items, status);
    hipLaunchKernelGGL((k_agains<REL>), grid_of(items), dim3(WAVE), lds, s, jobs, first_item, njobs,
                       items, status);
    hipLaunchKernelGGL((k_stitches<REL>), grid_of(rows), dim3(WAVE), lds, s, jobs, first_row, njobs,
                       rows, status);
}
}  // namespace

void launch_chains(const ChainJob *jobs, const int64_t *first_row, const int64_t *first_item,
                   int njobs, int64_t rows, int64_t items, int nmax, const int *status,
                   hipStream_t s)
{
    if (rows <= 0) return;
    const size_t lds = (size_t)chain_lds(nmax) * sizeof(int);
    if (items > rows) {
        chains_cut<CHAIN_RELAXED>(jobs, first_row, first_item, njobs, rows, items, nmax, lds,
                                  status, s);
        chains_cut<CHAIN_EXACT>(jobs, first_row, first_item, njobs, rows, items, nmax, lds, status,
                                s);
        return;
    }
    if (nmax <= 3)
        hipLaunchKernelGGL((k_chains<CHAIN_TWO_PASS, 1>), grid_of(rows), dim3(WAVE), lds, s, jobs,
                           first_row, njobs, rows, status);
    else
        hipLaunchKernelGGL((k_chains<CHAIN_TWO_PASS, NMAX - 2>), grid_of(rows), dim3(WAVE), lds, s,
                           jobs, first_row, njobs, rows, status);
}

// ------------------------------------------------------------------ siblings
namespace {

// mask[place][q], q = (type >> 6) * n_iv + h: bit (type & 63) is set where the
// type has an event in hop h's range after the event at the place (an entry of
// the lists): exact, ticks in (t + lo, t + hi]; relaxed, later events up to
// tick t + hi.  One thread per 32 types of a place and up to four hops: each
// type's list is searched once, at the ticks' narrowest start, and four entries
// from there on settle nearly every hop; the ticks ascend along a wave, so the
// reads are nearly coalesced.  Bound by those reads' latency: 0.17 ms exact and
// 0.22 ms relaxed for 1.06e6 places, 64 types and 3 hops.
constexpr int MH = 4;  // hops a thread takes
template <bool REL>
__global__ __launch_bounds__(256) void k_masks(ChainIdx ix, int places, int T, int n_iv,
                                               const int *__restrict__ ivlo,
                                               const int *__restrict__ ivhi,
                                               unsigned *__restrict__ mask, int Q)
{
    const int place = blockIdx.x * 256 + threadIdx.x;
    const int hg = (n_iv + MH - 1) / MH;
    const int h0 = blockIdx.y % hg * MH, w = blockIdx.y / hg;  // hops h0 .., types 32 w ..
    const int nh = n_iv - h0 < MH ? n_iv - h0 : MH;
    if (place >= places) return;
    const int t = ix.et[place];
    if (t == FAR_TICK || t == BEFORE) return;  // a guard
    int lo[MH], lim[MH], least = FAR_TICK;
#pragma unroll
    for (int h = 0; h < MH; ++h) {
        const int k = h0 + (h < nh ? h : 0);
        lo[h] = REL ? t : t + ivlo[k] + 1;
        lim[h] = t + ivhi[k];
        least = lo[h] < least ? lo[h] : least;
    }
    const int i = REL ? ix.ei[place] : 0;
    unsigned bits[MH] = {0, 0, 0, 0};
    const int e1 = (w + 1) * 32 < T ? (w + 1) * 32 : T;
    for (int e = w * 32; e < e1; ++e) {
        const TypeIdx ty = ix.ty[e];
        const int *et = ix.et + ty.start, *ei = ix.ei + ty.start;
        const int *tab = ix.tab + ty.boff;
        const int a = at(tab, bucket(least, ty.t0, ty.sh, ty.nb));
        const v4i v = at4(et, a);
        // relaxed: entries of tick t count from the first with a later index
        int tie = 0;
        if constexpr (REL) tie = (v[0] == t) | (v[1] == t) | (v[2] == t) | (v[3] == t);
        const unsigned bit = 1u << (e & 31);
#pragma unroll
        for (int h = 0; h < MH; ++h) {
            if (h >= nh) break;
            bool in = false;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                in |= (unsigned)(v[q] - lo[h]) <= (unsigned)(lim[h] - lo[h]);
            // (before the range still after four entries, or ties to settle)
            if ((!in & (v[3] < lo[h])) | (REL & (tie != 0))) {
                const int b = bucket(lo[h], ty.t0, ty.sh, ty.nb);
                int p = at(tab, b), z = at(tab, b + 1);
                while (p < z) {
                    const int mid = (p + z) >> 1;
                    const bool l = REL ? at(ei, mid) <= i : at(et, mid) < lo[h];
                    p = l ? mid + 1 : p;
                    z = l ? z : mid;
                }
                in = at(et, p) <= lim[h];
            }
            bits[h] |= in ? bit : 0u;
        }
    }
    for (int h = 0; h < nh; ++h)
        mask[((int64_t)place * Q + (w >> 1) * n_iv + h0 + h) * 2 + (w & 1)] = bits[h];
}

// The entries of node 1 of every pair of frequent types and interval, in the
// place of the second type's list within the pair's share; and the pair's
// count: each entry is a completion of the chain that starts at its first
// event (a chain's later ones start no later than the one taken).  An entry
// names its chain's first event by its position or, exact, where no two chains
// start at one tick, by its tick, which is then at hand where it is needed.
//   A wave a pair, bound by its instructions: 12288 pairs over 1.06e6 events of
// 64 types in 0.50 ms exact and 0.66 relaxed (0.62 and 1.25 from the first
// type's list); counting them as level 2 alone took the scan 0.95 and 3.9 ms.
template <bool REL> struct SeedOut {
    const ChainIdx &ix;
    const NodeRow &row;
    Count<REL, false, false> cnt;
    int *t, *a, *p;
    int64_t base;
    int n = 0;
    static constexpr bool SEARCHES = false, FIRSTS = true;
    __device__ __forceinline__ void direct(bool, unsigned long long, int, int) {}
    __device__ __forceinline__ void operator()(int c, bool on, int tk, int src, int own, int, v4i)
    {
        const int s = at(ix.ei + rdl(row.start, 0), src);
        const int i = at(ix.ei + rdl(row.start, 1), own);
        const int first = REL ? src : at(ix.et + rdl(row.start, 0), src);
        if (on) {
            const int64_t to = base + n + __lane_id();
            t[to] = tk;
            a[to] = first;
            p[to] = own;
        }
        cnt.choose(bal(on), s, i, cnt.r, cnt.cnt);
        n += c;
    }
};

template <bool REL, Source SRC>
__device__ __forceinline__ void pair_entries(const PairJob &j, const NodeRow &row, int64_t item,
                                             int ak, int *lds)
{
    SeedOut<REL> out{j.ix, row, Count<REL, false, false>(j.ix, row, 2, 0, nullptr, -1), j.sd.t,
                     j.sd.a, j.sd.p, (int64_t)ak * j.sd.stride + rdl(row.start, 1)};
    walk<REL, SRC, 1>(j.ix, row, 1, 0, rdl(row.count, SRC == FROM_SECOND ? 1 : 0), lds, out);
    if (__lane_id() != 0) return;
    j.sd.t[out.base + out.n] = FAR_TICK;  // (a list has its guards' room)
    j.sd.n[item] = out.n;
    if (!j.out) return;
    // in the level's order
    const int k = ak % j.n_iv, f = ak / j.n_iv, b = (int)(item % j.nF);
    const int64_t c = ((int64_t)f * j.nF + b) * j.n_iv + k;
    j.out[c] = j.upper && j.upper[c] < j.theta ? -1 : out.cnt.cnt;
}

template <bool REL>
__global__ __launch_bounds__(WAVE, 8) void k_pairs(PairJob j)
{
    extern __shared__ int lds[];
    const int64_t item = grid_item();
    if (item >= (int64_t)j.nF * j.nF * j.n_iv) return;
    const int lane = __lane_id();
    // ak = first type's rank * n_iv + k
    const int b = (int)(item % j.nF), ak = (int)(item / j.nF), k = ak % j.n_iv, f = ak / j.n_iv;
    const TypeIdx ty = j.ix.ty[lane == 1 ? j.F1[b] : j.F1[f]];
    NodeRow row;
    row.start = ty.start;
    row.count = ty.count;
    row.boff = ty.boff;
    row.nb = ty.nb;
    row.sh = ty.sh;
    row.t0 = __builtin_amdgcn_readfirstlane(ty.t0);
    row.lo = lane == 0 ? j.ivlo[k] : 0;
    row.hi = lane == 0 ? j.ivhi[k] : 0;
    if (pulls(row, 3)) pair_entries<REL, FROM_SECOND>(j, row, item, ak, lds);
    else pair_entries<REL, FROM_FIRST>(j, row, item, ak, lds);
}

// ---- 64 x 64 bits across a wave
// Lane i holds row i (bit j of the 64: column j); afterwards lane j holds
// column j (bit i: row i).  Halves are swapped between lanes 32 apart, then
// inside each 32-bit word 16-, 8-, 4-, 2- and 1-bit blocks between lanes as far
// apart.
struct Flip {
    unsigned s16, s8, r4, m4, r2, m2, r1, m1;
    __device__ __forceinline__ Flip()
    {
        const unsigned l = __lane_id();
        s16 = l & 16 ? 0x07060302u : 0x05040100u;
        s8 = l & 8 ? 0x03070105u : 0x06020400u;
        r4 = l & 4 ? 4 : 28;
        m4 = l & 4 ? 0xf0f0f0f0u : 0x0f0f0f0fu;
        r2 = l & 2 ? 2 : 30;
        m2 = l & 2 ? 0xccccccccu : 0x33333333u;
        r1 = l & 1 ? 1 : 31;
        m1 = l & 1 ? 0xaaaaaaaau : 0x55555555u;
    }
    template <int CTRL> static __device__ __forceinline__ unsigned dpp(unsigned v)
    {
        return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
    }
    static __device__ __forceinline__ unsigned mix(unsigned own, unsigned other, unsigned rot,
                                                   unsigned mask)
    {
        return (own & mask) | (__builtin_amdgcn_alignbit(other, other, rot) & ~mask);
    }
    __device__ __forceinline__ unsigned word(unsigned w) const
    {
        const auto r = __builtin_amdgcn_permlane16_swap(w, w, false, false);
        w = __builtin_amdgcn_perm(r[1], r[0], s16);
        w = __builtin_amdgcn_perm(dpp<0x128>(w), w, s8);        // lane ^ 8 (row_ror:8)
        w = mix(w, dpp<0x1b>(dpp<0x141>(w)), r4, m4);           // lane ^ 4 (mirrors of 8, of 4)
        w = mix(w, dpp<0x4e>(w), r2, m2);                       // lane ^ 2 (quad_perm)
        return mix(w, dpp<0xb1>(w), r1, m1);                    // lane ^ 1
    }
    __device__ __forceinline__ void operator()(unsigned &lo, unsigned &hi) const
    {
        const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        lo = word(r[0]);
        hi = word(r[1]);
    }
};

constexpr int QW = 4;  // mask words (64 types and a hop each) a wave counts at most
constexpr int64_t SIB_FILL = 8192;  // waves that fill the device

// Join siblings: one frequent episode's entries against 64 types at a time
// and a hop.  Of 64 entries, one per lane, the mask words (bit = type) are
// transposed, so that a lane holds, for its type, which entries have an event
// of it in range (bit = entry).  Of the entries of one chain only the first
// such can complete it, and if that one may not, none may: the lowest bit of
// each chain's stretch of bits is kept, all stretches at once (subtracting
// their first bits from the word with their last bits set borrows inside
// each stretch alone).  What is left counts, but for entries whose chain may
// start by the lane's last completion, and those are looked at one by one:
// where a chain starts within the hop's width of the last entry before it.
// The last completion is the first event in range of the last entry counted
// (tick tl), so after tl + lo (relaxed: not before tl) and by tl + hi; in
// between the event is looked up.
template <bool REL> struct Columns {
    const SibJob &j;
    const ChainIdx &ix;
    int q0, nq;                      // the words of this wave
    int start0, start_m;             // node 0's and the last shared node's lists
    int boff0, nb0, sh0, t0;         // node 0's table
    const int *seed_a;               // the source's chains' first events
    Flip flip;
    int lo[QW], hi[QW];              // the words' hops (wave-uniform)
    int cnt[QW], tl[QW], ol[QW];     // per type: completions, the last entry counted
    int t_last = -(1 << 30);
    static constexpr bool SEARCHES = false, FIRSTS = true;
    __device__ __forceinline__ void direct(bool, unsigned long long, int, int) {}
    // What a batch needs: its entries' ticks, places, chains' first events (as
    // a pair's entries name them) and mask words.
    struct In {
        int t, own, first;
        uint2 w[QW];
    };
    __device__ __forceinline__ void read(bool on, int src, int own, In &in) const
    {
        in.own = own;
        in.first = at(seed_a, src);
        const uint2 *row = j.mask + (int64_t)(start_m + own) * j.Q + q0;
#pragma unroll
        for (int q = 0; q < QW; ++q) in.w[q] = on && q < nq ? row[q] : make_uint2(0, 0);
    }
    __device__ __forceinline__ void operator()(int n, bool on, int t, int src, int own, int, v4i)
    {
        In in;
        in.t = t;
        read(on, src, own, in);
        take(n, on, in);
    }
    __device__ __forceinline__ void take(int n, bool on, const In &in)
    {
        const int lane = __lane_id();
        const int t = in.t, own = in.own;
        const int st = REL ? ix.et[start0 + in.first] : in.first;
        // chains' stretches: first and last bits, and the tick of the last
        // entry before the lane's own (a stretch that goes on from the batch
        // before has it among its own, and so within the width)
        const int before_first = __shfl_up(in.first, 1);
        const unsigned long long first = bal(in.first != before_first) | 1ull;
        const unsigned long long last = (first >> 1) | (1ull << 63);
        const int g = 63 - __builtin_clzll(first & ((2ull << lane) - 1ull));
        const int tb = __shfl(t, g > 0 ? g - 1 : 0);
        const int tp = g > 0 ? tb : t_last;
        t_last = rdl(t, n - 1);
#pragma unroll
        for (int q = 0; q < QW; ++q) {
            if (q >= nq) break;
            unsigned c0 = in.w[q].x, c1 = in.w[q].y;
            flip(c0, c1);
            {
                const unsigned long long c = c0 | (unsigned long long)c1 << 32, x = c | last;
                const unsigned long long low = c & ~(x - first);
                c0 = (unsigned)low;
                c1 = (unsigned)(low >> 32);
            }
            unsigned long long near = bal(on & (st <= tp + hi[q]));
            while (near) {
                const int e = (int)__builtin_ctzll(near);
                near &= near - 1;
                const bool has = ((e < 32 ? c0 : c1) >> (e & 31)) & 1u;
                if (bal(has) == 0) continue;
                const unsigned long long lower = (1ull << e) - 1ull;
                const unsigned b0 = c0 & (unsigned)lower, b1 = c1 & (unsigned)(lower >> 32);
                const int before = b1 ? 63 - __builtin_clz(b1) : b0 ? 31 - __builtin_clz(b0) : -1;
                const int tb = __shfl(t, before >= 0 ? before : 0);
                const int tj = before >= 0 ? tb : tl[q];
                const int te = rdl(st, e);
                bool cut = has & (te <= tj + hi[q]);
                const bool open = cut & (REL ? te >= tj : te > tj + lo[q]);
                if (bal(open) != 0) {
                    const int s = chain_start(rdl(in.first, e));
                    const int ob = __shfl(own, before >= 0 ? before : 0);
                    const int oj = before >= 0 ? ob : ol[q];
                    if (open) cut = s <= completed(q, tj, oj);
                }
                const unsigned bit = cut ? 1u << (e & 31) : 0u;
                if (e < 32) c0 &= ~bit;
                else c1 &= ~bit;
            }
            cnt[q] += __builtin_popcount(c0) + __builtin_popcount(c1);
            const int top = c1 ? 63 - __builtin_clz(c1) : c0 ? 31 - __builtin_clz(c0) : -1;
            const int tv = __shfl(t, top >= 0 ? top : 0);
            tl[q] = top >= 0 ? tv : tl[q];
            if constexpr (REL) {
                const int ov = __shfl(own, top >= 0 ? top : 0);
                ol[q] = top >= 0 ? ov : ol[q];
            }
        }
    }
    // stream index of a chain's first event (exact: the last at its tick)
    __device__ __forceinline__ int chain_start(int first) const
    {
        if (REL) return ix.ei[start0 + first];
        const int b = bucket(first, t0, sh0, nb0);
        int a = ix.tab[boff0 + b], z = ix.tab[boff0 + b + 1];
        while (a < z) {
            const int mid = (a + z) >> 1;
            const bool past = bal(ix.et[start0 + mid] > first) != 0;
            a = past ? a : mid + 1;
            z = past ? mid : z;
        }
        return ix.ei[start0 + a - 1];
    }
    // index of the completion of the entry at tick tj (relaxed: at place oj)
    // by the lane's type of word q: its first event in range
    __device__ __forceinline__ int completed(int q, int tj, int oj) const
    {
        const TypeIdx ty = ix.ty[(q0 + q) / j.n_iv * 64 + __lane_id()];
        const int x = REL ? tj : tj + lo[q] + 1;
        const int i = REL ? ix.ei[start_m + oj] : 0;
        const int *et = ix.et + ty.start, *ei = ix.ei + ty.start;
        const int b = bucket(x, ty.t0, ty.sh, ty.nb);
        int a = ix.tab[ty.boff + b], z = ix.tab[ty.boff + b + 1];
        while (a < z) {
            const int mid = (a + z) >> 1;
            const bool before = REL ? at(ei, mid) <= i : at(et, mid) < x;
            a = before ? mid + 1 : a;
            z = before ? z : mid;
        }
        return at(ei, a);
    }
};

// Episodes by their last type: counts by block (in LDS, then one atomic a
// block and type), a scan, places.
constexpr int ORDER_PER = 4096;  // episodes a block takes
template <bool PLACE>
__global__ __launch_bounds__(256) void k_order(const int *__restrict__ F, int w, int cnt, int T,
                                               int *__restrict__ next, int *__restrict__ order)
{
    extern __shared__ int sh[];
    for (int e = threadIdx.x; e < T; e += 256) sh[e] = 0;
    __syncthreads();
    const int a0 = blockIdx.x * ORDER_PER;
    const int a1 = a0 + ORDER_PER < cnt ? a0 + ORDER_PER : cnt;
    for (int a = a0 + threadIdx.x; a < a1; a += 256) atomicAdd(&sh[F[(int64_t)a * w + w - 1]], 1);
    __syncthreads();
    for (int e = threadIdx.x; e < T; e += 256)
        if (sh[e]) sh[e] = atomicAdd(&next[e], sh[e]);
    if (!PLACE) return;
    __syncthreads();
    for (int a = a0 + threadIdx.x; a < a1; a += 256)
        order[atomicAdd(&sh[F[(int64_t)a * w + w - 1]], 1)] = a;
}

// Waves a SIMD is given registers for, by length (2, 3, more shared nodes).  Two
// of the kernels keep a few vector registers in scratch for it: relaxed, two shared
// nodes, 12 (36 B a lane); exact, three, 4 (20 B).
constexpr int sib_waves(bool rel, int emax) { return emax == 1 ? 7 : emax == 2 && !rel ? 6 : 5; }

// One wave per frequent episode and QW mask words (grid z), by the episodes'
// last types: what a wave reads at random -- the last stage's list and the
// masks of its entries -- is then the same few lists for all waves at a time,
// and stays in every XCD's L2.
//   64 entries cost about 55 vector instructions for 64 types and a hop, where
// the scan of the whole stream it replaces costs about 60 for each 64 events
// and 64 siblings; an episode of 3 nodes has a few hundred entries in 1.06e6
// events.  It is bound by issue (0.85 of its rate at 3e5 episodes of 3 nodes)
// and, at fewer episodes, by the masks' latency at the waves its registers
// leave, so the lengths have kernels of their own:
// two and three shared nodes take the mask words of a batch while the one
// before is counted, 7 and 6 waves a SIMD instead of 4 and 5 -- 64 types and 3
// hops over 780 s, four-node level 4.94 -> 4.2 ms; 200 types, three-node
// level 1.04 -> 0.87 ms.
template <bool REL, int EMAX>
__global__ __launch_bounds__(WAVE, sib_waves(REL, EMAX)) void k_siblings(SibJob j, int64_t cnt)
{
    extern __shared__ int lds[];
    const int64_t item = grid_item();
    if (item >= cnt) return;
    const int64_t al = j.order[item];
    const int lane = __lane_id();
    const int q0 = (int)blockIdx.z * j.words;
    const int nq = j.Q - q0 < j.words ? j.Q - q0 : j.words;
    const int64_t out0 = j.off[al];
    const int len = (int)(j.off[al + 1] - out0);
    const int *sib = j.F + j.first[al] * j.w + (j.w - 3);  // (lo, hi, type) of a sibling
    // the sibling's mask word
    auto word_of = [&](int c) {
        const int *s = sib + (int64_t)c * j.w;
        int h = 0;
        for (int k = 1; k < j.n_iv; ++k) h = (j.ivlo[k] == s[0] && j.ivhi[k] == s[1]) ? k : h;
        return (s[2] >> 6) * j.n_iv + h;
    };
    if (len == 0) return;
    if (j.Q > QW) {
        // (none of this wave's words may have a sibling)
        bool any = false;
        for (int c = lane; c < len; c += WAVE) any |= (unsigned)(word_of(c) - q0) < (unsigned)nq;
        if (bal(any) == 0) return;
    }
    NodeRow row;
    Rows rows{};
    rows.ty = j.F;
    rows.lo = j.F + 1;
    rows.hi = j.F + 2;
    rows.ts = rows.hs = j.w;
    rows.tk = rows.hk = 3;
    rows.N = j.m;
    load_row(j.ix, rows, al, row);
    const int m = EMAX < NMAX - 2 ? EMAX + 1 : j.m;
    // the entries of its first pair (node 0, hop 0, node 1)
    const int *key = j.F + al * j.w;
    int k0 = 0;
    for (int k = 1; k < j.n_iv; ++k) k0 = (j.ivlo[k] == key[1] && j.ivhi[k] == key[2]) ? k : k0;
    const int64_t ak = (int64_t)j.rank[key[0]] * j.n_iv + k0;
    const int64_t sd = ak * j.sd.stride + rdl(row.start, 1);
    const Seeds seed{j.sd.t + sd, j.sd.a + sd, j.sd.p + sd};
    Columns<REL> sink{j,
                      j.ix,
                      q0,
                      nq,
                      rdl(row.start, 0),
                      rdl(row.start, m - 1),
                      rdl(row.boff, 0),
                      rdl(row.nb, 0),
                      rdl(row.sh, 0),
                      row.t0,
                      seed.a};
#pragma unroll
    for (int q = 0; q < QW; ++q) {
        const int h = (q0 + (q < nq ? q : 0)) % j.n_iv;
        sink.lo[q] = j.ivlo[h];
        sink.hi[q] = j.ivhi[h];
        sink.cnt[q] = 0;
        sink.tl[q] = -(1 << 30);
        sink.ol[q] = 0;
    }
    walk<REL, FROM_PAIR, EMAX>(j.ix, row, m - 1, 0, j.sd.n[ak * j.nF + j.rank[key[3]]], lds, sink, seed);
    // counts by type to the siblings
    int *tot = lds;
#pragma unroll
    for (int q = 0; q < QW; ++q) tot[q * WAVE + lane] = sink.cnt[q];
    __builtin_amdgcn_wave_barrier();
    for (int c = lane; c < len; c += WAVE) {
        const unsigned q = (unsigned)(word_of(c) - q0);
        if (q >= (unsigned)nq) continue;
        const int v = tot[q * WAVE + (sib[(int64_t)c * j.w + 2] & 63)];
        j.out[out0 + c] = j.upper && j.upper[out0 + c] < j.theta ? -1 : v;
    }
}

}  // namespace

void launch_masks(bool rel, const IndexPlan &p, const int *base, const int *ivlo, const int *ivhi,
                  int n_iv, uint2 *mask, hipStream_t s)
{
    const ChainIdx ix = index_view(p, const_cast<int *>(base));
    const int places = p.n + LIST_EXTRA * p.T, Q = mask_words(p.T, n_iv);
    const dim3 grid((unsigned)((places + 255) / 256), (unsigned)((p.T + 63) / 64 * 2 * ((n_iv + MH - 1) / MH)));
    if (rel)
        hipLaunchKernelGGL(k_masks<true>, grid, dim3(256), 0, s, ix, places, p.T, n_iv, ivlo, ivhi,
                           (unsigned *)mask, Q);
    else
        hipLaunchKernelGGL(k_masks<false>, grid, dim3(256), 0, s, ix, places, p.T, n_iv, ivlo,
                           ivhi, (unsigned *)mask, Q);
}

void launch_pairs(bool rel, const PairJob &j, hipStream_t s)
{
    const dim3 grid = grid_of((int64_t)j.nF * j.nF * j.n_iv);
    const size_t lds = RING_INTS * sizeof(int);
    if (rel) hipLaunchKernelGGL(k_pairs<true>, grid, dim3(WAVE), lds, s, j);
    else hipLaunchKernelGGL(k_pairs<false>, grid, dim3(WAVE), lds, s, j);
}

int64_t order_ints(int64_t cnt, int T) { return cnt + 2 * (int64_t)T + scan_scratch_ints(T); }

void launch_order(const int *F, int w, int64_t cnt, int T, int *order, hipStream_t s)
{
    if (cnt <= 0) return;
    int *hist = order + cnt, *next = hist + T;
    launch_fill(hist, 0, T, s);
    const dim3 grid((unsigned)((cnt + ORDER_PER - 1) / ORDER_PER));
    const size_t lds = (size_t)T * sizeof(int);
    hipLaunchKernelGGL(k_order<false>, grid, dim3(256), lds, s, F, w, (int)cnt, T, hist, order);
    launch_scan_excl(hist, T, next, next + T, s);
    hipLaunchKernelGGL(k_order<true>, grid, dim3(256), lds, s, F, w, (int)cnt, T, next, order);
}

namespace {
template <bool REL>
void siblings_by_length(const SibJob &j, int64_t cnt, dim3 grid, size_t lds, hipStream_t s)
{
    if (j.m == 2)
        hipLaunchKernelGGL((k_siblings<REL, 1>), grid, dim3(WAVE), lds, s, j, cnt);
    else if (j.m == 3)
        hipLaunchKernelGGL((k_siblings<REL, 2>), grid, dim3(WAVE), lds, s, j, cnt);
    else
        hipLaunchKernelGGL((k_siblings<REL, NMAX - 2>), grid, dim3(WAVE), lds, s, j, cnt);
}
}  // namespace

void launch_siblings(bool rel, const SibJob &job, int64_t cnt, hipStream_t s)
{
    if (cnt <= 0) return;
    SibJob j = job;
    // (few episodes leave the device to the latency of a wave's own steps: then
    // fewer words a wave, though each wave makes the entries anew.  Three words
    // in one wave each / in three: 1452 episodes of 2 nodes, relaxed, 2.6e5
    // events 3.96 / 1.96 ms; 1275 of 4 over 1.06e6 0.72 / 0.56; 158 of 5 0.54 /
    // 0.41.  From about as many waves as the device holds nothing is gained)
    auto blocks = [&](int words) { return (j.Q + words - 1) / words; };
    j.words = QW;
    while (j.words > 1 && cnt * blocks(j.words) < SIB_FILL && blocks(j.words / 2) < 65536)
        j.words /= 2;
    const dim3 grid = grid_of(cnt, blocks(j.words));
    // (rings of the stages between node 1 and the last; the counts at the end)
    const int rings = (j.m > 2 ? j.m - 2 : 0) * RING_INTS;
    const size_t lds = (size_t)(rings > QW * WAVE ? rings : QW * WAVE) * sizeof(int);
    if (rel) siblings_by_length<true>(j, cnt, grid, lds, s);
    else siblings_by_length<false>(j, cnt, grid, lds, s);
}

}  // namespace fe
