// Level-wise mining on the device: candidate generation by the join, and
// run-aligned tiling of a level's candidates for both passes of Algorithm 4.
//
// Input: the level's keys in generation order (per candidate t0 lo0 hi0 t1
// ... t_{m-1}) and, for the exact pass, the relaxed counts: the survivors are
// the candidates with upper >= theta (the elimination step), kept in
// generation order.  They are grouped by list-depth class (stable), and in
// each class cut into maximal runs of equal first m-1 types (join siblings).
// A run fills whole tiles; a remainder of at least half a tile gets a padded
// tile of its own, shorter remainders are packed, in run order, into the
// class's last tiles.  Output: orig[tile*64 + lane] = candidate index (-1 =
// padding), classes in order, and per class its tile count -- the same lane
// assignment as the host tiler, without taking the keys or the relaxed
// counts to the host.
//
// Every step is a map, an exclusive scan, or a scatter by scanned offsets;
// counts that size later steps stay on the device (kernels past them exit
// early), so the host waits once, for the per-class tile counts.
#include "fe_internal.h"

namespace fe {
namespace {

constexpr int TB = 256;           // threads per block
constexpr int TPT = 4;            // items per thread in the scans
constexpr int CHUNK = TB * TPT;   // items per scan block

__device__ __forceinline__ int key_dcls(const int *k, int m)
{
    int bound = 1;
    for (int j = 0; j < m - 1; ++j) {
        const int b = window_bound(k[3 * j + 1], k[3 * j + 2]);
        bound = b > bound ? b : bound;
    }
    return depth_class(bound);
}

// cls[i] = list-depth class of a kept candidate (0 for the relaxed pass),
// -1 for a pruned one
__global__ void k_tl_class(const int *__restrict__ key, int m, int64_t M,
                           const int *__restrict__ up, int theta, int exact, int *__restrict__ cls)
{
    const int64_t i = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (i >= M) return;
    const int w = 3 * m - 2;
    const bool keep = !up || up[i] >= theta;
    cls[i] = !keep ? -1 : exact ? key_dcls(key + i * w, m) : 0;
}

// ---------------------------------------------------------------- scan
// Exclusive scan of v(i), i < n (n read from *np when np is set, else
// nfix): out[i] = sum of v(j), j < i; *total = sum of all.
struct ClassFlag {
    const int *cls;
    int c;
    __device__ int operator()(int64_t i) const { return cls[i] == c ? 1 : 0; }
};
struct AtLeast {
    const int *a;
    int theta;
    __device__ int operator()(int64_t i) const { return a[i] >= theta ? 1 : 0; }
};
struct Arr {
    const int *a;
    __device__ int operator()(int64_t i) const { return a[i]; }
};

__device__ __forceinline__ int64_t count_of(const int *np, int64_t nfix)
{
    return np ? (int64_t)*np : nfix;
}

// block sum of the values, and the block's exclusive prefix within LDS
__device__ __forceinline__ int block_excl(int v, int *sh, int &tot)
{
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == WAVE - 1) sh[wv] = x;
    __syncthreads();
    int base = 0, all = 0;
    for (int k = 0; k < TB / WAVE; ++k) {
        base += k < wv ? sh[k] : 0;
        all += sh[k];
    }
    __syncthreads();
    tot = all;
    return base + x - v;
}

template <class F>
__global__ void k_scan_up(F f, const int *np, int64_t nfix, int *__restrict__ bsum)
{
    __shared__ int sh[TB / WAVE];
    const int64_t n = count_of(np, nfix);
    const int64_t b0 = blockIdx.x * (int64_t)CHUNK;
    if (b0 >= n) {
        if (threadIdx.x == 0) bsum[blockIdx.x] = 0;
        return;
    }
    int s = 0;
    for (int k = 0; k < TPT; ++k) {
        const int64_t i = b0 + threadIdx.x * (int64_t)TPT + k;
        s += i < n ? f(i) : 0;
    }
    int tot;
    block_excl(s, sh, tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// one block: exclusive scan of the nb block sums in place, total to *total
__global__ void k_scan_top(int *__restrict__ bsum, int64_t nb, int *__restrict__ total)
{
    __shared__ int sh[TB / WAVE];
    const int64_t per = (nb + TB - 1) / TB;
    const int64_t b = threadIdx.x * per, e = b + per < nb ? b + per : nb;
    int s = 0;
    for (int64_t i = b; i < e; ++i) s += bsum[i];
    int tot;
    int run = block_excl(s, sh, tot);
    for (int64_t i = b; i < e; ++i) {
        const int v = bsum[i];
        bsum[i] = run;
        run += v;
    }
    if (threadIdx.x == 0) *total = tot;
}

template <class F>
__global__ void k_scan_down(F f, const int *np, int64_t nfix, const int *__restrict__ bsum,
                            int *__restrict__ out)
{
    __shared__ int sh[TB / WAVE];
    const int64_t n = count_of(np, nfix);
    const int64_t b0 = blockIdx.x * (int64_t)CHUNK;
    if (b0 >= n) return;
    int v[TPT], s = 0;
    for (int k = 0; k < TPT; ++k) {
        const int64_t i = b0 + threadIdx.x * (int64_t)TPT + k;
        v[k] = i < n ? f(i) : 0;
        s += v[k];
    }
    int tot;
    int run = bsum[blockIdx.x] + block_excl(s, sh, tot);
    for (int k = 0; k < TPT; ++k) {
        const int64_t i = b0 + threadIdx.x * (int64_t)TPT + k;
        if (i < n) out[i] = run;
        run += v[k];
    }
}

template <class F>
void scan(F f, const int *np, int64_t nmax, int *out, int *bsum, int *total, hipStream_t s)
{
    const int64_t nb = (nmax + CHUNK - 1) / CHUNK;
    if (nb == 0) {
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(TB), 0, s, bsum, (int64_t)0, total);
        return;
    }
    hipLaunchKernelGGL(k_scan_up<F>, dim3((unsigned)nb), dim3(TB), 0, s, f, np, nmax, bsum);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(TB), 0, s, bsum, nb, total);
    hipLaunchKernelGGL(k_scan_down<F>, dim3((unsigned)nb), dim3(TB), 0, s, f, np, nmax, bsum,
                       out);
}

// ---------------------------------------------------------------- steps
// seg[c] = first position of class c in the partition, seg[NDCLS] = kept
__global__ void k_tl_seg(const int *__restrict__ ctot, int *__restrict__ seg)
{
    int acc = 0;
    for (int c = 0; c < NDCLS; ++c) {
        seg[c] = acc;
        acc += ctot[c];
    }
    seg[NDCLS] = acc;
}

// class c's candidates to part[] after those of classes 0..c-1
__global__ void k_tl_part(const int *__restrict__ cls, int64_t M, int c,
                          const int *__restrict__ pos, const int *__restrict__ ctot,
                          int *__restrict__ part)
{
    const int64_t i = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (i >= M || cls[i] != c) return;
    int base = 0;
    for (int d = 0; d < c; ++d) base += ctot[d];
    part[base + pos[i]] = (int)i;
}

__device__ __forceinline__ int class_at(const int *seg, int j)
{
    int c = 0;
    for (int k = 1; k < NDCLS; ++k) c = j >= seg[k] ? k : c;
    return c;
}

// flag[j] = 1 where a run starts: a class's first position, or first m-1
// types differing from position j-1's
__global__ void k_tl_runflag(const int *__restrict__ part, const int *__restrict__ seg,
                             const int *__restrict__ key, int m, int *__restrict__ flag)
{
    const int64_t j = blockIdx.x * (int64_t)TB + threadIdx.x;
    const int S = seg[NDCLS];
    if (j >= S) return;
    bool start = j == 0;
    for (int c = 1; c < NDCLS; ++c) start |= j == seg[c];
    if (!start) {
        const int w = 3 * m - 2;
        const int *a = key + (int64_t)part[j - 1] * w, *b = key + (int64_t)part[j] * w;
        for (int k = 0; k < m - 1; ++k) start |= a[3 * k] != b[3 * k];
    }
    flag[j] = start ? 1 : 0;
}

__global__ void k_tl_runstart(const int *__restrict__ flag, const int *__restrict__ rx,
                              const int *__restrict__ seg, int *__restrict__ rs)
{
    const int64_t j = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (j >= seg[NDCLS] || !flag[j]) return;
    rs[rx[j]] = (int)j;
}

// per run: tiles of its own (whole tiles, plus one padded when the remainder
// is at least half a tile) and lanes left for the class's packed tiles
__global__ void k_tl_runvals(const int *__restrict__ rs, const int *__restrict__ R,
                             const int *__restrict__ seg, int *__restrict__ rt,
                             int *__restrict__ rm)
{
    const int64_t r = blockIdx.x * (int64_t)TB + threadIdx.x;
    const int nr = *R;
    if (r >= nr) return;
    const int len = (r + 1 < nr ? rs[r + 1] : seg[NDCLS]) - rs[r];
    const int rem = len % WAVE;
    rt[r] = len / WAVE + (rem >= WAVE / 2 ? 1 : 0);
    rm[r] = rem >= WAVE / 2 ? 0 : rem;
}

// info[c]: tiles of class c; info[NDCLS + c]: its first tile; info[2*NDCLS +
// c]: its run tiles; info[3*NDCLS + c]: its first run; info[4*NDCLS + c]:
// candidates; info[5*NDCLS]: total tiles
__global__ void k_tl_groups(const int *__restrict__ seg, const int *__restrict__ rx,
                            const int *__restrict__ R, const int *__restrict__ toff,
                            const int *__restrict__ ttot, const int *__restrict__ moff,
                            const int *__restrict__ mtot, int *__restrict__ info)
{
    const int nr = *R;
    int base = 0;
    for (int c = 0; c < NDCLS; ++c) {
        const int n = seg[c + 1] - seg[c];
        int tiles = 0, rt = 0, fr = 0;
        if (n > 0) {
            fr = rx[seg[c]];
            int er = nr;  // first run of the next non-empty class
            for (int d = c + 1; d < NDCLS; ++d)
                if (seg[d + 1] > seg[d]) {
                    er = rx[seg[d]];
                    break;
                }
            const int t0 = toff[fr], t1 = er < nr ? toff[er] : *ttot;
            const int m0 = moff[fr], m1 = er < nr ? moff[er] : *mtot;
            rt = t1 - t0;
            tiles = rt + (m1 - m0 + WAVE - 1) / WAVE;
        }
        info[c] = tiles;
        info[NDCLS + c] = base;
        info[2 * NDCLS + c] = rt;
        info[3 * NDCLS + c] = fr;
        info[4 * NDCLS + c] = n;
        base += tiles;
    }
    info[5 * NDCLS] = base;
}

__global__ void k_tl_lanes(const int *__restrict__ part, const int *__restrict__ seg,
                           const int *__restrict__ flag, const int *__restrict__ rx,
                           const int *__restrict__ rs, const int *__restrict__ R,
                           const int *__restrict__ toff, const int *__restrict__ moff,
                           const int *__restrict__ info, int *__restrict__ orig)
{
    const int64_t j = blockIdx.x * (int64_t)TB + threadIdx.x;
    const int S = seg[NDCLS];
    if (j >= S) return;
    const int nr = *R;
    const int r = rx[j] + flag[j] - 1;
    const int len = (r + 1 < nr ? rs[r + 1] : S) - rs[r];
    const int k = (int)j - rs[r];
    const int full = len / WAVE, rem = len % WAVE;
    const int c = class_at(seg, (int)j);
    const int fr = info[3 * NDCLS + c], gbase = info[NDCLS + c];
    int tile, lane;
    if (k < full * WAVE || rem >= WAVE / 2) {
        const int q = toff[r] - toff[fr];
        tile = gbase + q + k / WAVE;
        lane = k % WAVE;
    } else {
        const int q = moff[r] - moff[fr] + (k - full * WAVE);
        tile = gbase + info[2 * NDCLS + c] + q / WAVE;
        lane = q % WAVE;
    }
    orig[(int64_t)tile * WAVE + lane] = part[j];
}

}  // namespace

int64_t tile_scratch_ints(int64_t M)
{
    // cls, pos, part, flag, rx, rs, rt, rm, toff, moff: M each; block sums
    // and small counters after them
    return 10 * M + (M + CHUNK - 1) / CHUNK + 64;
}

void launch_tile_plan(const int *key, int m, int64_t M, const int *up, int theta, bool exact,
                      int *scratch, int *info, hipStream_t s)
{
    int *cls = scratch, *pos = cls + M, *part = pos + M, *flag = part + M, *rx = flag + M;
    int *rs = rx + M, *rt = rs + M, *rm = rt + M, *toff = rm + M, *moff = toff + M;
    int *bsum = moff + M;
    int *small = bsum + (M + CHUNK - 1) / CHUNK;
    int *ctot = small, *seg = ctot + NDCLS, *R = seg + NDCLS + 1, *ttot = R + 1,
        *mtot = ttot + 1;
    const unsigned gM = (unsigned)((M + TB - 1) / TB);
    if (gM) hipLaunchKernelGGL(k_tl_class, dim3(gM), dim3(TB), 0, s, key, m, M, up, theta,
                               exact ? 1 : 0, cls);
    const int ncls = exact ? NDCLS : 1;
    for (int c = 0; c < NDCLS; ++c) {
        if (c < ncls) {
            scan(ClassFlag{cls, c}, nullptr, M, pos, bsum, ctot + c, s);
            if (gM) hipLaunchKernelGGL(k_tl_part, dim3(gM), dim3(TB), 0, s, cls, M, c, pos, ctot,
                                       part);
        } else {
            hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(TB), 0, s, bsum, (int64_t)0, ctot + c);
        }
    }
    hipLaunchKernelGGL(k_tl_seg, dim3(1), dim3(1), 0, s, ctot, seg);
    if (gM) hipLaunchKernelGGL(k_tl_runflag, dim3(gM), dim3(TB), 0, s, part, seg, key, m, flag);
    scan(Arr{flag}, seg + NDCLS, M, rx, bsum, R, s);
    if (gM) hipLaunchKernelGGL(k_tl_runstart, dim3(gM), dim3(TB), 0, s, flag, rx, seg, rs);
    if (gM) hipLaunchKernelGGL(k_tl_runvals, dim3(gM), dim3(TB), 0, s, rs, R, seg, rt, rm);
    scan(Arr{rt}, R, M, toff, bsum, ttot, s);
    scan(Arr{rm}, R, M, moff, bsum, mtot, s);
    hipLaunchKernelGGL(k_tl_groups, dim3(1), dim3(1), 0, s, seg, rx, R, toff, ttot, moff, mtot,
                       info);
}

void launch_tile_lanes(int64_t M, const int *scratch, const int *info, int *orig, hipStream_t s)
{
    const int *part = scratch + 2 * M, *flag = scratch + 3 * M, *rx = scratch + 4 * M;
    const int *rs = scratch + 5 * M, *toff = scratch + 8 * M, *moff = scratch + 9 * M;
    const int *small = scratch + 10 * M + (M + CHUNK - 1) / CHUNK;
    const int *seg = small + NDCLS, *R = seg + NDCLS + 1;
    const unsigned gM = (unsigned)((M + TB - 1) / TB);
    if (gM) hipLaunchKernelGGL(k_tl_lanes, dim3(gM), dim3(TB), 0, s, part, seg, flag, rx, rs, R,
                               toff, moff, info, orig);
}

// ---------------------------------------------------------------- join
// Level m+1 candidates from the frequent m-node episodes F (sorted keys, w
// ints each): alpha's candidates are alpha's first node and hop followed by
// each beta in F whose first m-1 nodes and hops equal alpha's last m-1
// (first[a]: the first such beta; off[a]..off[a+1]: alpha's output range).
namespace {
__global__ void k_join(const int *__restrict__ F, int w, const int64_t *__restrict__ first,
                       const int64_t *__restrict__ off, int64_t cnt, int64_t M,
                       int *__restrict__ out)
{
    const int64_t j = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (j >= M) return;
    int64_t lo = 0, hi = cnt;  // last a with off[a] <= j
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (off[mid] <= j) lo = mid;
        else hi = mid;
    }
    const int64_t a = lo, b = first[a] + (j - off[a]);
    const int wo = w + 3;
    int *o = out + j * wo;
    const int *al = F + a * w, *be = F + b * w;
    o[0] = al[0];
    o[1] = al[1];
    o[2] = al[2];
    for (int k = 0; k < w; ++k) o[3 + k] = be[k];
}

// Candidate j of the join, without the others: alpha is the last a with
// off[a] <= j.
__global__ void k_join_sel(const int *__restrict__ F, int w, const int64_t *__restrict__ first,
                           const int64_t *__restrict__ off, int64_t cnt,
                           const int *__restrict__ sel, int nsel, int *__restrict__ out)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i >= nsel) return;
    const int64_t j = sel[i];
    int64_t lo = 0, hi = cnt;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (off[mid] <= j) lo = mid;
        else hi = mid;
    }
    const int *al = F + lo * w, *be = F + (first[lo] + (j - off[lo])) * w;
    int *o = out + (int64_t)i * (w + 3);
    o[0] = al[0];
    o[1] = al[1];
    o[2] = al[2];
    for (int k = 0; k < w; ++k) o[3 + k] = be[k];
}

// The values of at least theta, in order: their indices and both arrays'
// values there.
__global__ void k_pick(const int *__restrict__ up, const int *__restrict__ ex, int64_t M,
                       int theta, const int *__restrict__ pos, int *__restrict__ sel,
                       int *__restrict__ out_up, int *__restrict__ out_ex)
{
    const int64_t i = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (i >= M) return;
    const int x = ex[i];
    if (x < theta) return;
    const int at = pos[i];
    sel[at] = (int)i;
    out_ex[at] = x;
    if (out_up) out_up[at] = up[i];
}

// Join plan: the range of beta for each alpha of the sorted F (the first
// m - 1 nodes and hops of beta equal alpha's last m - 1), its length in num;
// *total += all lengths.
__global__ void k_join_plan(const int *__restrict__ F, int w, int cnt,
                            int64_t *__restrict__ first, int *__restrict__ num,
                            unsigned long long *__restrict__ total)
{
    const int a = blockIdx.x * TB + threadIdx.x;
    const int ov = w - 3;
    int n = 0;
    if (a < cnt) {
        const int *suf = F + (int64_t)a * w + 3;
        // F[b]'s prefix against the suffix: -1, 0, 1
        auto cmp = [&](int b) {
            const int *p = F + (int64_t)b * w;
            for (int k = 0; k < ov; ++k)
                if (p[k] != suf[k]) return p[k] < suf[k] ? -1 : 1;
            return 0;
        };
        int lo = 0, hi = cnt;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cmp(mid) < 0) lo = mid + 1;
            else hi = mid;
        }
        int lo2 = lo, hi2 = cnt;
        while (lo2 < hi2) {
            const int mid = (lo2 + hi2) >> 1;
            if (cmp(mid) <= 0) lo2 = mid + 1;
            else hi2 = mid;
        }
        n = lo2 - lo;
        first[a] = lo;
        num[a] = n;
    }
    unsigned long long s = n;
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & (WAVE - 1)) == 0 && s) atomicAdd(total, s);
}

__global__ void k_widen(const int *__restrict__ a, const int *__restrict__ total, int cnt,
                        int64_t *__restrict__ out)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i < cnt) out[i] = a[i];
    if (i == cnt) out[i] = *total;
}

// Level 2 by position: candidate (a, b, k) of the frequent types' ranks and
// interval k is number (a * nF + b) * n_iv + k.  In key order a's candidates
// go by interval, b and then equal intervals: ord holds the intervals sorted,
// then for each sorted place the first place with the same interval and their
// number.
struct PairAt {
    int nF, n_iv;
    const int *ord;
    __device__ int64_t operator()(int64_t i) const
    {
        const int64_t per = (int64_t)nF * n_iv, a = i / per, r = i - a * per;
        const int at = (int)(r / nF), g = ord[n_iv + at], same = ord[2 * n_iv + at];
        const int64_t q = r - (int64_t)g * nF, b = q / same;
        return (a * nF + b) * n_iv + ord[g + (int)(q - b * same)];
    }
};
struct PairAtLeast {
    const int *a;
    int theta;
    PairAt at;
    __device__ int operator()(int64_t i) const { return a[at(i)] >= theta ? 1 : 0; }
};
__global__ void k_pick_pairs(const int *__restrict__ up, const int *__restrict__ ex, int64_t M,
                             int theta, PairAt at, const int *__restrict__ pos,
                             int *__restrict__ sel, int *__restrict__ out_up,
                             int *__restrict__ out_ex)
{
    const int64_t i = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (i >= M) return;
    const int64_t c = at(i);
    const int x = ex[c];
    if (x < theta) return;
    const int to = pos[i];
    sel[to] = (int)c;
    out_ex[to] = x;
    if (out_up) out_up[to] = up[c];
}

// keys of level 2's candidates sel[0..n) (all of them in order: sel null)
__global__ void k_pair_keys(const int *__restrict__ F1, int nF, const int *__restrict__ ivlo,
                            const int *__restrict__ ivhi, int n_iv, const int *__restrict__ sel,
                            int64_t n, int *__restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (i >= n) return;
    const int64_t c = sel ? sel[i] : i;
    const int k = (int)(c % n_iv);
    const int64_t ab = c / n_iv;
    int *o = out + i * 4;
    o[0] = F1[ab / nF];
    o[1] = ivlo[k];
    o[2] = ivhi[k];
    o[3] = F1[ab % nF];
}

// n keys of m nodes to rows of types, lo and hi (in that order in out)
__global__ void k_split_keys(const int *__restrict__ key, int m, int64_t n, int *__restrict__ out)
{
    const int w = 3 * m - 2;
    const int64_t t = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * TB + threadIdx.x;
    if (t >= n * w) return;
    const int64_t i = t / w;
    const int q = (int)(t - i * w), k = q / 3, r = q % 3;
    const int v = key[t];
    if (r == 0) out[i * m + k] = v;
    else out[n * m + (r - 1) * n * (m - 1) + i * (m - 1) + k] = v;
}

__global__ void k_gather_keys(const int *__restrict__ key, int w, const int *__restrict__ sel,
                              int nsel, int *__restrict__ out)
{
    const int64_t t = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (t >= (int64_t)nsel * w) return;
    const int64_t i = t / w;
    const int k = (int)(t - i * w);
    out[t] = key[(int64_t)sel[i] * w + k];
}
// Keys of a sample of the level: every SAMPLE_STRIDE-th block of WAVE
// consecutive candidates (whole blocks keep runs of join siblings together).
__global__ void k_sample_keys(const int *__restrict__ key, int w, int64_t ns,
                              int *__restrict__ out)
{
    const int64_t t = blockIdx.x * (int64_t)TB + threadIdx.x;
    if (t >= ns * w) return;
    const int64_t i = t / w;
    const int k = (int)(t - i * w);
    const int64_t j = i / WAVE * WAVE * SAMPLE_STRIDE + i % WAVE;
    out[t] = key[j * w + k];
}
}  // namespace

int64_t sample_count(int64_t M)
{
    const int64_t span = (int64_t)WAVE * SAMPLE_STRIDE;
    const int64_t r = M % span;
    return M / span * WAVE + (r < WAVE ? r : WAVE);
}

void launch_sample_keys(const int *key, int w, int64_t M, int *out, hipStream_t s)
{
    const int64_t n = sample_count(M) * w;
    if (n <= 0) return;
    hipLaunchKernelGGL(k_sample_keys, dim3((unsigned)((n + TB - 1) / TB)), dim3(TB), 0, s, key, w,
                       sample_count(M), out);
}

int64_t scan_scratch_ints(int64_t n) { return (n + CHUNK - 1) / CHUNK + 1; }

void launch_scan_excl(const int *in, int64_t n, int *out, int *scratch, hipStream_t s)
{
    scan(Arr{in}, nullptr, n, out, scratch + 1, scratch, s);
}

int64_t pick_scratch_ints(int64_t M) { return M + (M + CHUNK - 1) / CHUNK; }

void launch_pick(const int *up, const int *ex, int64_t M, int theta, int *scratch, int *total,
                 int *sel, int *out_up, int *out_ex, hipStream_t s)
{
    scan(AtLeast{ex, theta}, nullptr, M, scratch, scratch + M, total, s);
    if (M > 0)
        hipLaunchKernelGGL(k_pick, dim3((unsigned)((M + TB - 1) / TB)), dim3(TB), 0, s, up, ex, M,
                           theta, scratch, sel, out_up, out_ex);
}

int64_t join_plan_ints(int64_t cnt) { return 2 * cnt + 2 + scan_scratch_ints(cnt); }

void launch_join_plan(const int *F, int w, int64_t cnt, int64_t *first, int64_t *off,
                      unsigned long long *total, int *scratch, hipStream_t s)
{
    launch_fill((int *)total, 0, 2, s);
    if (cnt <= 0) return;
    int *num = scratch, *pos = num + cnt, *sc = pos + cnt;
    hipLaunchKernelGGL(k_join_plan, dim3((unsigned)((cnt + TB - 1) / TB)), dim3(TB), 0, s, F, w,
                       (int)cnt, first, num, total);
    launch_scan_excl(num, cnt, pos, sc, s);
    hipLaunchKernelGGL(k_widen, dim3((unsigned)((cnt + TB) / TB)), dim3(TB), 0, s, pos, sc,
                       (int)cnt, off);
}

void launch_pick_pairs(const int *up, const int *ex, int nF, int n_iv, const int *ord, int theta,
                       int *scratch, int *total, int *sel, int *out_up, int *out_ex,
                       hipStream_t s)
{
    const int64_t M = (int64_t)nF * nF * n_iv;
    const PairAt at{nF, n_iv, ord};
    scan(PairAtLeast{ex, theta, at}, nullptr, M, scratch, scratch + M, total, s);
    if (M > 0)
        hipLaunchKernelGGL(k_pick_pairs, dim3((unsigned)((M + TB - 1) / TB)), dim3(TB), 0, s, up,
                           ex, M, theta, at, scratch, sel, out_up, out_ex);
}

void launch_pair_keys(const int *F1, int nF, const int *ivlo, const int *ivhi, int n_iv,
                      const int *sel, int64_t n, int *out, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_pair_keys, dim3((unsigned)((n + TB - 1) / TB)), dim3(TB), 0, s, F1, nF,
                       ivlo, ivhi, n_iv, sel, n, out);
}

void launch_split_keys(const int *key, int m, int64_t n, int *out, hipStream_t s)
{
    const int64_t t = n * (3 * m - 2);
    if (t <= 0) return;
    // (a grid's dimension holds fewer than 2^32 threads)
    const int64_t blocks = (t + TB - 1) / TB, x = blocks < (1 << 22) ? blocks : 1 << 22;
    hipLaunchKernelGGL(k_split_keys, dim3((unsigned)x, (unsigned)((blocks + x - 1) / x)), dim3(TB),
                       0, s, key, m, n, out);
}

void launch_join_sel(const int *F, int w, const int64_t *first, const int64_t *off, int64_t cnt,
                     const int *sel, int nsel, int *out, hipStream_t s)
{
    if (nsel <= 0) return;
    hipLaunchKernelGGL(k_join_sel, dim3((unsigned)((nsel + TB - 1) / TB)), dim3(TB), 0, s, F, w,
                       first, off, cnt, sel, nsel, out);
}

void launch_join(const int *F, int w, const int64_t *first, const int64_t *off, int64_t cnt,
                 int64_t M, int *out, hipStream_t s)
{
    if (M <= 0 || cnt <= 0) return;
    hipLaunchKernelGGL(k_join, dim3((unsigned)((M + TB - 1) / TB)), dim3(TB), 0, s, F, w, first,
                       off, cnt, M, out);
}

void launch_gather_keys(const int *key, int w, const int *sel, int nsel, int *out, hipStream_t s)
{
    const int64_t n = (int64_t)nsel * w;
    if (n <= 0) return;
    hipLaunchKernelGGL(k_gather_keys, dim3((unsigned)((n + TB - 1) / TB)), dim3(TB), 0, s, key, w,
                       sel, nsel, out);
}

}  // namespace fe
