// Transposed neighbour graph: for every point, the list of centres that name
// it as a neighbour (CSR: in_off / in_src), each list ascending, so that the
// result does not depend on the order in which atomics land (and so that
// repeated sources sit next to each other).
//
// Small clouds: one launch (edge_small_kernel).  Else two ways.  Up to EDGE_BUCKETS_MAX buckets (16384 << bucket_shift(K) points, 16.7 M
// at K = 8): edges are first dealt into buckets of consecutive target points, then
// each bucket is sorted in LDS by one workgroup.  Global atomics per (workgroup, bucket) instead of per edge:
// a random-address atomic per edge (twice) and the scattered 4-byte writes behind
// it were 600 us of the 650 us that 1M points x 8 neighbours in the sensor's
// order took; this takes 95 us, 78 in Z-order.  Beyond that: counting sort by target point with
// an atomic per edge (count -> exclusive scan -> fill -> sort each list).
#include "flex_common.hpp"
#include <stdlib.h>

namespace flex {

static constexpr int SCAN_ITEMS = 8;                    // per thread
static constexpr int SCAN_CHUNK = 256 * SCAN_ITEMS;     // per block
static constexpr int SORT_LOCAL = 32;                   // lists up to here sort in registers

__global__ __launch_bounds__(256) void inedge_count_kernel(const int32_t *__restrict__ nbr,
                                                           int32_t *__restrict__ cnt, int64_t E,
                                                           int N, int64_t KN)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < E;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = i / KN;
        atomicAdd(&cnt[b * N + nbr[i]], 1);
    }
}

// Lists over a subset of the centres (pooling with subsampling): edge i = (cloud b, slot k, kept
// centre j) names point nbr[b, k, sel[b,j]]; the lists hold j.  Entries of sel outside [0,N) are clamped.
__device__ __forceinline__ int64_t sub_edge_target(const int32_t *__restrict__ nbr, const int32_t *__restrict__ sel,
                                                   int64_t i, int N, int Ns, int K, int &j)
{
    const int64_t KNs = (int64_t)K * Ns;
    const int64_t b = i / KNs, r = i - b * KNs;
    const int k = (int)(r / Ns);
    j = (int)(r - (int64_t)k * Ns);
    const int l = min(max(sel[b * Ns + j], 0), N - 1);
    return b * N + nbr[(b * K + k) * N + l];
}

__global__ __launch_bounds__(256) void inedge_sub_count_kernel(const int32_t *__restrict__ nbr,
                                                               const int32_t *__restrict__ sel,
                                                               int32_t *__restrict__ cnt, int64_t E, int N,
                                                               int Ns, int K)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < E;
         i += (int64_t)gridDim.x * blockDim.x) {
        int j;
        atomicAdd(&cnt[sub_edge_target(nbr, sel, i, N, Ns, K, j)], 1);
    }
}

__global__ __launch_bounds__(256) void inedge_sub_fill_kernel(const int32_t *__restrict__ nbr,
                                                              const int32_t *__restrict__ sel,
                                                              const int32_t *__restrict__ off,
                                                              int32_t *__restrict__ cnt,
                                                              int32_t *__restrict__ src, int64_t E, int N,
                                                              int Ns, int K)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < E;
         i += (int64_t)gridDim.x * blockDim.x) {
        int j;
        const int64_t g = sub_edge_target(nbr, sel, i, N, Ns, K, j);
        const int slot = atomicSub(&cnt[g], 1) - 1;
        src[off[g] + slot] = j;
    }
}

__device__ __forceinline__ int block_exclusive_scan(int v, int *s_wave, int &block_total)
{
    // inclusive scan inside the wave, then across the 4 waves
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wave[w] = x;
    __syncthreads();
    int base = 0;
    for (int i = 0; i < w; ++i) base += s_wave[i];
    block_total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    __syncthreads();
    return base + x - v;
}

__global__ __launch_bounds__(256) void scan_block_sums_kernel(const int32_t *__restrict__ cnt,
                                                              int32_t *__restrict__ bsum, int64_t n)
{
    __shared__ int s_wave[4];
    const int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + (int64_t)threadIdx.x * SCAN_ITEMS;
    int v = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i)
        if (base + i < n) v += cnt[base + i];
    int total;
    block_exclusive_scan(v, s_wave, total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// single block: exclusive scan of bsum[0..nblk) in place; bsum[nblk] = grand total
__global__ __launch_bounds__(256) void scan_of_sums_kernel(int32_t *__restrict__ bsum, int nblk)
{
    __shared__ int s_wave[4];
    int carry = 0;
    for (int c0 = 0; c0 < nblk; c0 += 256) {
        const int i = c0 + threadIdx.x;
        const int v = (i < nblk) ? bsum[i] : 0;
        int total;
        const int ex = block_exclusive_scan(v, s_wave, total);
        if (i < nblk) bsum[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) bsum[nblk] = carry;
}

__global__ __launch_bounds__(256) void scan_apply_kernel(const int32_t *__restrict__ cnt,
                                                         const int32_t *__restrict__ bsum,
                                                         int32_t *__restrict__ off, int64_t n,
                                                         int nblk)
{
    __shared__ int s_wave[4];
    const int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + (int64_t)threadIdx.x * SCAN_ITEMS;
    int v[SCAN_ITEMS], sum = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        v[i] = (base + i < n) ? cnt[base + i] : 0;
        sum += v[i];
    }
    int total;
    int run = bsum[blockIdx.x] + block_exclusive_scan(sum, s_wave, total);
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (base + i < n) off[base + i] = run;
        run += v[i];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) off[n] = bsum[nblk];
}

__global__ __launch_bounds__(256) void inedge_fill_kernel(const int32_t *__restrict__ nbr,
                                                          const int32_t *__restrict__ off,
                                                          int32_t *__restrict__ cnt,
                                                          int32_t *__restrict__ src, int64_t E,
                                                          int N, int64_t KN)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < E;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = i / KN;
        const int l = (int)(i % N);
        const int64_t g = b * N + nbr[i];
        const int slot = atomicSub(&cnt[g], 1) - 1;     // counts run down to zero
        src[off[g] + slot] = l;
    }
}

// Sorts the d ids at p ascending (one thread).
__device__ void sort_list(int32_t *__restrict__ p, int d)
{
    if (d < 2) return;
    if (d <= SORT_LOCAL) {
        int v[SORT_LOCAL];
#pragma unroll
        for (int i = 0; i < SORT_LOCAL; ++i) v[i] = (i < d) ? p[i] : 0x7fffffff;
        // odd-even transposition network: data-independent, stays in registers
#pragma unroll 1
        for (int pass = 0; pass < d; ++pass) {
#pragma unroll
            for (int i = 0; i + 1 < SORT_LOCAL; i += 2) {
                const int a = v[i], c = v[i + 1];
                v[i] = min(a, c); v[i + 1] = max(a, c);
            }
#pragma unroll
            for (int i = 1; i + 1 < SORT_LOCAL; i += 2) {
                const int a = v[i], c = v[i + 1];
                v[i] = min(a, c); v[i + 1] = max(a, c);
            }
        }
#pragma unroll
        for (int i = 0; i < SORT_LOCAL; ++i)
            if (i < d) p[i] = v[i];
    } else if (d <= 256) {
        for (int i = 1; i < d; ++i) {                 // rare: insertion sort in place
            const int x = p[i];
            int j = i - 1;
            while (j >= 0 && p[j] > x) { p[j + 1] = p[j]; --j; }
            p[j + 1] = x;
        }
    } else {
        // very rare (a point named by hundreds of centres): heapsort in place, O(d log d)
        auto sift = [&](int root, int end) {
            const int x = p[root];
            for (;;) {
                int child = 2 * root + 1;
                if (child >= end) break;
                if (child + 1 < end && p[child + 1] > p[child]) ++child;
                if (p[child] <= x) break;
                p[root] = p[child];
                root = child;
            }
            p[root] = x;
        };
        for (int i = d / 2 - 1; i >= 0; --i) sift(i, d);
        for (int end = d - 1; end > 0; --end) {
            const int x = p[end]; p[end] = p[0]; p[0] = x;
            sift(0, end);
        }
    }
}

__global__ __launch_bounds__(256) void inedge_sort_kernel(const int32_t *__restrict__ off,
                                                          int32_t *__restrict__ src, int64_t BN)
{
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < BN;
         g += (int64_t)gridDim.x * blockDim.x)
        sort_list(src + off[g], off[g + 1] - off[g]);
}

// ---- edges through buckets -------------------------------------------------------------------------
// bucket = 2^shift consecutive target points (over all clouds), about BUCKET_EDGES edges on average.
//   count    every workgroup takes a run of edges, counts them per bucket in LDS, adds the counts to the buckets'
//   scan     exclusive running sum over the buckets (one workgroup)
//   deal     the same runs again: a workgroup reserves a stretch of every bucket it has edges for (one atomic each)
//            and writes source and target-within-bucket of its edges there
//   sort     one workgroup per bucket: its edges into registers, counts per target and their running sum in LDS
//            (= the list bounds), the lists put together in LDS and sorted there, the bucket out as one contiguous write
static constexpr int BUCKET_EDGES_LOG2 = 13;
static constexpr int BUCKET_NT = 1024;                           // threads per workgroup, all four steps
static constexpr int BUCKET_PER_THREAD = 12;                     // edges a thread of the sort keeps
static constexpr int BUCKET_CAP = BUCKET_NT * BUCKET_PER_THREAD; // edges a bucket sorts in LDS (1.5 x the average)
static constexpr int BUCKET_TARGETS_MAX = 2048;
static constexpr int EDGE_BUCKETS_MAX = 16384;                   // counters of the count / deal steps: 64 KB of LDS

static constexpr int DEAL_PER_THREAD = 32;                       // edges a thread of the deal step keeps
static constexpr int DEAL_BUCKETS_MAX = 3 * BUCKET_NT;           // buckets up to which it orders them in LDS (152 KB)
static constexpr int DEAL_RUN_MIN = 16 * BUCKET_NT;              // edges a workgroup from which it does

struct EdgeRuns {
    const int32_t *nbr, *sel;        // sel == nullptr: every point is a centre
    int N, Nc, K;                    // points and centres per cloud
    int E;                           // edges
    int run;                         // edges per workgroup
    int shift;                       // target >> shift = bucket
};

// Walks a workgroup's run of edges (cloud b, slot k, centre j), BUCKET_NT apart, without a division per edge.
struct EdgeWalk {
    int i, b, k, j;
    __device__ __forceinline__ EdgeWalk(const EdgeRuns &p, int64_t first) : i((int)first)
    {
        const int bk = i / p.Nc;
        j = i - bk * p.Nc;
        b = bk / p.K;
        k = bk - b * p.K;
    }
    __device__ __forceinline__ void next(const EdgeRuns &p)
    {
        i += BUCKET_NT;
        j += BUCKET_NT;
        while (j >= p.Nc) {
            j -= p.Nc;
            if (++k == p.K) { k = 0; ++b; }
        }
    }
};

// Targets (over all clouds; -1: past the n edges of the run) and centres of a thread's next UN edges, the first of them e0 edges into the
// run.  Places first, then the loads, none of them under a condition: behind one, each waits for the one before it.  Past the end the last
// edge is read again.  Entries of sel outside [0,N) are clamped.  us of the build, a load at a time and so: 1M points, K = 8, 104 and 95,
// in Z-order 91 and 78, 500k, K = 16, 116 and 106, 3000 points (one launch) 20 and 17.
template <int UN>
__device__ __forceinline__ void edge_targets(const EdgeRuns &p, EdgeWalk &w, int e0, int n, int *t, int *j)
{
    int at[UN], base[UN], row[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
        j[u] = w.j;
        base[u] = w.b * p.N;
        at[u] = p.sel ? w.b * p.Nc + w.j : w.i;
        row[u] = (w.b * p.K + w.k) * p.N;
        if (e0 + BUCKET_NT * (u + 1) < n) w.next(p);
    }
    if (p.sel) {
#pragma unroll
        for (int u = 0; u < UN; ++u) at[u] = p.sel[at[u]];
#pragma unroll
        for (int u = 0; u < UN; ++u) at[u] = row[u] + min(max(at[u], 0), p.N - 1);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) t[u] = p.nbr[at[u]];
#pragma unroll
    for (int u = 0; u < UN; ++u) t[u] = e0 + BUCKET_NT * u < n ? t[u] + base[u] : -1;
}

// counter[key] += 1 for every lane with on, returning the value before the lane's own addition.  On a cloud stored with
// locality most of a wave's lanes share a key, and as many atomics on one LDS word would queue up: the lanes of the
// first two keys met are counted by a ballot, only the rest go one by one (alone: how often this lane did).
__device__ __forceinline__ int lds_count(int *counter, int key, bool on, int &alone)
{
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    int old = 0;
    bool todo = on;
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        const uint64_t left = __ballot(todo);
        if (left == 0) return old;
        const int first = __ffsll((long long)left) - 1;
        const int lead = __builtin_amdgcn_readlane(key, first);
        const uint64_t same = __ballot(todo && key == lead);
        int base = 0;
        if (lane == first) base = atomicAdd(&counter[lead], __popcll(same));
        base = __builtin_amdgcn_readlane(base, first);
        if (todo && key == lead) { old = base + __popcll(same & below); todo = false; }
    }
    if (todo) { old = atomicAdd(&counter[key], 1); ++alone; }
    return old;
}

template <int UN>                             // edges a thread has under way
__global__ __launch_bounds__(BUCKET_NT) void edge_count_kernel(const EdgeRuns p, int32_t *__restrict__ bucket_cnt,
                                                               int buckets)
{
    extern __shared__ int s_cnt[];
    for (int i = threadIdx.x; i < buckets; i += BUCKET_NT) s_cnt[i] = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * p.run;
    const int n = (int)min((int64_t)p.run, p.E - first);
    int alone = 0;
    EdgeWalk w(p, min(first + threadIdx.x, (int64_t)p.E - 1));
    for (int e0 = 0; e0 < n; e0 += BUCKET_NT * UN) {
        int t[UN], j[UN];
        edge_targets<UN>(p, w, e0 + (int)threadIdx.x, n, t, j);
#pragma unroll
        for (int u = 0; u < UN; ++u) lds_count(s_cnt, t[u] >> p.shift, t[u] >= 0, alone);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < buckets; i += BUCKET_NT)
        if (s_cnt[i]) atomicAdd(&bucket_cnt[i], s_cnt[i]);
}

// off[0..buckets] = exclusive running sum of cnt; cur = a copy of it for the deal step's reservations; one workgroup
__global__ __launch_bounds__(BUCKET_NT) void edge_scan_kernel(const int32_t *__restrict__ cnt, int32_t *__restrict__ off,
                                                              int32_t *__restrict__ cur, int buckets)
{
    __shared__ int s_wave[BUCKET_NT / 64];
    const int per = (buckets + BUCKET_NT - 1) / BUCKET_NT, i0 = threadIdx.x * per;      // at most 16
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int v[EDGE_BUCKETS_MAX / BUCKET_NT], sum = 0;
#pragma unroll
    for (int i = 0; i < EDGE_BUCKETS_MAX / BUCKET_NT; ++i) {
        v[i] = (i < per && i0 + i < buckets) ? cnt[i0 + i] : 0;
        sum += v[i];
    }
    int x = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    int run = x - sum;
    for (int w = 0; w < wave; ++w) run += s_wave[w];
#pragma unroll
    for (int i = 0; i < EDGE_BUCKETS_MAX / BUCKET_NT; ++i) {
        if (i < per && i0 + i < buckets) { off[i0 + i] = run; cur[i0 + i] = run; }
        run += v[i];
    }
    if (threadIdx.x == BUCKET_NT - 1) off[buckets] = run;
}

// What bounds it is the stores: on a cloud stored without locality the edges of a wave go to as many buckets, 64 lines a store
// where a line would hold 32 edges of one bucket.  STAGED: where that is so (most lanes met neither of the first two
// keys of their wave), the run is put in bucket order in LDS first, targets, then sources through the same array, and leaves in
// that order.  1M points of a room in the sensor's order, K = 8: this kernel 81 -> 49 us, the build 135 -> 104; 2.9M in a cube 322 us less.  On clouds with
// locality the waves' own stores are whole lines already (Z-order, 1M points: the build 3 us longer with every run ordered in LDS).
// Up to DEAL_BUCKETS_MAX buckets, what LDS holds beside a run, and from DEAL_RUN_MIN edges a run on: 300k and 100k points in the sensor's
// order, K = 8, runs of 10 and 4 edges a thread: the build 1.5 and 6 us shorter than by LDS; 600k, 19 edges, 13 longer.
template <bool STAGED>
__global__ __launch_bounds__(BUCKET_NT) void edge_deal_kernel(const EdgeRuns p, int32_t *__restrict__ bucket_cur,
                                                              int32_t *__restrict__ st_src, uint16_t *__restrict__ st_tgt,
                                                              int buckets)
{
    constexpr int MAXE = DEAL_PER_THREAD;        // p.run <= MAXE * BUCKET_NT
    constexpr int BPT = DEAL_BUCKETS_MAX / BUCKET_NT;
    __shared__ int s_edge[STAGED ? MAXE * BUCKET_NT : 1], s_move[STAGED ? DEAL_BUCKETS_MAX : 1], s_wave[BUCKET_NT / 64 + 1], s_alone;
    extern __shared__ int s_cnt[];
    const int tid = threadIdx.x;
    for (int i = tid; i < buckets; i += BUCKET_NT) s_cnt[i] = 0;
    if (tid == 0) s_alone = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * p.run;
    const int n = (int)min((int64_t)p.run, p.E - first);
    int t[MAXE], rank[MAXE], alone = 0;
    {
        constexpr int UN = 8;
        EdgeWalk w(p, min(first + tid, (int64_t)p.E - 1));
        int j[UN];
#pragma unroll
        for (int u = 0; u < MAXE; u += UN) {
            if (BUCKET_NT * u < n) {             // uniform
                edge_targets<UN>(p, w, BUCKET_NT * u + tid, n, t + u, j);
            } else {
#pragma unroll
                for (int v = 0; v < UN; ++v) t[u + v] = -1;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < MAXE; ++u)
        if (BUCKET_NT * u < n) rank[u] = lds_count(s_cnt, t[u] >> p.shift, t[u] >= 0, alone);
    if constexpr (STAGED) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) alone += __shfl_xor(alone, d, 64);
        if ((tid & 63) == 0) atomicAdd(&s_alone, alone);
    }
    __syncthreads();
    if (STAGED && 2 * s_alone > n) {             // (the same for the whole workgroup)
        // counts -> the buckets' starts in the run; s_move: from there to the reserved stretch
        const int lane = tid & 63, wave = tid >> 6;
        int c[BPT], sum = 0;
#pragma unroll
        for (int i = 0; i < BPT; ++i) {
            c[i] = BPT * tid + i < buckets ? s_cnt[BPT * tid + i] : 0;
            sum += c[i];
        }
        int x = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        if (lane == 63) s_wave[wave] = x;
        __syncthreads();
        int at = x - sum;
        for (int w = 0; w < wave; ++w) at += s_wave[w];
#pragma unroll
        for (int i = 0; i < BPT; ++i)
            if (c[i]) {
                const int g = BPT * tid + i;
                s_cnt[g] = at;
                s_move[g] = atomicAdd(&bucket_cur[g], c[i]) - at;
                at += c[i];
            }
        if (tid == BUCKET_NT - 1) s_wave[BUCKET_NT / 64] = at;
        __syncthreads();
        const int all = s_wave[BUCKET_NT / 64];  // the run's edges
#pragma unroll
        for (int u = 0; u < MAXE; ++u)
            if (BUCKET_NT * u < n) {
                rank[u] = t[u] >= 0 ? rank[u] + s_cnt[t[u] >> p.shift] : -1;
                if (t[u] >= 0) s_edge[rank[u]] = t[u];
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < MAXE; ++u) {
            const int i = BUCKET_NT * u + tid;
            if (i < all) {
                const int target = s_edge[i];
                t[u] = i + s_move[target >> p.shift];
                st_tgt[t[u]] = (uint16_t)(target & ((1 << p.shift) - 1));
            }
        }
        __syncthreads();
        EdgeWalk w(p, min(first + tid, (int64_t)p.E - 1));
#pragma unroll
        for (int u = 0; u < MAXE; ++u)
            if (BUCKET_NT * u < n) {
                if (rank[u] >= 0) s_edge[rank[u]] = w.j;
                if (BUCKET_NT * (u + 1) + tid < n) w.next(p);
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < MAXE; ++u)
            if (BUCKET_NT * u + tid < all) st_src[t[u]] = s_edge[BUCKET_NT * u + tid];
        return;
    }
    for (int i = tid; i < buckets; i += BUCKET_NT)
        if (const int c = s_cnt[i]) s_cnt[i] = atomicAdd(&bucket_cur[i], c);
    __syncthreads();
    EdgeWalk w(p, min(first + tid, (int64_t)p.E - 1));
#pragma unroll
    for (int u = 0; u < MAXE; ++u)
        if (BUCKET_NT * u < n) {
            if (t[u] >= 0) {
                const int at = s_cnt[t[u] >> p.shift] + rank[u];
                st_src[at] = w.j;
                st_tgt[at] = (uint16_t)(t[u] & ((1 << p.shift) - 1));
            }
            if (BUCKET_NT * (u + 1) + tid < n) w.next(p);
        }
}

// The d ids at p ascending, 1 <= d <= W, one thread: Batcher's odd-even merge exchange in registers.
template <int W>
__device__ __forceinline__ void sort_short(int *p, int d)
{
    int v[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int x = p[min(i, d - 1)];
        v[i] = i < d ? x : 0x7fffffff;
    }
#pragma unroll
    for (int run = 1; run < W; run *= 2)
#pragma unroll
        for (int step = run; step >= 1; step /= 2)
#pragma unroll
            for (int i = 0; i + step < W; ++i)
                if (i >= step % run && (i - step % run) / step % 2 == 0 && i / (2 * run) == (i + step) / (2 * run)) {
                    const int a = v[i], c = v[i + step];
                    v[i] = min(a, c); v[i + step] = max(a, c);
                }
#pragma unroll
    for (int i = 0; i < W; ++i)
        if (i < d) p[i] = v[i];
}

// Lists of up to W edges are sorted by a thread each, up to 64 by a wave, longer ones by the whole workgroup.  What bounded it was LDS:
// a rank for every edge, by reading all of its list, is some 13 reads an edge at K = 8 with 64 lanes in as many places (the longest list of
// a wave's counts), and the arrays for it left one workgroup to a CU; a list in registers is read and written once, target and slot share
// a register, and two workgroups fit (in 64 registers a thread: one is spilled, six with W = 32).  us of the build, ranks and so: 1M points, K = 8, 135 and 104 (Z-order 121 and 91), 100k, K = 16, 64
// and 52, 500k, K = 16, 167 and 116, K = 12 110 and 76, 400k, K = 10, 84 and 61, 200k, K = 32, 199 and 156.  With W = 32 at K = 16 the
// 100k were 66.
template <int W>
__global__ __launch_bounds__(BUCKET_NT, 8) void edge_sort_kernel(const int32_t *__restrict__ bucket_off,
                                                              const int32_t *__restrict__ st_src,
                                                              const uint16_t *__restrict__ st_tgt,
                                                              int32_t *__restrict__ in_off, int32_t *__restrict__ in_src,
                                                              int64_t BN, int E, int shift)
{
    __shared__ int s_off[BUCKET_TARGETS_MAX + 1];     // counts, then list starts inside the bucket
    __shared__ int s_src[BUCKET_CAP];
    __shared__ int s_wave[BUCKET_NT / 64], s_more[BUCKET_CAP / (W + 1) + 1], s_most[BUCKET_CAP / 65 + 1], s_long[2];
    const int targets = 1 << shift, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int beg = bucket_off[blockIdx.x], n = bucket_off[blockIdx.x + 1] - beg;
    const int64_t g0 = (int64_t)blockIdx.x << shift;
    for (int i = tid; i < targets; i += BUCKET_NT) s_off[i] = 0;
    if (tid < 2) s_long[tid] = 0;
    auto starts = [&] {   // counts -> list starts, two targets per thread
        __syncthreads();
        const int i0 = 2 * tid;
        const int a = i0 < targets ? s_off[i0] : 0, c = i0 + 1 < targets ? s_off[i0 + 1] : 0;
        int x = a + c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        if (lane == 63) s_wave[wave] = x;
        __syncthreads();
        int run = x - (a + c);
        for (int w = 0; w < wave; ++w) run += s_wave[w];
        if (i0 < targets) { s_off[i0] = run; if (g0 + i0 < BN) in_off[g0 + i0] = beg + run; }
        if (i0 + 1 < targets) { s_off[i0 + 1] = run + a; if (g0 + i0 + 1 < BN) in_off[g0 + i0 + 1] = beg + run + a; }
        if (tid == 0) {
            s_off[targets] = n;
            if (blockIdx.x == gridDim.x - 1) in_off[BN] = E;
        }
        __syncthreads();
    };
    if (n <= BUCKET_CAP) {
        constexpr unsigned NONE = ~0u;
        static_assert(BUCKET_TARGETS_MAX <= 1 << 12 && BUCKET_CAP <= 1 << 15, "");
        int src[BUCKET_PER_THREAD];
        unsigned own[BUCKET_PER_THREAD];              // target, and above 12 bits the slot in its list
        const int from = min(beg, E - 1);             // (an empty bucket's beginning may lie past the last edge)
        const int32_t *const my_src = st_src + from;
        const uint16_t *const my_tgt = st_tgt + from;
#pragma unroll
        for (int u = 0; u < BUCKET_PER_THREAD; ++u) {
            const unsigned i = min((unsigned)(tid + BUCKET_NT * u), (unsigned)max(n - 1, 0));
            src[u] = my_src[i];
            own[u] = my_tgt[i];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < BUCKET_PER_THREAD; ++u) {
            if (tid + BUCKET_NT * u < n) own[u] |= (unsigned)atomicAdd(&s_off[own[u]], 1) << 12;
            else own[u] = NONE;
        }
        starts();
#pragma unroll
        for (int u = 0; u < BUCKET_PER_THREAD; ++u)
            if (own[u] != NONE) s_src[s_off[own[u] & 0xfff] + (own[u] >> 12)] = src[u];
        __syncthreads();
        for (int i = tid; i < targets; i += BUCKET_NT) {
            const int lo = s_off[i], d = s_off[i + 1] - lo;
            if (d < 2) continue;             // (an empty list's place may lie past the last edge)
            if (d <= W) sort_short<W>(s_src + lo, d);
            else if (d <= 64) s_more[atomicAdd(&s_long[0], 1)] = i;
            else s_most[atomicAdd(&s_long[1], 1)] = i;
        }
        __syncthreads();
        // rank inside the list: sources before mine (equal ones: in the order that they stand in)
        for (int m = wave; m < s_long[0]; m += BUCKET_NT / 64) {
            const int lo = __builtin_amdgcn_readfirstlane(s_off[s_more[m]]);
            const int d = __builtin_amdgcn_readfirstlane(s_off[s_more[m] + 1]) - lo;
            const int me = lane < d ? s_src[lo + lane] : 0x7fffffff;
            int r = lo;
            for (int i = 0; i < d; ++i) {
                const int o = __builtin_amdgcn_readlane(me, i);
                r += (o < me || (o == me && i < lane)) ? 1 : 0;
            }
            if (lane < d) s_src[r] = me;
        }
        // bitonic, every exchange ascending (the first of a merge between mirrored places): what lies past the end counts as larger
        for (int m = 0; m < s_long[1]; ++m) {
            const int lo = s_off[s_most[m]], d = s_off[s_most[m] + 1] - lo;
            for (int size = 2; size < 2 * d; size *= 2)
                for (int step = size / 2; step >= 1; step /= 2) {
                    for (int q = tid; 2 * q < d + size; q += BUCKET_NT) {
                        const int at = q / step * 2 * step, in = q % step;
                        const int i = at + in, j = step == size / 2 ? at + 2 * step - 1 - in : i + step;
                        if (j < d) {
                            const int x = s_src[lo + i], y = s_src[lo + j];
                            if (x > y) { s_src[lo + i] = y; s_src[lo + j] = x; }
                        }
                    }
                    __syncthreads();
                }
        }
        __syncthreads();
        for (int i = tid; i < n; i += BUCKET_NT) in_src[beg + i] = s_src[i];
        return;
    }
    // a bucket of far more edges than its share (hub points): the lists are filled and sorted in global memory
    __syncthreads();
    for (int i = tid; i < n; i += BUCKET_NT) atomicAdd(&s_off[st_tgt[beg + i]], 1);
    starts();
    for (int i = tid; i < targets; i += BUCKET_NT) s_src[i] = s_off[i];
    __syncthreads();
    for (int i = tid; i < n; i += BUCKET_NT) in_src[beg + atomicAdd(&s_src[st_tgt[beg + i]], 1)] = st_src[beg + i];
    __syncthreads();                              // the workgroup's own writes, read back below
    for (int i = tid; i < targets; i += BUCKET_NT) sort_list(in_src + beg + s_off[i], s_off[i + 1] - s_off[i]);
}

// Small clouds, one launch: a workgroup owns a stretch of consecutive targets of one cloud and walks all of that cloud's edges
// twice, counting its own and those of earlier targets (which gives its lists' place), then taking its own to LDS; the lists
// are ordered as above.  The five launches in its place are what such a cloud waits for.  No edge of another cloud names its targets.
static constexpr int SMALL_CAP = 8192;                           // edges a workgroup orders in LDS (four times the average)

__global__ __launch_bounds__(BUCKET_NT) void edge_small_kernel(const EdgeRuns p, int per_cloud, int targets,
                                                               int32_t *__restrict__ in_off, int32_t *__restrict__ in_src, int64_t BN)
{
    __shared__ int s_off[BUCKET_TARGETS_MAX + 1], s_cur[BUCKET_TARGETS_MAX];      // list starts inside the stretch, next places
    __shared__ int s_src[SMALL_CAP];
    __shared__ uint16_t s_tgt[SMALL_CAP];
    __shared__ int s_wave[BUCKET_NT / 64], s_before;
    constexpr int UN = 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x / per_cloud, t0 = (int)(blockIdx.x - b * per_cloud) * targets, nt = min(targets, p.N - t0);
    const int edges = p.K * p.Nc;
    const int64_t first = (int64_t)b * edges;
    for (int i = tid; i < targets; i += BUCKET_NT) s_cur[i] = 0;
    if (tid == 0) s_before = 0;
    __syncthreads();
    // take(t, j): edge of centre j to the stretch's target t; earlier targets' edges are counted
    auto walk = [&](auto &&take) {
        int earlier = 0;
        EdgeWalk w(p, first + min(tid, edges - 1));
        for (int e0 = 0; e0 < edges; e0 += BUCKET_NT * UN) {
            int t[UN], j[UN];
            edge_targets<UN>(p, w, e0 + tid, edges, t, j);
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                t[u] = t[u] >= 0 ? t[u] - b * p.N - t0 : nt;
                earlier += t[u] < 0;
                if (t[u] >= 0 && t[u] < nt) take(t[u], j[u]);
            }
        }
        return earlier;
    };
    {
        int earlier = walk([&](int t, int) { atomicAdd(&s_cur[t], 1); });
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) earlier += __shfl_xor(earlier, d, 64);
        if (lane == 0 && earlier) atomicAdd(&s_before, earlier);
    }
    __syncthreads();
    const int64_t beg = first + s_before;
    {   // counts -> list starts, two targets per thread
        const int i0 = 2 * tid;
        const int a = i0 < nt ? s_cur[i0] : 0, c = i0 + 1 < nt ? s_cur[i0 + 1] : 0;
        int x = a + c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        if (lane == 63) s_wave[wave] = x;
        __syncthreads();
        int run = x - (a + c);
        for (int w = 0; w < wave; ++w) run += s_wave[w];
        if (i0 < nt) { s_off[i0] = s_cur[i0] = run; in_off[(int64_t)b * p.N + t0 + i0] = (int)(beg + run); }
        if (i0 + 1 < nt) { s_off[i0 + 1] = s_cur[i0 + 1] = run + a; in_off[(int64_t)b * p.N + t0 + i0 + 1] = (int)(beg + run + a); }
        if (tid == BUCKET_NT - 1) {
            s_off[nt] = run + a + c;
            if (blockIdx.x == gridDim.x - 1) in_off[BN] = p.E;
        }
    }
    __syncthreads();
    const int n = s_off[nt];
    const bool fits = n <= SMALL_CAP;
    walk([&](int t, int j) {
        const int at = atomicAdd(&s_cur[t], 1);
        if (fits) { s_src[at] = j; s_tgt[at] = (uint16_t)t; }
        else in_src[beg + at] = j;
    });
    __syncthreads();                              // (the workgroup's own writes, read back below)
    if (!fits) {
        for (int i = tid; i < nt; i += BUCKET_NT) sort_list(in_src + beg + s_off[i], s_off[i + 1] - s_off[i]);
        return;
    }
    for (int me = tid; me < n; me += BUCKET_NT) {
        const int src = s_src[me], lo = s_off[s_tgt[me]], hi = s_off[s_tgt[me] + 1];
        int r = lo;
        for (int i = lo; i < hi; ++i) {
            const int o = s_src[i];
            r += (o < src || (o == src && i < me)) ? 1 : 0;
        }
        in_src[beg + r] = src;
    }
}

// the bucketed way's geometry; buckets == 0: too many of them
static int bucket_shift(int K)
{
    int shift = BUCKET_EDGES_LOG2;
    while (shift > 0 && ((int64_t)K << shift) > (1 << BUCKET_EDGES_LOG2)) --shift;
    return shift > 11 ? 11 : shift;               // BUCKET_TARGETS_MAX
}
// (FLEX_EDGE_BUCKETS in the environment lowers the most there may be: 0 = always the counting sort)
static int64_t bucket_count(int64_t BN, int K)
{
    static const int most = [] {
        const char *v = getenv("FLEX_EDGE_BUCKETS");
        const int n = v ? atoi(v) : EDGE_BUCKETS_MAX;
        return n >= 0 && n < EDGE_BUCKETS_MAX ? n : EDGE_BUCKETS_MAX;
    }();
    const int64_t n = cdiv64(BN, (int64_t)1 << bucket_shift(K));
    return n <= most ? n : 0;
}

size_t inedges_ws_bytes(int64_t BN, int K)
{
    if (const int64_t buckets = bucket_count(BN, K)) {
        const size_t E = (size_t)BN * K;
        return align256(sizeof(int32_t) * (size_t)(3 * buckets + 1)) + align256(sizeof(int32_t) * E) + align256(sizeof(uint16_t) * E);
    }
    const int64_t nblk = cdiv64(BN, SCAN_CHUNK);
    return align256(sizeof(int32_t) * (size_t)BN) + align256(sizeof(int32_t) * (size_t)(nblk + 1));
}

// Targets a workgroup of the one-launch build owns; 0: the cloud is not for it.  Every workgroup of a cloud walks all of its edges, so
// those are at most 24576, and 2^15 a CU over all workgroups; more than 2048 workgroups are a launch longer than five.  us, five launches
// and one, K = 8, before the loads went out together (which took up to 3 us off either): 300 points 21 and 10.7, 2048 22.3 and 16.3, 3000 22.5
// and 20.1, 4096 22.2 and 24.5, 1024 with K = 16 22.3 and 18.4, 2048 22.6 and 27.1, 100 x 300 24.5 and 10.5, 30 x 2000 26.2 and 16.5, 4 x 4096
// 24.6 and 24.0, 2000 x 300 67.1 and 65.3; with the edges ranked, 60 x 4096 41 and 65, 3000 x 64 47 and 56.
static int small_targets(int64_t B, int64_t N, int64_t Nc, int K)
{
    const int64_t edges = K * Nc, cus = device_cu_count();
    if (bucket_count(B * N, K) == 0 || edges > 3 << 13) return 0;
    const int64_t own = B * edges > 2048 * cus ? 4096 : 2048;
    auto clamped = [](int64_t x) { return x < 1 ? 1 : x < BUCKET_TARGETS_MAX ? x : BUCKET_TARGETS_MAX; };
    int64_t targets = clamped(own / K);
    // Lists over kept centres are short: where there is more than a workgroup a CU, as many edges are given more targets, and the five launches
    // are overtaken earlier.  us, those, a workgroup to 2048 / K targets and this: 8 x 9.3k points, K = 9, to a quarter 19.9, 32.8 and 18.3; 30 x 1079, K = 32,
    // 21.1, 32.0 and 18.3, to a half 24.5, 42 and those; 1000 x 100, K = 8, to a quarter 19.6, 25.3 and those.
    if (B * cdiv64(N, targets) > cus) targets = clamped(own * N / edges);
    const int64_t groups = B * cdiv64(N, targets);
    return groups <= (Nc < N ? 768 : 2048) && groups * edges <= cus << (Nc < N ? 14 : 15) ? (int)targets : 0;
}

hipError_t launch_inedges_build(const int32_t *nbr, int B, int N, int K, int32_t *in_off,
                                int32_t *in_src, void *ws, hipStream_t s)
{
    return launch_inedges_build_sub(nbr, nullptr, B, N, N, K, in_off, in_src, ws, s);
}

// sel == nullptr: every point is a centre (Ns = N); else the centres are the kept points sel[b, 0..Ns)
// and the lists hold their row numbers j
hipError_t launch_inedges_build_sub(const int32_t *nbr, const int32_t *sel, int B, int N, int Ns, int K,
                                    int32_t *in_off, int32_t *in_src, void *ws, hipStream_t s)
{
    const int64_t BN = (int64_t)B * N, KN = (int64_t)K * N, E = (int64_t)B * K * (sel ? Ns : N);
    if (const int targets = small_targets(B, N, sel ? Ns : N, K)) {
        const int per_cloud = (int)cdiv64(N, targets);
        const EdgeRuns p{nbr, sel, N, sel ? Ns : N, K, (int)E, 0, 0};
        hipLaunchKernelGGL(edge_small_kernel, dim3((unsigned)((int64_t)B * per_cloud)), dim3(BUCKET_NT), 0, s, p, per_cloud, targets, in_off,
                           in_src, BN);
        return hipGetLastError();
    }
    if (const int buckets = (int)bucket_count(BN, K)) {
        int32_t *cnt = (int32_t *)ws, *off = cnt + buckets, *cur = off + buckets + 1;
        int32_t *st_src = (int32_t *)((char *)ws + align256(sizeof(int32_t) * (size_t)(3 * buckets + 1)));
        uint16_t *st_tgt = (uint16_t *)((char *)st_src + align256(sizeof(int32_t) * (size_t)BN * K));
        // runs of edges: a workgroup per CU while they are short, at most what the deal step's registers hold
        int64_t run = cdiv64(cdiv64(E, device_cu_count()), BUCKET_NT) * BUCKET_NT;
        if (run > DEAL_PER_THREAD * BUCKET_NT) run = DEAL_PER_THREAD * BUCKET_NT;
        const EdgeRuns p{nbr, sel, N, sel ? Ns : N, K, (int)E, (int)run, bucket_shift(K)};
        const dim3 g((unsigned)cdiv64(E, run)), blk(BUCKET_NT);
        const size_t lds = sizeof(int) * (size_t)buckets;
        hipError_t e = launch_fill_zero(cnt, sizeof(int32_t) * (size_t)buckets, s);
        if (e != hipSuccess) return e;
        // (34k points of 4 neighbours to a quarter, a run of one edge a thread, eight asked for: 4.8 us, two 3.9)
        hipLaunchKernelGGL(run <= 2 * BUCKET_NT ? edge_count_kernel<2> : edge_count_kernel<8>, g, blk, lds, s, p, cnt, buckets);
        hipLaunchKernelGGL(edge_scan_kernel, dim3(1), blk, 0, s, cnt, off, cur, buckets);
        if (buckets <= DEAL_BUCKETS_MAX && run >= DEAL_RUN_MIN) hipLaunchKernelGGL(edge_deal_kernel<true>, g, blk, lds, s, p, cur, st_src, st_tgt, buckets);
        else hipLaunchKernelGGL(edge_deal_kernel<false>, g, blk, lds, s, p, cur, st_src, st_tgt, buckets);
        // by the mean list; us of the build with W = 8 and 16: a mean of one, 140k points 22.2 and 24.1, 1M 44.6 and 48.6 (K = 8 to a quarter); K = 4,
        // all points, 30k 22.5 and 23.7; a mean of four from K = 8, half the points, 77k 25.1 and 24.6; K = 6, all points, 18k 25 and 21
        const auto sort = E <= 3 * BN || K <= 4 ? edge_sort_kernel<8> : E <= 10 * BN ? edge_sort_kernel<16> : E <= 16 * BN ? edge_sort_kernel<24>
                                                                                                                         : edge_sort_kernel<32>;
        hipLaunchKernelGGL(sort, dim3((unsigned)buckets), blk, 0, s, off, st_src, st_tgt, in_off, in_src, BN, (int)E, p.shift);
        return hipGetLastError();
    }
    const int64_t nblk64 = cdiv64(BN, SCAN_CHUNK);
    const int nblk = (int)nblk64;
    int32_t *cnt = (int32_t *)ws;
    int32_t *bsum = (int32_t *)((char *)ws + align256(sizeof(int32_t) * (size_t)BN));
    hipError_t e = launch_fill_zero(cnt, sizeof(int32_t) * (size_t)BN, s);
    if (e != hipSuccess) return e;
    int64_t eb = (E + 255) / 256;
    if (eb > (1 << 18)) eb = 1 << 18;
    if (sel)
        hipLaunchKernelGGL(inedge_sub_count_kernel, dim3((unsigned)eb), dim3(256), 0, s, nbr, sel, cnt, E, N, Ns, K);
    else
        hipLaunchKernelGGL(inedge_count_kernel, dim3((unsigned)eb), dim3(256), 0, s, nbr, cnt, E, N, KN);
    hipLaunchKernelGGL(scan_block_sums_kernel, dim3(nblk), dim3(256), 0, s, cnt, bsum, BN);
    hipLaunchKernelGGL(scan_of_sums_kernel, dim3(1), dim3(256), 0, s, bsum, nblk);
    hipLaunchKernelGGL(scan_apply_kernel, dim3(nblk), dim3(256), 0, s, cnt, bsum, in_off, BN, nblk);
    if (sel)
        hipLaunchKernelGGL(inedge_sub_fill_kernel, dim3((unsigned)eb), dim3(256), 0, s, nbr, sel, in_off, cnt, in_src,
                           E, N, Ns, K);
    else
        hipLaunchKernelGGL(inedge_fill_kernel, dim3((unsigned)eb), dim3(256), 0, s, nbr, in_off, cnt, in_src, E, N, KN);
    int64_t sb = (BN + 255) / 256;
    if (sb > (1 << 18)) sb = 1 << 18;
    hipLaunchKernelGGL(inedge_sort_kernel, dim3((unsigned)sb), dim3(256), 0, s, in_off, in_src, BN);
    return hipGetLastError();
}

}  // namespace flex
