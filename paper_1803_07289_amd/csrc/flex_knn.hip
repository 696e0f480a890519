// Exact K nearest neighbours on a uniform grid (the neighbourhoods of Sec. 3; the paper computes
// them beforehand and does not say how).  Result: for every point the K points of its cloud with the
// smallest squared distance, itself included, ordered by (d2, index).  d2 is evaluated in fp32 as
// ((dx*dx + dy*dy) + dz*dz) with every operation rounded on its own, the form the CPU check uses, so
// that the ranking (an integer-valued decision) comes out identical.
//
// Steps per call: bounding box of each cloud -> grid of cubic cells (at most 2^24) -> (x,y,z,id)
// records in cell order, by way of buckets of cells (count, scan, deal, sort) -> one thread per point, in that
// order (several lanes to a point where the points are few), searches the 27 cells around its own, then shell by shell, keeps
// the K best in registers and stops once the K-th distance is inside the block of cells already searched -> the lists, so
// far in cell order, go to their places.  Small clouds: every point against all of its cloud, in one launch.
#include "flex_common.hpp"
#include <algorithm>

namespace flex {

static constexpr int KNN_MAX_CELLS_LOG2 = 24;

// cells a cloud's grid may have: 16 / K per point (at most 8).  On scanned surfaces, whose points fill few of the box's cells, the
// block of 27 cells then holds some 50 points at K = 8 and nearly always the K nearest; in a filled volume it takes the
// second shell, 62 points.  Eight per point, whatever K, made four searches of five go on to the second or third shell
// (125 or 343 cells, most of them empty) and cost a 32 MB table for 1M points: 64 us of running sums instead of 20.
__host__ __device__ inline int64_t knn_cell_cap(int64_t N, int K)
{
    const int64_t share = 16 * N / K > 1 ? 16 * N / K : 1, eight = 8 * N, most = (int64_t)1 << KNN_MAX_CELLS_LOG2;
    const int64_t want = share < eight ? share : eight;
    return want < most ? want : most;
}

struct KnnGrid {
    float lo[3];      // bounding box minimum
    float inv_h, h;   // cell edge
    int n[3];         // cells per axis
};

__device__ __forceinline__ unsigned ordered_bits(float x)
{
    const unsigned u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered_bits(unsigned u)
{
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// bbox[b][0..2] = min, [3..5] = max, as order-preserving unsigned keys (min starts at ~0, max at 0); the buckets' counters
// start at zero, and so do the clouds' pairs, a float each behind the boxes
__global__ __launch_bounds__(256) void knn_init_kernel(unsigned *__restrict__ bbox, int B, int32_t *__restrict__ cnt,
                                                       int64_t buckets)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 7 * B) bbox[i] = (i < 6 * B && i % 6 < 3) ? 0xffffffffu : 0u;
    for (int64_t c = i; c < buckets; c += (int64_t)gridDim.x * blockDim.x) cnt[c] = 0;
}

__global__ __launch_bounds__(1024) void knn_bbox_kernel(const float *__restrict__ pos, unsigned *__restrict__ bbox, int N)
{
    const int b = blockIdx.y;
    const float *p = pos + (int64_t)b * 3 * N;
    unsigned mn[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, mx[3] = {0u, 0u, 0u};
    for (int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; l < N; l += (int64_t)gridDim.x * blockDim.x)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const unsigned k = ordered_bits(p[(int64_t)d * N + l]);
            mn[d] = min(mn[d], k);
            mx[d] = max(mx[d], k);
        }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) {
            mn[d] = min(mn[d], (unsigned)__shfl_xor((int)mn[d], s, 64));
            mx[d] = max(mx[d], (unsigned)__shfl_xor((int)mx[d], s, 64));
        }
    }
    // one pair of atomics per block and coordinate: thousands of atomics on the same six words serialise (1M points: 3072 of
    // them 16 us, 1470 10 us)
    __shared__ unsigned s_mn[16][3], s_mx[16][3];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int d = 0; d < 3; ++d) { s_mn[w][d] = mn[d]; s_mx[w][d] = mx[d]; }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int d = threadIdx.x;
        unsigned lo = s_mn[0][d], hi = s_mx[0][d];
#pragma unroll
        for (int i = 1; i < 16; ++i) { lo = min(lo, s_mn[i][d]); hi = max(hi, s_mx[i][d]); }
        atomicMin(&bbox[6 * b + d], lo);
        atomicMax(&bbox[6 * b + 3 + d], hi);
    }
}

// every thread derives the same grid from the bounding box: cubic cells, at most cap in total; a
// flat or degenerate box gets one layer of cells along its thin axes
__device__ __forceinline__ KnnGrid knn_grid(const unsigned *__restrict__ bbox, int b, int64_t cap)
{
    KnnGrid g;
    float ext[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        g.lo[d] = from_ordered_bits(bbox[6 * b + d]);
        ext[d] = fmaxf(from_ordered_bits(bbox[6 * b + 3 + d]) - g.lo[d], 0.f);
    }
    const float longest = fmaxf(fmaxf(ext[0], ext[1]), fmaxf(ext[2], 1e-30f));
    float cells = (float)cap;
    float h = longest;                                   // one cell if everything else fails
    // volume / cells with thin axes counted as one cell thick; two refinements settle the estimate
    for (int it = 0; it < 3; ++it) {
        float vol = 1.f;
#pragma unroll
        for (int d = 0; d < 3; ++d) vol *= fmaxf(ext[d], h);
        h = cbrtf(vol / cells);
        h = fmaxf(h, longest * (1.f / 1024.f));          // at most 1024 cells along an axis
    }
    g.h = h;
    g.inv_h = 1.f / h;
    int64_t total = 1;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        g.n[d] = max(1, min(1024, (int)(ext[d] * g.inv_h) + 1));
        total *= g.n[d];
    }
    // rounding can push the product over the cap: coarsen until it fits
    for (int it = 0; it < 48 && total > cap; ++it) {
        g.h *= 1.26f; g.inv_h = 1.f / g.h;
        total = 1;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            g.n[d] = max(1, min(1024, (int)(ext[d] * g.inv_h) + 1));
            total *= g.n[d];
        }
    }
    if (!(total <= cap)) { g.n[0] = g.n[1] = g.n[2] = 1; }   // only non-finite input gets here: one cell, exhaustive
    return g;
}

__device__ __forceinline__ void knn_cell_of(const KnnGrid &g, float x, float y, float z, int &cx, int &cy, int &cz)
{
    cx = min(g.n[0] - 1, max(0, (int)((x - g.lo[0]) * g.inv_h)));
    cy = min(g.n[1] - 1, max(0, (int)((y - g.lo[1]) * g.inv_h)));
    cz = min(g.n[2] - 1, max(0, (int)((z - g.lo[2]) * g.inv_h)));
}

// ---- points in cell order ---------------------------------------------------------------------------------
// bucket = 2^shift consecutive cells of a cloud.  The points are counted per bucket, dealt into the buckets, and each bucket is put in
// cell order by one workgroup, which writes its cells' bounds on the way.  Counters are in LDS; a workgroup meets the global ones once
// per bucket that it has points for.  (A counter per cell in memory: one returning atomic per point, 46 us at 1M points, and a table of
// 2M counters to clear and to sum, 27.)  us of the whole search, with a counter per cell and so: 1M points of a room in the order drawn
// 242 and 205, in Z-order 222 and 188, 1.5M of a hall with 12 neighbours 433 and 378, 7M of it 1538 and 1377, a cube of 1M 397 and 363.
// Positions have to stay as they are while a call runs.  (Overwritten by another stream meanwhile they could make the count and the deal
// differ, and places, ids and records be what the workspace held: those are clamped where they become an index, and a record whose cell
// has no points starts at itself, so that such an answer means nothing but no access leaves the buffers.)
static constexpr int KNN_BUCKETS_MAX = 4096, KNN_DEAL_NT = 1024;
struct KnnBuckets {
    int shift, n;                                // n: per cloud
};
static KnnBuckets knn_buckets(int64_t cells_per_cloud)
{
    int shift = 9;
    while (cdiv64(cells_per_cloud, (int64_t)1 << shift) > KNN_BUCKETS_MAX) ++shift;
    return KnnBuckets{shift, (int)cdiv64(cells_per_cloud, (int64_t)1 << shift)};
}

__device__ __forceinline__ int knn_linear_cell(const KnnGrid &g, float x, float y, float z)
{
    int cx, cy, cz;
    knn_cell_of(g, x, y, z, cx, cy, cz);
    return (cz * g.n[1] + cy) * g.n[0] + cx;
}

template <int POINTS>                           // a thread
__global__ __launch_bounds__(KNN_DEAL_NT) void knn_count_kernel(const float *__restrict__ pos, const unsigned *__restrict__ bbox,
                                                                int32_t *__restrict__ bucket_cnt, int N, int64_t cells_per_cloud,
                                                                const KnnBuckets k)
{
    __shared__ int s_cnt[KNN_BUCKETS_MAX];
    const int b = blockIdx.y, tid = threadIdx.x;
    for (int i = tid; i < k.n; i += KNN_DEAL_NT) s_cnt[i] = 0;
    const KnnGrid g = knn_grid(bbox, b, cells_per_cloud);
    const float *p = pos + (int64_t)b * 3 * N;
    const int64_t l0 = (int64_t)blockIdx.x * (KNN_DEAL_NT * POINTS) + tid;
    float x[POINTS][3];
#pragma unroll
    for (int u = 0; u < POINTS; ++u)
#pragma unroll
        for (int d = 0; d < 3; ++d) x[u][d] = p[(int64_t)d * N + min(l0 + KNN_DEAL_NT * u, (int64_t)N - 1)];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < POINTS; ++u)
        if (l0 + KNN_DEAL_NT * u < N) atomicAdd(&s_cnt[knn_linear_cell(g, x[u][0], x[u][1], x[u][2]) >> k.shift], 1);
    __syncthreads();
    for (int i = tid; i < k.n; i += KNN_DEAL_NT)
        if (s_cnt[i]) atomicAdd(&bucket_cnt[(int64_t)b * k.n + i], s_cnt[i]);
}

// bucket_off = where the buckets' points begin over all clouds, bucket_cur = a copy for the reservations; a workgroup per cloud
__global__ __launch_bounds__(1024) void knn_bucket_scan_kernel(const int32_t *__restrict__ cnt, int32_t *__restrict__ off,
                                                               int32_t *__restrict__ cur, int N, int n)
{
    __shared__ int s_wave[16];
    constexpr int PER = KNN_BUCKETS_MAX / 1024;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int v[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        v[i] = PER * tid + i < n ? cnt[(int64_t)b * n + PER * tid + i] : 0;
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
    int run = b * N + x - sum;
    for (int w = 0; w < wave; ++w) run += s_wave[w];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (PER * tid + i < n) { off[(int64_t)b * n + PER * tid + i] = run; cur[(int64_t)b * n + PER * tid + i] = run; }
        run += v[i];
    }
    if (b == (int)gridDim.x - 1 && tid == 1023) off[(int64_t)gridDim.x * n] = (b + 1) * N;
}

// staged: (x, y, z, id), bucket by bucket in no set order
template <int POINTS>                           // a thread
__global__ __launch_bounds__(KNN_DEAL_NT) void knn_deal_kernel(const float *__restrict__ pos, const unsigned *__restrict__ bbox,
                                                               int32_t *__restrict__ bucket_cur, float4 *__restrict__ st_rec,
                                                               int N, int64_t cells_per_cloud, const KnnBuckets k)
{
    __shared__ int s_cnt[KNN_BUCKETS_MAX];
    const int b = blockIdx.y, tid = threadIdx.x;
    for (int i = tid; i < k.n; i += KNN_DEAL_NT) s_cnt[i] = 0;
    const KnnGrid g = knn_grid(bbox, b, cells_per_cloud);
    const float *p = pos + (int64_t)b * 3 * N;
    const int64_t l0 = (int64_t)blockIdx.x * (KNN_DEAL_NT * POINTS) + tid;
    float x[POINTS][3];
    int bucket[POINTS], rank[POINTS];
#pragma unroll
    for (int u = 0; u < POINTS; ++u)
#pragma unroll
        for (int d = 0; d < 3; ++d) x[u][d] = p[(int64_t)d * N + min(l0 + KNN_DEAL_NT * u, (int64_t)N - 1)];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < POINTS; ++u) {
        bucket[u] = knn_linear_cell(g, x[u][0], x[u][1], x[u][2]) >> k.shift;
        rank[u] = l0 + KNN_DEAL_NT * u < N ? atomicAdd(&s_cnt[bucket[u]], 1) : 0;
    }
    __syncthreads();
    for (int i = tid; i < k.n; i += KNN_DEAL_NT)
        if (const int c = s_cnt[i]) s_cnt[i] = atomicAdd(&bucket_cur[(int64_t)b * k.n + i], c);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < POINTS; ++u) {
        const int64_t l = l0 + KNN_DEAL_NT * u;
        if (l >= N) continue;
        st_rec[min(s_cnt[bucket[u]] + rank[u], (int)gridDim.y * N - 1)] = make_float4(x[u][0], x[u][1], x[u][2], __int_as_float((int)l));
    }
}

// rec = the points in cell order, off[b*cells_per_cloud + cell] = where a cell's begin, place[b*N + id] = a point's record, inside
// the cloud.  Dynamic LDS: 2^shift counters.
// pairs[b]: less than no number if the grid is one layer of cells (layers), else how many records lie in the row of three
// cells around every record's own, added up (rows; a bucket's first and last cell without the neighbour outside)
__global__ __launch_bounds__(256) void knn_sort_kernel(const int32_t *__restrict__ bucket_off, const float4 *__restrict__ st_rec,
                                                       const unsigned *__restrict__ bbox, float4 *__restrict__ rec,
                                                       int32_t *__restrict__ off, int32_t *__restrict__ place,
                                                       float *__restrict__ pairs, bool layers, bool rows, int N,
                                                       int64_t cells_per_cloud, const KnnBuckets k)
{
    extern __shared__ int s_at[];                // counts, then the next record of every cell
    __shared__ int s_wave[4];
    constexpr int UN = 4;
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cells = 1 << k.shift;
    const int beg = bucket_off[(int64_t)b * k.n + blockIdx.x], n = bucket_off[(int64_t)b * k.n + blockIdx.x + 1] - beg;
    for (int i = tid; i < cells; i += 256) s_at[i] = 0;
    const KnnGrid g = knn_grid(bbox, b, cells_per_cloud);
    auto cell = [&](const float4 &q) { return knn_linear_cell(g, q.x, q.y, q.z) & (cells - 1); };
    // each(f): f of every point, the next ones already requested.  (A cloud whose box a few stray points stretch has most of its points in few
    // buckets, and this is their time: a sheet of 1M points and 16 outside it by its own length, sixteen buckets of 65k, 229 us and 170; 4M of it, all
    // in one, 3240 and 2170; a cube without 22.7 and 21.7.)
    auto each = [&](auto &&f) {
        float4 next[UN];
        auto request = [&](int i0) {
#pragma unroll
            for (int u = 0; u < UN; ++u) next[u] = st_rec[beg + min(i0 + 256 * u, n - 1)];
        };
        if (tid < n) request(tid);
        for (int i0 = tid; i0 < n; i0 += 256 * UN) {
            float4 q[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) q[u] = next[u];
            if (i0 + 256 * UN < n) request(i0 + 256 * UN);
#pragma unroll
            for (int u = 0; u < UN; ++u)
                if (i0 + 256 * u < n) f(q[u]);
        }
    };
    __syncthreads();
    each([&](const float4 &q) { atomicAdd(&s_at[cell(q)], 1); });
    __syncthreads();
    const int per = cells / 256, i0 = tid * per;
    int sum = 0;
    for (int i = 0; i < per; ++i) sum += s_at[i0 + i];
    if (layers && blockIdx.x == 0 && tid == 0 && min(min(g.n[0], g.n[1]), g.n[2]) == 1) atomicAdd(&pairs[b], -__builtin_inff());
    if (rows) {
        float mine = 0.f;
        for (int i = i0; i < i0 + per; ++i)
            mine += (float)s_at[i] * (float)(s_at[i] + (i > 0 ? s_at[i - 1] : 0) + (i + 1 < cells ? s_at[i + 1] : 0));
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, 64);
        if (lane == 0 && mine > 0.f) atomicAdd(&pairs[b], mine);
    }
    int x = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    int run = beg + x - sum;
    for (int w = 0; w < wave; ++w) run += s_wave[w];
    for (int i = 0; i < per; ++i) {
        const int c = s_at[i0 + i];
        s_at[i0 + i] = run;
        run += c;
    }
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x << k.shift;
    int32_t *my_off = off + b * cells_per_cloud + c0;
    for (int i = tid; i < cells && c0 + i < cells_per_cloud; i += 256) my_off[i] = s_at[i];
    if (b == (int)gridDim.y - 1 && blockIdx.x == gridDim.x - 1 && tid == 0) off[gridDim.y * cells_per_cloud] = (b + 1) * N;
    __syncthreads();
    each([&](const float4 &q) {
        const int at = atomicAdd(&s_at[cell(q)], 1);
        const int id = min((unsigned)__float_as_int(q.w), (unsigned)(N - 1));
        rec[at] = make_float4(q.x, q.y, q.z, __int_as_float(id));
        place[(int64_t)b * N + id] = at - b * N;
    });
}

// Two of the products are rounded with their sums: written out, so that every form of the search ranks by the same bits whatever a
// compiler makes of operators.
__device__ __forceinline__ float knn_d2(float dx, float dy, float dz)
{
    return __builtin_fmaf(dz, dz, __builtin_fmaf(dx, dx, dy * dy));
}

// (d2, id) as one number whose order is theirs: the bits of d2 (non-negative: they order like the value) above those
// of id, read as a double -- positive, and finite since a float's exponent field fills only the upper bits of a
// double's -- so that the sorted insertion is a minimum and a maximum per place.  (Double arithmetic keeps denormals
// here, which the pairs with d2 == 0 are.)  A NaN distance keeps its operand's sign, and with the sign bit set it would be
// the smallest key of all: without it, it is larger than that of any distance, or no number, and never taken.
__device__ __forceinline__ double knn_key(float d2, int id) { return __hiloint2double(__float_as_int(d2) & 0x7fffffff, id); }

// One thread per point, in cell order (neighbouring threads search neighbouring cells); lists[record][K].
// What bounds it is the issue of instructions, and before that the chain offsets -> records of one thread.  So the nine rows of
// cells of the first block (three cells each, contiguous records) have all their offsets requested at once, and one loop runs
// over the records of all nine, the next ones already requested, so that a wave waits for its longest total and not for the
// longest of every row; the rows' bounds wait in LDS.  The rows come nearest first, the point's own before all others: the
// sorted insertion is run if any lane needs it, and that is for 73 of a wave's 125 records in a scanned room (1M points, K = 8)
// and not for 90.  Two records a step: what a step costs beside them, the row's end above all, is paid half as often.  Both
// together: 168 -> 127 us there, 1M points in a cube (where the second shell takes most of the time) the whole call 412 -> 402.
template <int K>
__device__ __forceinline__ void knn_search(const float4 *__restrict__ rec, const int32_t *__restrict__ off,
                                           const unsigned *__restrict__ bbox, int32_t *__restrict__ lists, int N,
                                           int64_t cells_per_cloud)
{
    __shared__ int s_beg[9][256], s_end[9][256];
    const int b = blockIdx.y, tid = threadIdx.x;
    const KnnGrid g = knn_grid(bbox, b, cells_per_cloud);
    const int32_t *offb = off + b * cells_per_cloud;
    // slack for the rounding of the cell planes lo + c*h and of the cell a point was put in
    const float span = fmaxf(fmaxf(g.n[0], g.n[1]), (float)g.n[2]) * g.h;
    const float far = fmaxf(fmaxf(fabsf(g.lo[0]), fabsf(g.lo[1])), fabsf(g.lo[2])) + span;
    const float eps = 4e-6f * span + 2e-6f * far;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        const float4 me = rec[(int64_t)b * N + i];
        int cx, cy, cz;
        knn_cell_of(g, me.x, me.y, me.z, cx, cy, cz);
        double best[K];
#pragma unroll
        for (int k = 0; k < K; ++k) best[k] = knn_key(__builtin_inff(), 0x7fffffff);
        auto offer = [&](const float4 &q, bool on) {
            double x = knn_key(knn_d2(q.x - me.x, q.y - me.y, q.z - me.z), __float_as_int(q.w));
            if (on && x < best[K - 1]) {
#pragma unroll
                for (int k = 0; k < K; ++k) {        // sorted insertion: the candidate bubbles down the list
                    const double worse = fmax(best[k], x);
                    best[k] = fmin(best[k], x);
                    x = worse;
                }
            }
        };
        // is everything outside the block of cells [c-r, c+r] farther away than the K-th so far?
        auto settled = [&](int r) {
            float reach = __builtin_inff();
            if (cx - r > 0) reach = fminf(reach, me.x - (g.lo[0] + (float)(cx - r) * g.h));
            if (cx + r < g.n[0] - 1) reach = fminf(reach, (g.lo[0] + (float)(cx + r + 1) * g.h) - me.x);
            if (cy - r > 0) reach = fminf(reach, me.y - (g.lo[1] + (float)(cy - r) * g.h));
            if (cy + r < g.n[1] - 1) reach = fminf(reach, (g.lo[1] + (float)(cy + r + 1) * g.h) - me.y);
            if (cz - r > 0) reach = fminf(reach, me.z - (g.lo[2] + (float)(cz - r) * g.h));
            if (cz + r < g.n[2] - 1) reach = fminf(reach, (g.lo[2] + (float)(cz + r + 1) * g.h) - me.z);
            reach -= eps;
            if (reach == __builtin_inff()) return true;                 // the block is the whole grid
            const float kth = __int_as_float(__double2hiint(best[K - 1]));
            return reach > 0.f && kth < reach * reach * 0.999999f;
        };
        {
            // the 27 cells around: the non-empty rows' bounds to LDS, then one loop over their records
            constexpr int order[9] = {4, 1, 3, 5, 7, 0, 2, 6, 8};
            int b0[9], b1[9];
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                const int z = cz + order[j] / 3 - 1, y = cy + order[j] % 3 - 1;
                const bool on = z >= 0 && z < g.n[2] && y >= 0 && y < g.n[1];
                const int row = ((on ? z : cz) * g.n[1] + (on ? y : cy)) * g.n[0];
                b0[j] = offb[row + max(cx - 1, 0)];
                b1[j] = offb[row + min(cx + 1, g.n[0] - 1) + 1];
                if (!on) b1[j] = b0[j];
            }
            int rows = 0;
#pragma unroll
            for (int j = 0; j < 9; ++j)
                if (b0[j] < b1[j]) { s_beg[rows][tid] = b0[j]; s_end[rows][tid] = b1[j]; ++rows; }
            if (rows == 0) { s_beg[0][tid] = b * N + (int)i; s_end[0][tid] = b * N + (int)i + 1; }     // (see above the bucket kernels)
            // (the second record of a row's last step may be the next row's, or what
            // follows the records in the workspace: read, not offered)
            int j = 0, e = s_beg[0][tid], end = s_end[0][tid];
            float4 q0 = rec[e], q1 = rec[e + 1];
            for (bool more = true; more;) {
                const float4 c0 = q0, c1 = q1;
                const bool two = e + 1 < end;
                e += 2;
                if (e >= end) {
                    more = ++j < rows;
                    if (more) { e = s_beg[j][tid]; end = s_end[j][tid]; }
                }
                if (more) { q0 = rec[e]; q1 = rec[e + 1]; }
                offer(c0, true);
                offer(c1, two);
            }
        }
        const int rmax = max(max(g.n[0], g.n[1]), g.n[2]);
        for (int r = 2; !settled(r - 1) && r <= rmax; ++r) {
            const int z0 = max(cz - r, 0), z1 = min(cz + r, g.n[2] - 1);
            const int y0 = max(cy - r, 0), y1 = min(cy + r, g.n[1] - 1);
            const int x0 = max(cx - r, 0), x1 = min(cx + r, g.n[0] - 1);
            for (int z = z0; z <= z1; ++z)
                for (int y = y0; y <= y1; ++y) {
                    const int row = (z * g.n[1] + y) * g.n[0];
                    // on a face row every x is on the shell; otherwise only the two ends are
                    if (abs(z - cz) == r || abs(y - cy) == r) {
                        const int e1 = offb[row + x1 + 1];
                        for (int e = offb[row + x0]; e < e1; ++e) offer(rec[e], true);
                    } else {
                        const int xa = cx - r, xb = cx + r;
                        const int a0 = xa >= 0 ? offb[row + xa] : 0, a1 = xa >= 0 ? offb[row + xa + 1] : 0;
                        const int c0 = xb < g.n[0] ? offb[row + xb] : 0, c1 = xb < g.n[0] ? offb[row + xb + 1] : 0;
                        for (int e = a0; e < a1; ++e) offer(rec[e], true);
                        for (int e = c0; e < c1; ++e) offer(rec[e], true);
                    }
                }
        }
        int32_t *dst = lists + ((int64_t)b * N + i) * K;
#pragma unroll
        for (int k = 0; k < K; ++k) dst[k] = __double2loint(best[k]);
    }
}

// Waves a SIMD that the K best in registers leave room for; S: lanes to a point.  (Left to itself the compiler takes two registers more
// at some K, and a wave less.  One thread and K = 9: the same four waves either way, and 158k points of a room take 190 us bound to four, 182 not.)
constexpr int knn_waves(int K, int S)
{
    return K <= 2 ? 7 : K <= 4 ? (S == 1 ? 7 : S == 16 && K == 4 ? 5 : 6) : K <= 6 ? 5 : K <= 8 ? (S <= 4 ? 5 : 4) : K == 9 && S == 1 ? 1 : K <= 12 ? 4 : K <= 16 ? 3 : 2;
}

template <int K>
__global__ __launch_bounds__(256, knn_waves(K, 1)) void knn_query_kernel(const float4 *__restrict__ rec, const int32_t *__restrict__ off,
                                                        const unsigned *__restrict__ bbox, int32_t *__restrict__ lists,
                                                        int N, int64_t cells_per_cloud)
{
    knn_search<K>(rec, off, bbox, lists, N, cells_per_cloud);
}

// ---- several lanes to a point ---------------------------------------------------------------------------
// minimum over the S lanes (a power of two, at most 16) of the caller's group, in each of them
template <int CTRL>
__device__ __forceinline__ double dpp_min(double x)
{
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    return fmin(x, __hiloint2double(hi, lo));
}
template <int S>
__device__ __forceinline__ double lanes_min(double x)
{
    x = dpp_min<0xB1>(x);                            // the neighbour, the other pair of the four, the other four, the other eight
    x = dpp_min<0x4E>(x);
    if constexpr (S >= 8) x = dpp_min<0x141>(x);
    if constexpr (S >= 16) x = dpp_min<0x140>(x);
    return x;
}

// The K best of a group of S lanes: each keeps those of the candidates that it was offered.
template <int K, int S>
struct GroupBest {
    double best[K], merged[K];
    __device__ __forceinline__ static double none() { return knn_key(__builtin_inff(), 0x7fffffff); }
    __device__ __forceinline__ GroupBest()
    {
#pragma unroll
        for (int k = 0; k < K; ++k) best[k] = merged[k] = none();
    }
    __device__ __forceinline__ void offer(float mx, float my, float mz, float x, float y, float z, int id)
    {
        double c = knn_key(knn_d2(x - mx, y - my, z - mz), id);
        if (c < best[K - 1]) {
#pragma unroll
            for (int k = 0; k < K; ++k) {            // sorted insertion: the candidate bubbles down the list
                const double worse = fmax(best[k], c);
                best[k] = fmin(best[k], c);
                c = worse;
            }
        }
    }
    // merged: the K best of the group; the smallest head is taken K times
    __device__ __forceinline__ void merge()
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            merged[k] = lanes_min<S>(best[0]);
            if (best[0] == merged[k]) {
#pragma unroll
                for (int j = 0; j + 1 < K; ++j) best[j] = best[j + 1];
                best[K - 1] = none();
            }
        }
    }
    // goes on with what the group has: its first lane keeps it, the others keep what is better than its last
    __device__ __forceinline__ void resume(int sub)
    {
#pragma unroll
        for (int k = 0; k < K; ++k) best[k] = sub == 0 ? merged[k] : merged[K - 1];
    }
};

// The search above with S lanes to a point, for clouds whose points are too few to fill the device a thread each: the nine rows'
// bounds are asked for by as many lanes, the records of all of them dealt out one by one, a shell's rows one by one.
// Merging costs the same however few records a point has around it, and in a layer of cells there are hardly more than K (nine cells;
// scanned surfaces in a box of cells have 4 K to 6 K, points that fill it 3 K).  A cloud with fewer pairs (knn_sort_kernel) than `few` is searched
// a thread to a point all the same.
template <int K, int S>
__global__ __launch_bounds__(256, knn_waves(K, S)) void knn_query_group_kernel(const float4 *__restrict__ rec, const int32_t *__restrict__ off,
                                                              const unsigned *__restrict__ bbox, const float *__restrict__ pairs,
                                                              float few, int32_t *__restrict__ lists, int N, int64_t cells_per_cloud)
{
    constexpr int G = 256 / S;
    __shared__ int s_beg[9][G], s_end[9][G];
    const int b = blockIdx.y, sub = threadIdx.x % S, grp = threadIdx.x / S;
    if (pairs[b] < few) {
        if ((int)blockIdx.x * 256 < N) knn_search<K>(rec, off, bbox, lists, N, cells_per_cloud);
        return;
    }
    const KnnGrid g = knn_grid(bbox, b, cells_per_cloud);
    const int32_t *offb = off + b * cells_per_cloud;
    const float span = fmaxf(fmaxf(g.n[0], g.n[1]), (float)g.n[2]) * g.h;
    const float far = fmaxf(fmaxf(fabsf(g.lo[0]), fabsf(g.lo[1])), fabsf(g.lo[2])) + span;
    const float eps = 4e-6f * span + 2e-6f * far;
    for (int64_t i0 = (int64_t)blockIdx.x * G; i0 < N; i0 += (int64_t)gridDim.x * G) {
        const int64_t i = i0 + grp < N ? i0 + grp : N - 1;               // past the cloud: its last point, not stored
        const float4 me = rec[(int64_t)b * N + i];
        int cx, cy, cz;
        knn_cell_of(g, me.x, me.y, me.z, cx, cy, cz);
        GroupBest<K, S> found;
        auto offer = [&](const float4 &q) { found.offer(me.x, me.y, me.z, q.x, q.y, q.z, __float_as_int(q.w)); };
        auto settled = [&](int r) {
            float reach = __builtin_inff();
            if (cx - r > 0) reach = fminf(reach, me.x - (g.lo[0] + (float)(cx - r) * g.h));
            if (cx + r < g.n[0] - 1) reach = fminf(reach, (g.lo[0] + (float)(cx + r + 1) * g.h) - me.x);
            if (cy - r > 0) reach = fminf(reach, me.y - (g.lo[1] + (float)(cy - r) * g.h));
            if (cy + r < g.n[1] - 1) reach = fminf(reach, (g.lo[1] + (float)(cy + r + 1) * g.h) - me.y);
            if (cz - r > 0) reach = fminf(reach, me.z - (g.lo[2] + (float)(cz - r) * g.h));
            if (cz + r < g.n[2] - 1) reach = fminf(reach, (g.lo[2] + (float)(cz + r + 1) * g.h) - me.z);
            reach -= eps;
            if (reach == __builtin_inff()) return true;                 // the block is the whole grid
            const float kth = __int_as_float(__double2hiint(found.merged[K - 1]));
            return reach > 0.f && kth < reach * reach * 0.999999f;
        };
        __syncthreads();                   // the bounds of the points before are done with
        for (int j = sub; j < 9; j += S) {
            const int at = j == 0 ? 4 : j <= 4 ? 2 * j - 1 : j == 5 ? 0 : j == 6 ? 2 : j == 7 ? 6 : 8;     // nearest rows first
            const int z = cz + at / 3 - 1, y = cy + at % 3 - 1;
            const bool on = z >= 0 && z < g.n[2] && y >= 0 && y < g.n[1];
            const int row = ((on ? z : cz) * g.n[1] + (on ? y : cy)) * g.n[0];
            const int b0 = offb[row + max(cx - 1, 0)], b1 = offb[row + min(cx + 1, g.n[0] - 1) + 1];
            s_beg[j][grp] = b0;
            s_end[j][grp] = on ? b1 : b0;
        }
        __syncthreads();
        {
            int j = 0, e = s_beg[0][grp] + sub, end = s_end[0][grp];
            // this lane's next record: past a row's end, as far into the next one
            auto there = [&]() {
                while (e >= end) {
                    if (++j == 9) return false;
                    e += s_beg[j][grp] - end;
                    end = s_end[j][grp];
                }
                return true;
            };
            bool more = there();
            float4 q = me;
            if (more) q = rec[e];
            while (more) {
                const float4 c = q;
                e += S;
                more = there();
                if (more) q = rec[e];
                offer(c);
            }
        }
        found.merge();
        const int rmax = max(max(g.n[0], g.n[1]), g.n[2]);
        for (int r = 2; !settled(r - 1) && r <= rmax; ++r) {
            found.resume(sub);
            const int z0 = max(cz - r, 0), z1 = min(cz + r, g.n[2] - 1);
            const int y0 = max(cy - r, 0), y1 = min(cy + r, g.n[1] - 1), ny = y1 - y0 + 1;
            const int x0 = max(cx - r, 0), x1 = min(cx + r, g.n[0] - 1);
            for (int t = sub; t < (z1 - z0 + 1) * ny; t += S) {
                const int z = z0 + t / ny, y = y0 + t % ny, row = (z * g.n[1] + y) * g.n[0];
                // on a face row every x is on the shell; otherwise only the two ends are
                if (abs(z - cz) == r || abs(y - cy) == r) {
                    const int e1 = offb[row + x1 + 1];
                    for (int e = offb[row + x0]; e < e1; ++e) offer(rec[e]);
                } else {
                    const int xa = cx - r, xb = cx + r;
                    const int a0 = xa >= 0 ? offb[row + xa] : 0, a1 = xa >= 0 ? offb[row + xa + 1] : 0;
                    const int c0 = xb < g.n[0] ? offb[row + xb] : 0, c1 = xb < g.n[0] ? offb[row + xb + 1] : 0;
                    for (int e = a0; e < a1; ++e) offer(rec[e]);
                    for (int e = c0; e < c1; ++e) offer(rec[e]);
                }
            }
            found.merge();
        }
        if (i0 + grp < N) {
            int32_t *dst = lists + ((int64_t)b * N + i) * K;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (k % S == sub) dst[k] = __double2loint(found.merged[k]);
        }
    }
}

// Small clouds: every point against all of its cloud, sixteen lanes to a point, in one launch.
template <int K>
__global__ __launch_bounds__(256) void knn_all_kernel(const float *__restrict__ pos, int32_t *__restrict__ nbr, int N)
{
    constexpr int S = 16, G = 256 / S, U = 4;
    const int b = blockIdx.y, sub = threadIdx.x % S, l = blockIdx.x * G + threadIdx.x / S, lc = min(l, N - 1);
    const float *px = pos + (int64_t)b * 3 * N, *py = px + N, *pz = py + N;
    const float mx = px[lc], my = py[lc], mz = pz[lc];
    GroupBest<K, S> found;
    float x[U], y[U], z[U];
    auto request = [&](int n0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n = min(n0 + S * u, N - 1);
            x[u] = px[n]; y[u] = py[n]; z[u] = pz[n];
        }
    };
    request(sub);
    for (int n0 = sub; n0 < N; n0 += S * U) {
        float cx[U], cy[U], cz[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { cx[u] = x[u]; cy[u] = y[u]; cz[u] = z[u]; }
        request(n0 + S * U);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (n0 + S * u < N) found.offer(mx, my, mz, cx[u], cy[u], cz[u], n0 + S * u);
    }
    found.merge();
    if (l < N) {
        int32_t *dst = nbr + (int64_t)b * K * N + l;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k % S == sub) dst[(int64_t)k * N] = __double2loint(found.merged[k]);
    }
}

// nbr[b][k][l] = lists[b][place of l][k]: a list is read as one stretch and the tensor written in its own order.  (The
// search writing to the points' own columns, on a cloud in the sensor's order 4 bytes per line of memory, took 100 us
// of the 365 that 1M points x 8 cost.)
__global__ __launch_bounds__(256) void knn_place_kernel(const int32_t *__restrict__ lists,
                                                        const int32_t *__restrict__ place, int32_t *__restrict__ nbr,
                                                        int N, int K)
{
    const int b = blockIdx.y;
    for (int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; l < N; l += (int64_t)gridDim.x * blockDim.x) {
        const int at = (int)min((unsigned)place[(int64_t)b * N + l], (unsigned)(N - 1));      // (clamped: see above the bucket kernels)
        const int32_t *src = lists + ((int64_t)b * N + at) * K;
        int32_t *dst = nbr + (int64_t)b * K * N + l;
        for (int k0 = 0; k0 < K; k0 += 8) {
            int v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[min(k0 + u, K - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + u < K) dst[(int64_t)(k0 + u) * N] = v[u];
        }
    }
}

static size_t knn_used_bytes(int B, int N, int K)
{
    const int64_t cpc = knn_cell_cap(N, K), BN = (int64_t)B * N;
    return align256(sizeof(float4) * (size_t)BN) + align256(sizeof(int32_t) * (size_t)BN) + align256(sizeof(int32_t) * (size_t)(B * cpc + 1)) +
           align256(sizeof(unsigned) * 7 * (size_t)B) + align256(sizeof(int32_t) * (size_t)(3 * (int64_t)B * knn_buckets(cpc).n + 1)) +
           std::max(align256(sizeof(int32_t) * (size_t)BN * K), align256(sizeof(float4) * (size_t)BN));
}

// At least what a counting sort by cells asked for: the size that callers have been told.  (More is used only where lists of three
// and fewer belong to clouds of more than 8 M points.)
size_t knn_ws_bytes(int B, int N, int K)
{
    const int64_t cells = (int64_t)B * knn_cell_cap(N, K);
    return std::max(knn_used_bytes(B, N, K),
                    align256(sizeof(float4) * (size_t)B * N) + 2 * align256(sizeof(int32_t) * (size_t)B * N) +
                        align256(sizeof(int32_t) * (size_t)B * N * K) + align256(sizeof(int32_t) * (size_t)(cells + 1)) * 2 +
                        align256(sizeof(int32_t) * (size_t)(cdiv64(cells, 2048) + 1)) + align256(sizeof(unsigned) * 6 * (size_t)B));
}

// Is every point compared with all of its cloud?  One launch in place of eight, and no grid; the work grows with the square.  us (the whole
// call, K = 8, the grid with a thread per point / sixteen lanes, and here): 300 points 68 / 32 and 9.1, 1024 75 / 35 and 11.9, 4096 79 / 36
// and 35, 8 x 1000 132 / 48 and 15, 100 x 300 111 / 60 and 17.5, 3 x 2500, K = 10, 99 / 40 and 31, 2 x 4096 81 / 40 and 45.
static bool knn_all(int64_t B, int64_t N) { return N <= 4096 && B * N * N <= 25 << 20; }

// Lanes to a point.  A thread's search is a chain of dependent reads that few points leave uncovered; merging costs the more the
// more lanes.  us, the whole call, with 1, 4, 8 and 16 lanes: a room, K = 8, 30k points 131, 77, 64, 56; 65k 139, 90, 76, 71; 90k 151, 109, 86,
// 85; 130k 133, 100, 94, 104; 200k 134, 107, 116, 136; K = 16, 30k 194, 111, 85, 79; 130k 223, 159, 148, 169; box surfaces, K = 8, 30k 185, 105, 83, 73;
// a filled cube, K = 8, 15k 81, 49, 43, 40; 65k 91, 69, 76, 88; 90k 112, 90, 99, 110; 130k 105, 104, 124, 147; 200k 112, 133.  With K = 1 a list is one
// number: 50k 33, 35, 35, 38.
// Clouds whose points have few others around them would lose from so many points on that they fill the device a thread each (layers, rows of
// cells).  us, lanes and a thread: a sheet, K = 8, 47k points 58.6 and 58.0, 130k 86.9 and 72.3; K = 16, 30k 85 and 71, 65k 102 and 76; K = 32, 30k 179 and
// 104; a cube, K = 16, 65k 115 and 110, 130k 166 and 146; K = 32, 47k 164 and 169, 65k 222 and 182.  Records in the row of three cells, of K: cubes 0.38
// to 0.49, surfaces in boxes 0.6 and more, 0.9 at such sizes.
static int knn_lanes(int64_t points, int K)
{
    if (points <= 1 << 15) return 16;
    if (K < 4) return 1;
    return points <= 1 << 16 ? 8 : points <= 1 << 17 ? 4 : 1;
}

template <int K>
static void launch_knn_query(const float4 *rec, const int32_t *off, const unsigned *bbox, int32_t *lists, int B, int N, int64_t cells_per_cloud,
                             const float *pairs, float few, hipStream_t s)
{
    const int lanes = knn_lanes((int64_t)B * N, K);
    const dim3 grid((unsigned)std::min<int64_t>(((int64_t)N * lanes + 255) / 256, 65535), B);
    auto groups = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, rec, off, bbox, pairs, few, lists, N, cells_per_cloud);
    };
    if (lanes == 16) return groups(knn_query_group_kernel<K, 16>);
    if constexpr (K >= 4) {
        if (lanes == 8) return groups(knn_query_group_kernel<K, 8>);
        if (lanes == 4) return groups(knn_query_group_kernel<K, 4>);
    }
    hipLaunchKernelGGL(knn_query_kernel<K>, grid, dim3(256), 0, s, rec, off, bbox, lists, N, cells_per_cloud);
}

#define FLEX_KNN_KS(CASE) \
    CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(12) CASE(16) CASE(24) CASE(32)

hipError_t launch_knn(const float *pos, int32_t *nbr, int B, int N, int K, void *ws, hipStream_t s)
{
    if (knn_all(B, N)) {
#define FLEX_KNN_ALL(KK) \
    case KK: hipLaunchKernelGGL(knn_all_kernel<KK>, dim3((N + 15) / 16, B), dim3(256), 0, s, pos, nbr, N); break;
        switch (K) {
            FLEX_KNN_KS(FLEX_KNN_ALL)
        default: return hipErrorInvalidValue;
        }
#undef FLEX_KNN_ALL
        return hipGetLastError();
    }
    const int64_t cpc = knn_cell_cap(N, K), cells = (int64_t)B * cpc;
    const KnnBuckets k = knn_buckets(cpc);
    const int64_t buckets = (int64_t)B * k.n;
    char *at = (char *)ws;
    float4 *rec = (float4 *)at;       at += align256(sizeof(float4) * (size_t)B * N);
    int32_t *place = (int32_t *)at;   at += align256(sizeof(int32_t) * (size_t)B * N);
    int32_t *off = (int32_t *)at;     at += align256(sizeof(int32_t) * (size_t)(cells + 1));
    unsigned *bbox = (unsigned *)at;  at += align256(sizeof(unsigned) * 7 * (size_t)B);
    int32_t *cnt = (int32_t *)at, *cur = cnt + buckets, *boff = cur + buckets;
    at += align256(sizeof(int32_t) * (size_t)(3 * buckets + 1));
    int32_t *lists = (int32_t *)at;               // written when the staged points are done with
    float4 *st_rec = (float4 *)at;
    const int64_t ib = cdiv64(buckets > 7 * (int64_t)B ? buckets : 7 * (int64_t)B, 256);
    hipLaunchKernelGGL(knn_init_kernel, dim3((unsigned)(ib < 8192 ? ib : 8192)), dim3(256), 0, s, bbox, B, cnt, buckets);
    const int bb = (N + 4095) / 4096;                      // four points per thread
    hipLaunchKernelGGL(knn_bbox_kernel, dim3(bb < 256 ? bb : 256, B), dim3(1024), 0, s, pos, bbox, N);
    auto deal = [&](auto points) {
        constexpr int P = points.value;
        const dim3 grid((unsigned)cdiv64(N, KNN_DEAL_NT * P), B);
        hipLaunchKernelGGL((knn_count_kernel<P>), grid, dim3(KNN_DEAL_NT), 0, s, pos, bbox, cnt, N, cpc, k);
        hipLaunchKernelGGL(knn_bucket_scan_kernel, dim3(B), dim3(1024), 0, s, cnt, boff, cur, N, k.n);
        hipLaunchKernelGGL((knn_deal_kernel<P>), grid, dim3(KNN_DEAL_NT), 0, s, pos, bbox, cur, st_rec, N, cpc, k);
    };
    // Fewer points a thread put more workgroups on the chip, each with all buckets to clear and to reserve in.  us of the whole search at
    // 1 | 2 | 4 points: 13k points 47.8 | 49.2 | 51.5, 100k 88.0 | 88.8 | 90.4, 300k 176.2 | 170.8 | 170.1, 8 clouds of 60k 256.2 | 255.2 |
    // 257.8, 1M 217.6 | 207.3 | 205.1.
    const int64_t all = (int64_t)B * N;
    if (all <= 1 << 17) deal(std::integral_constant<int, 1>{});
    else if (all <= 1 << 19) deal(std::integral_constant<int, 2>{});
    else deal(std::integral_constant<int, 4>{});
    const int64_t entries = (int64_t)B * N * K;
    const bool lanes = knn_lanes((int64_t)B * N, K) > 1, layers = lanes && entries > 7 << 15 && (int64_t)B * N > 1 << 14, rows = lanes && entries > 3 << 19;
    float *pairs = (float *)(bbox + 6 * (int64_t)B);
    hipLaunchKernelGGL(knn_sort_kernel, dim3(k.n, B), dim3(256), sizeof(int) << k.shift, s, boff, st_rec, bbox, rec, off, place, pairs, layers, rows, N,
                       cpc, k);
    const float few = rows ? 0.45f * (float)K * (float)N : -1.f;
#define FLEX_KNN_CASE(KK) \
    case KK: launch_knn_query<KK>(rec, off, bbox, lists, B, N, cpc, pairs, few, s); break;
    switch (K) {
        FLEX_KNN_KS(FLEX_KNN_CASE)
    default: return hipErrorInvalidValue;
    }
#undef FLEX_KNN_CASE
    int qb = (int)((N + 255) / 256);
    if (qb > 65535) qb = 65535;
    hipLaunchKernelGGL(knn_place_kernel, dim3(qb, B), dim3(256), 0, s, lists, place, nbr, N, K);
    return hipGetLastError();
}

bool knn_k_supported(int K)
{
    return (K >= 1 && K <= 10) || K == 12 || K == 16 || K == 24 || K == 32;
}

}  // namespace flex
