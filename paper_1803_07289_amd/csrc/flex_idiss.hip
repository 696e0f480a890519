// Inverse density importance sub-sampling (Sec. 3.2): phi = sum of the distances to the K
// neighbours, then Ns points per cloud drawn with probability proportional to phi in one pass
// over the points (stratified sampling on the running sum).  Every decision of the draw is an
// integer comparison: phi is put on an integer scale of `bits` bits relative to the cloud's
// maximum (one float division, one float product per point), the running sums are 64-bit
// integers (exact in any summation order, so the parallel scan here and a sequential loop give
// the same table), the strata and thresholds are integer expressions of the caller's random
// words.
#include "flex_common.hpp"
#include <climits>

namespace flex {

static constexpr int IDISS_ITEMS = 8;                       // points per thread in the scans
static constexpr int IDISS_CHUNK = 256 * IDISS_ITEMS;       // points per block

// What bounds it is the lines that the neighbours' locations lie in.  PACKED: they come from records (x, y, z, 0) (pos4), one
// line each instead of three: 1M points of a room in the sensor's order, K = 8, 84 -> 45 us and 5 for the packing.  The point's own
// too, which some neighbour asks for anyway (Z-order, 2.9M points, tensors in a cache: the call 49.9 us with it from pos, 46.2).
template <bool PACKED>
__global__ __launch_bounds__(256) void idiss_phi_kernel(const float *__restrict__ pos, const float *__restrict__ pos4,
                                                        const int32_t *__restrict__ nbr, float *__restrict__ phi, int64_t BN,
                                                        int N, int K)
{
    constexpr int UN = 8;
    for (int64_t gp = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; gp < BN; gp += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = gp / N;
        const int l = (int)(gp - b * N);
        const float *p = pos + b * 3 * N;
        const v4f *p4 = reinterpret_cast<const v4f *>(pos4) + b * N;
        const int32_t *nb = nbr + b * K * N + l;
        float cx, cy, cz;
        if constexpr (PACKED) {
            const v4f me = p4[l];
            cx = me[0]; cy = me[1]; cz = me[2];
        } else {
            cx = p[l]; cy = p[(int64_t)N + l]; cz = p[2 * (int64_t)N + l];
        }
        // the ids of eight neighbours together, then their 24 position components: on a cloud stored without locality
        // every one of those is a line of its own, and what counts is how many are on their way
        float s = 0.f;
        for (int k0 = 0; k0 < K; k0 += UN) {
            int n[UN];
            float x[UN], y[UN], z[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) n[u] = nb[(int64_t)min(k0 + u, K - 1) * N];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                if constexpr (PACKED) {
                    const v4f q = p4[n[u]];
                    x[u] = q[0]; y[u] = q[1]; z[u] = q[2];
                } else {
                    x[u] = p[n[u]]; y[u] = p[(int64_t)N + n[u]]; z[u] = p[2 * (int64_t)N + n[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const float dx = x[u] - cx, dy = y[u] - cy, dz = z[u] - cz;
                if (k0 + u < K) s += sqrtf(dx * dx + dy * dy + dz * dz);
            }
        }
        phi[gp] = s;
    }
}

// per-cloud maximum; phi >= 0, so the float order is the order of the bit patterns
__global__ __launch_bounds__(1024) void idiss_max_kernel(const float *__restrict__ phi, unsigned *__restrict__ mx, int N)
{
    const int b = blockIdx.y;
    unsigned m = 0;
    for (int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; l < N; l += (int64_t)gridDim.x * blockDim.x)
        m = max(m, __float_as_uint(phi[(int64_t)b * N + l]));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d, 64));
    // one atomic per workgroup: they serialise on the cloud's word (one per wave of 489 workgroups: 25 us at 1M points)
    __shared__ unsigned s_max[16];
    if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < 16; ++w) m = max(m, s_max[w]);
        if (m) atomicMax(&mx[b], m);
    }
}

__device__ __forceinline__ unsigned idiss_quantum(float x, float mx, int bits)
{
    if (!(mx > 0.f)) return 1u;                                // coincident points: a uniform draw
    const float scale = (float)((int64_t)1 << bits) / mx;      // the same two float operations as the CPU check
    return (unsigned)(x * scale);
}

__device__ __forceinline__ unsigned long long block_exclusive_scan64(unsigned long long v, unsigned long long *s_wave,
                                                                     unsigned long long &block_total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned long long x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wave[w] = x;
    __syncthreads();
    unsigned long long base = 0;
    for (int i = 0; i < w; ++i) base += s_wave[i];
    block_total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    __syncthreads();
    return base + x - v;
}

// bsum[b][blk] = sum of the quanta of chunk blk of cloud b
__global__ __launch_bounds__(256) void idiss_chunk_sums_kernel(const float *__restrict__ phi,
                                                               const unsigned *__restrict__ mx,
                                                               unsigned long long *__restrict__ bsum, int N, int nblk,
                                                               int bits)
{
    __shared__ unsigned long long s_wave[4];
    const int b = blockIdx.y;
    const float m = __uint_as_float(mx[b]);
    const int64_t base = (int64_t)blockIdx.x * IDISS_CHUNK + (int64_t)threadIdx.x * IDISS_ITEMS;
    unsigned long long v = 0;
#pragma unroll
    for (int i = 0; i < IDISS_ITEMS; ++i)
        if (base + i < N) v += idiss_quantum(phi[(int64_t)b * N + base + i], m, bits);
    unsigned long long total;
    block_exclusive_scan64(v, s_wave, total);
    if (threadIdx.x == 0) bsum[(int64_t)b * (nblk + 1) + blockIdx.x] = total;
}

// one block per cloud: exclusive scan of its chunk sums in place; entry nblk = the cloud's total Q
__global__ __launch_bounds__(256) void idiss_scan_sums_kernel(unsigned long long *__restrict__ bsum, int nblk)
{
    __shared__ unsigned long long s_wave[4];
    unsigned long long *row = bsum + (int64_t)blockIdx.x * (nblk + 1);
    unsigned long long carry = 0;
    for (int c0 = 0; c0 < nblk; c0 += 256) {
        const int i = c0 + threadIdx.x;
        const unsigned long long v = (i < nblk) ? row[i] : 0;
        unsigned long long total;
        const unsigned long long ex = block_exclusive_scan64(v, s_wave, total);
        if (i < nblk) row[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) row[nblk] = carry;
}

// C[b][l] = inclusive running sum of the quanta
__global__ __launch_bounds__(256) void idiss_running_sum_kernel(const float *__restrict__ phi,
                                                                const unsigned *__restrict__ mx,
                                                                const unsigned long long *__restrict__ bsum,
                                                                unsigned long long *__restrict__ C, int N, int nblk,
                                                                int bits)
{
    __shared__ unsigned long long s_wave[4];
    const int b = blockIdx.y;
    const float m = __uint_as_float(mx[b]);
    const int64_t base = (int64_t)blockIdx.x * IDISS_CHUNK + (int64_t)threadIdx.x * IDISS_ITEMS;
    unsigned q[IDISS_ITEMS];
    unsigned long long sum = 0;
#pragma unroll
    for (int i = 0; i < IDISS_ITEMS; ++i) {
        q[i] = (base + i < N) ? idiss_quantum(phi[(int64_t)b * N + base + i], m, bits) : 0u;
        sum += q[i];
    }
    unsigned long long total;
    unsigned long long run = bsum[(int64_t)b * (nblk + 1) + blockIdx.x] + block_exclusive_scan64(sum, s_wave, total);
#pragma unroll
    for (int i = 0; i < IDISS_ITEMS; ++i) {
        run += q[i];
        if (base + i < N) C[(int64_t)b * N + base + i] = run;
    }
}

// The draw of stratum j: the first point whose running sum exceeds its threshold.  sum(l): the inclusive running sum of point l; Q: the last.
template <class Sum>
__device__ __forceinline__ int idiss_pick(Sum &&sum, unsigned long long Q, uint32_t u, int j, int N, int Ns)
{
    const unsigned long long width = Q / (unsigned long long)Ns, rem = Q % (unsigned long long)Ns;
    const unsigned long long jj = (unsigned long long)j;
    const unsigned long long start = jj * width + (jj < rem ? jj : rem);
    const unsigned long long len = width + (jj < rem ? 1u : 0u);
    const unsigned long long t = start + __umul64hi((unsigned long long)u << 32, len);
    int lo = 0, hi = N - 1;            // Q > t, so the last point always qualifies
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (sum(mid) > t) hi = mid; else lo = mid + 1;
    }
    return lo;
}

__global__ __launch_bounds__(256) void idiss_select_kernel(const unsigned long long *__restrict__ C,
                                                           const unsigned long long *__restrict__ bsum,
                                                           const uint32_t *__restrict__ u, int32_t *__restrict__ sel,
                                                           int N, int Ns, int nblk)
{
    const int b = blockIdx.y;
    const unsigned long long Q = bsum[(int64_t)b * (nblk + 1) + nblk];
    const unsigned long long *Cb = C + (int64_t)b * N;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < Ns; j += gridDim.x * blockDim.x)
        sel[(int64_t)b * Ns + j] = idiss_pick([&](int l) { return Cb[l]; }, Q, u[(int64_t)b * Ns + j], j, N, Ns);
}

// Clouds of up to IDISS_SMALL points: one workgroup per cloud, maximum, running sums (in LDS) and draw in one launch where the
// steps above are six.  What bounds either is the chain of launches and block-wide steps: 1k points 23.6 us, here 9.6; 16k 23.7 and 12.3.
static constexpr int IDISS_SMALL_NT = 1024, IDISS_SMALL_ITEMS = 16, IDISS_SMALL = IDISS_SMALL_NT * IDISS_SMALL_ITEMS;
// a place in an array that 16 consecutive entries of belong to a thread: one in seventeen is left out, for the banks
__device__ __forceinline__ int small_at(int i) { return i + (i >> 4); }

__global__ __launch_bounds__(IDISS_SMALL_NT) void idiss_sample_small_kernel(const float *__restrict__ phi, const uint32_t *__restrict__ u,
                                                                            int32_t *__restrict__ sel, int N, int Ns, int bits)
{
    extern __shared__ unsigned long long s_C[];                  // inclusive running sums of the quanta, small_at(N)
    __shared__ unsigned long long s_wave[IDISS_SMALL_NT / 64];
    __shared__ unsigned s_max[IDISS_SMALL_NT / 64];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    float x[IDISS_SMALL_ITEMS];
    unsigned m = 0;                                              // phi >= 0: the float order is the order of the bit patterns
#pragma unroll
    for (int i = 0; i < IDISS_SMALL_ITEMS; ++i) {
        const int l = tid + IDISS_SMALL_NT * i;
        x[i] = l < N ? phi[(int64_t)b * N + l] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < IDISS_SMALL_ITEMS; ++i) m = max(m, __float_as_uint(x[i]));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d, 64));
    if (lane == 0) s_max[w] = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IDISS_SMALL_NT / 64; ++i) m = max(m, s_max[i]);
#pragma unroll
    for (int i = 0; i < IDISS_SMALL_ITEMS; ++i) {
        const int l = tid + IDISS_SMALL_NT * i;
        if (l < N) s_C[small_at(l)] = idiss_quantum(x[i], __uint_as_float(m), bits);
    }
    __syncthreads();
    const int l0 = tid * IDISS_SMALL_ITEMS;
    unsigned long long sum = 0;
    for (int i = 0; i < IDISS_SMALL_ITEMS && l0 + i < N; ++i) sum += s_C[small_at(l0 + i)];
    unsigned long long run = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(run, d, 64);
        if (lane >= d) run += y;
    }
    if (lane == 63) s_wave[w] = run;
    __syncthreads();
    run -= sum;
    for (int i = 0; i < w; ++i) run += s_wave[i];
    for (int i = 0; i < IDISS_SMALL_ITEMS && l0 + i < N; ++i) {
        run += s_C[small_at(l0 + i)];
        s_C[small_at(l0 + i)] = run;
    }
    __syncthreads();
    const unsigned long long Q = s_C[small_at(N - 1)];
    for (int j = tid; j < Ns; j += IDISS_SMALL_NT)
        sel[(int64_t)b * Ns + j] = idiss_pick([&](int l) { return s_C[small_at(l)]; }, Q, u[(int64_t)b * Ns + j], j, N, Ns);
}

// ---- repeats removed from an ascending selection ---------------------------------------------
// Sequential rule: sel[j] = max(sel[j], sel[j-1] + 1), then sel[j] = min(sel[j], N - Ns + j).  The first is
// a running maximum of sel[i] - i (plus j), so it runs as a three-kernel scan; the second is elementwise.
__device__ __forceinline__ int block_inclusive_max(int v, int *s_wave, int &block_max)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x = max(x, y);
    }
    if (lane == 63) s_wave[w] = x;
    __syncthreads();
    int before = INT_MIN;
    for (int i = 0; i < w; ++i) before = max(before, s_wave[i]);
    block_max = max(max(s_wave[0], s_wave[1]), max(s_wave[2], s_wave[3]));
    __syncthreads();
    return max(before, x);
}

__global__ __launch_bounds__(256) void distinct_chunk_max_kernel(const int32_t *__restrict__ sel, int *__restrict__ cm,
                                                                 int Ns, int nblk)
{
    __shared__ int s_wave[4];
    const int b = blockIdx.y;
    const int64_t base = (int64_t)blockIdx.x * IDISS_CHUNK + (int64_t)threadIdx.x * IDISS_ITEMS;
    int v = INT_MIN;
#pragma unroll
    for (int i = 0; i < IDISS_ITEMS; ++i)
        if (base + i < Ns) v = max(v, sel[(int64_t)b * Ns + base + i] - (int)(base + i));
    int total;
    block_inclusive_max(v, s_wave, total);
    if (threadIdx.x == 0) cm[(int64_t)b * nblk + blockIdx.x] = total;
}

// one block per cloud: cm[blk] <- maximum over the chunks before blk (INT_MIN for the first)
__global__ __launch_bounds__(256) void distinct_scan_max_kernel(int *__restrict__ cm, int nblk)
{
    __shared__ int s_wave[4];
    __shared__ int s_inc[256];
    int *row = cm + (int64_t)blockIdx.x * nblk;
    int carry = INT_MIN;
    for (int c0 = 0; c0 < nblk; c0 += 256) {
        const int i = c0 + threadIdx.x;
        const int v = (i < nblk) ? row[i] : INT_MIN;
        int total;
        s_inc[threadIdx.x] = block_inclusive_max(v, s_wave, total);
        __syncthreads();
        const int before = threadIdx.x > 0 ? s_inc[threadIdx.x - 1] : INT_MIN;
        if (i < nblk) row[i] = max(carry, before);
        carry = max(carry, total);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void distinct_apply_kernel(int32_t *__restrict__ sel, const int *__restrict__ cm, int N,
                                                             int Ns, int nblk)
{
    __shared__ int s_wave[4];
    const int b = blockIdx.y;
    const int64_t base = (int64_t)blockIdx.x * IDISS_CHUNK + (int64_t)threadIdx.x * IDISS_ITEMS;
    int v[IDISS_ITEMS], mine = INT_MIN;
#pragma unroll
    for (int i = 0; i < IDISS_ITEMS; ++i) {
        v[i] = (base + i < Ns) ? sel[(int64_t)b * Ns + base + i] - (int)(base + i) : INT_MIN;
        mine = max(mine, v[i]);
    }
    int total;
    const int inc = block_inclusive_max(mine, s_wave, total);       // includes this thread's items
    // maximum over everything before this thread's first item
    __shared__ int s_inc[256];
    s_inc[threadIdx.x] = inc;
    __syncthreads();
    int run = max(cm[(int64_t)b * nblk + blockIdx.x], threadIdx.x > 0 ? s_inc[threadIdx.x - 1] : INT_MIN);
#pragma unroll
    for (int i = 0; i < IDISS_ITEMS; ++i) {
        run = max(run, v[i]);
        if (base + i < Ns) {
            const int j = (int)(base + i);
            sel[(int64_t)b * Ns + j] = min(run + j, N - Ns + j);
        }
    }
}

// Up to IDISS_SMALL kept points a cloud: the same in one launch, a workgroup per cloud (256 of them 12.9 us, here 7.2; 7.5k 12.7 and 7.1).
__global__ __launch_bounds__(IDISS_SMALL_NT) void distinct_small_kernel(int32_t *__restrict__ sel, int N, int Ns)
{
    extern __shared__ int s_v[];                                 // sel[j] - j, small_at(Ns)
    __shared__ int s_wave[IDISS_SMALL_NT / 64];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int32_t *mine = sel + (int64_t)b * Ns;
    for (int j = tid; j < Ns; j += IDISS_SMALL_NT) s_v[small_at(j)] = mine[j] - j;
    __syncthreads();
    const int j0 = tid * IDISS_SMALL_ITEMS;
    int most = INT_MIN;
    for (int i = 0; i < IDISS_SMALL_ITEMS && j0 + i < Ns; ++i) most = max(most, s_v[small_at(j0 + i)]);
    int run = most;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(run, d, 64);
        if (lane >= d) run = max(run, y);
    }
    if (lane == 63) s_wave[w] = run;
    run = __shfl_up(run, 1, 64);                                 // of the threads before
    if (lane == 0) run = INT_MIN;
    __syncthreads();
    for (int i = 0; i < w; ++i) run = max(run, s_wave[i]);
    for (int i = 0; i < IDISS_SMALL_ITEMS && j0 + i < Ns; ++i) {
        run = max(run, s_v[small_at(j0 + i)]);
        s_v[small_at(j0 + i)] = run;
    }
    __syncthreads();
    for (int j = tid; j < Ns; j += IDISS_SMALL_NT) mine[j] = min(s_v[small_at(j)], N - Ns) + j;
}

size_t distinct_ws_bytes(int B, int Ns) { return align256(sizeof(int) * (size_t)B * cdiv64(Ns, IDISS_CHUNK)); }

hipError_t launch_selection_make_distinct(int32_t *sel, int B, int N, int Ns, void *ws, hipStream_t s)
{
    if (Ns <= IDISS_SMALL) {
        hipLaunchKernelGGL(distinct_small_kernel, dim3(B), dim3(IDISS_SMALL_NT), sizeof(int) * (Ns + Ns / 16 + 1), s, sel, N, Ns);
        return hipGetLastError();
    }
    const int nblk = (int)cdiv64(Ns, IDISS_CHUNK);
    int *cm = (int *)ws;
    hipLaunchKernelGGL(distinct_chunk_max_kernel, dim3(nblk, B), dim3(256), 0, s, sel, cm, Ns, nblk);
    hipLaunchKernelGGL(distinct_scan_max_kernel, dim3(B), dim3(256), 0, s, cm, nblk);
    hipLaunchKernelGGL(distinct_apply_kernel, dim3(nblk, B), dim3(256), 0, s, sel, cm, N, Ns, nblk);
    return hipGetLastError();
}

int idiss_bits(int N)
{
    int lg = 0;
    while (((int64_t)1 << lg) < N) ++lg;
    return (51 - lg) < 28 ? (51 - lg) : 28;
}

static int idiss_nblk(int N) { return (int)cdiv64(N, IDISS_CHUNK); }

size_t idiss_ws_bytes(int B, int N)
{
    return align256(sizeof(unsigned long long) * (size_t)B * N) +
           align256(sizeof(unsigned long long) * (size_t)B * (idiss_nblk(N) + 1)) + align256(sizeof(unsigned) * (size_t)B);
}

// pos4: room for the records, 16 bytes a point, or null
hipError_t launch_idiss_phi(const float *pos, const int32_t *nbr, float *phi, float *pos4, int B, int N, int K, hipStream_t s)
{
    const int64_t BN = (int64_t)B * N;
    int64_t blocks = (BN + 255) / 256;
    if (blocks > (1 << 20)) blocks = 1 << 20;
    if (pos4 == nullptr) {
        hipLaunchKernelGGL(idiss_phi_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s, pos, pos4, nbr, phi, BN, N, K);
        return hipGetLastError();
    }
    PrepList prep;
    prep.pack_pos(pos, pos4, B, N);
    const hipError_t e = prep.launch(s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(idiss_phi_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, pos, pos4, nbr, phi, BN, N, K);
    return hipGetLastError();
}

hipError_t launch_idiss_sample(const float *phi, const uint32_t *u, int32_t *sel, int B, int N, int Ns, void *ws,
                               hipStream_t s)
{
    const int nblk = idiss_nblk(N), bits = idiss_bits(N);
    if (N <= IDISS_SMALL) {
        const size_t lds = sizeof(unsigned long long) * (size_t)(N + N / 16 + 1);
        hipLaunchKernelGGL(idiss_sample_small_kernel, dim3(B), dim3(IDISS_SMALL_NT), lds, s, phi, u, sel, N, Ns, bits);
        return hipGetLastError();
    }
    unsigned long long *C = (unsigned long long *)ws;
    unsigned long long *bsum = (unsigned long long *)((char *)ws + align256(sizeof(unsigned long long) * (size_t)B * N));
    unsigned *mx = (unsigned *)((char *)bsum + align256(sizeof(unsigned long long) * (size_t)B * (nblk + 1)));
    hipError_t e = launch_fill_zero(mx, sizeof(unsigned) * (size_t)B, s);
    if (e != hipSuccess) return e;
    const int mb = (N + 4095) / 4096;                      // four values per thread
    hipLaunchKernelGGL(idiss_max_kernel, dim3(mb < 256 ? mb : 256, B), dim3(1024), 0, s, phi, mx, N);
    hipLaunchKernelGGL(idiss_chunk_sums_kernel, dim3(nblk, B), dim3(256), 0, s, phi, mx, bsum, N, nblk, bits);
    hipLaunchKernelGGL(idiss_scan_sums_kernel, dim3(B), dim3(256), 0, s, bsum, nblk);
    hipLaunchKernelGGL(idiss_running_sum_kernel, dim3(nblk, B), dim3(256), 0, s, phi, mx, bsum, C, N, nblk, bits);
    int sb = (Ns + 255) / 256;
    if (sb > 4096) sb = 4096;
    hipLaunchKernelGGL(idiss_select_kernel, dim3(sb, B), dim3(256), 0, s, C, bsum, u, sel, N, Ns, nblk);
    return hipGetLastError();
}

}  // namespace flex
