// Small support kernels: fp32 parameter packing, the partial-sum reduction of
// grad_theta, range check, zero fill, and the generic (any Din/Dout)
// direct-form flex-conv kernels used when no tiled kernel fits.
#include "flex_common.hpp"

namespace flex {

int device_cu_count()
{
    static int cached = 0;
    if (cached == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cached = n;
        else
            cached = 256;   // MI355X; also the answer on a host without a GPU
    }
    return cached;
}

int persistent_grid(int64_t total_tiles, int wg_per_cu)
{
    int64_t g = (int64_t)device_cu_count() * wg_per_cu;
    if (total_tiles < g) g = total_tiles;
    if (g < 8) g = 8;
    return (int)((g + 7) / 8 * 8);
}

// ---- theta packing ----------------------------------------------------------
__global__ void pack_theta_kernel(const float *__restrict__ theta, const float *__restrict__ bias,
                                  float *__restrict__ thetaP, int Din, int Dout, int RP, int CP,
                                  int transpose)
{
    const int total = 4 * RP * CP;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const int c = i % CP, r = (i / CP) % RP, j = i / (CP * RP);
        const int ci = transpose ? c : r;   // input channel
        const int co = transpose ? r : c;   // output channel
        float v = 0.f;
        if (ci < Din && co < Dout)
            v = (j < 3) ? theta[((int64_t)j * Din + ci) * Dout + co] : bias[(int64_t)ci * Dout + co];
        thetaP[i] = v;
    }
}

hipError_t launch_pack_theta(const float *theta, const float *bias, float *thetaP, int Din,
                             int Dout, int RP, int CP, int transpose, hipStream_t s)
{
    const int total = 4 * RP * CP;
    const int blocks = (total + 255) / 256;
    hipLaunchKernelGGL(pack_theta_kernel, dim3(blocks > 1024 ? 1024 : blocks), dim3(256), 0, s,
                       theta, bias, thetaP, Din, Dout, RP, CP, transpose);
    return hipGetLastError();
}

// ---- grad_theta partial reduction --------------------------------------------
// partials [n_wg][DEPTH][DOP] -> grad_theta [3,Din,Dout], grad_bias [Din,Dout]; the cross-workgroup sum runs in double
// and in a fixed order, so its error does not grow with n_wg and results are bit-reproducible.
// A workgroup owns 64 consecutive sums (256 bytes of every partial): 16 lanes of four floats per partial, 64 partials
// at a time over its 1024 threads, up to four such rounds requested together.  What bounds it is the latency of those
// reads, so everything a thread reads is in flight at once: 256 partials of 64 KB take 5.5 us; a 256-thread workgroup
// per row whose threads walked 64 partials each took 17.5.
struct ReduceArgs {
    int n_wg;                    // partials per block of the result
    int DIP, DOP;                // rows per component and columns of a partial
    int Din, Dout;               // the result's real widths
    int n_ho;                    // blocks of the result per row of blocks (blocks of DIP x DOP channels)
};

__device__ __forceinline__ void reduce_store(const ReduceArgs &p, int block, int e, double v,
                                             float *__restrict__ grad_theta, float *__restrict__ grad_bias)
{
    const int kd = e / p.DOP, o0 = e - kd * p.DOP;
    const int j = kd / p.DIP, bi = block / p.n_ho, bo = block - bi * p.n_ho;
    const int c = bi * p.DIP + kd - j * p.DIP, o = bo * p.DOP + o0;
    if (c >= p.Din || o >= p.Dout) return;
    (j < 3 ? grad_theta + (int64_t)j * p.Din * p.Dout : grad_bias)[(int64_t)c * p.Dout + o] = (float)v;
}

// Returns the sum that thread t < 64 stored (element 64 * segment + t).  GROUPS: partials at a time, 16 threads each.
template <int GROUPS>
__device__ __forceinline__ double reduce_segment(const float *__restrict__ partials, const ReduceArgs &p, int block,
                                                 int segment, float *__restrict__ grad_theta,
                                                 float *__restrict__ grad_bias, double (*s_sum)[64])
{
    constexpr int UN = 4;                    // rounds requested together
    const int64_t E = (int64_t)4 * p.DIP * p.DOP;
    const int tid = threadIdx.x, q = tid & 15, grp = tid >> 4, wave = tid >> 6;
    const float *src = partials + (int64_t)block * p.n_wg * E + 64 * (int64_t)segment + 4 * q;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int g0 = grp; g0 < p.n_wg; g0 += UN * GROUPS) {
        v4f x[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int g = g0 + GROUPS * u;
            x[u] = g < p.n_wg ? *reinterpret_cast<const v4f *>(src + g * E) : v4f{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] += (double)x[u][i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        sum[i] += __shfl_xor(sum[i], 16, 64);
        sum[i] += __shfl_xor(sum[i], 32, 64);
        if ((tid & 63) < 16) s_sum[wave][4 * q + i] = sum[i];
    }
    __syncthreads();
    if (tid >= 64) return 0.0;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < GROUPS / 4; ++w) v += s_sum[w][tid];
    reduce_store(p, block, 64 * segment + tid, v, grad_theta, grad_bias);
    return v;
}

// Few partials per block (a deep, wide layer has many blocks of the result and few workgroups on each): a thread per
// four elements reads them all.  512 x 512 channels, four partials per block: 9 us (61 in the form above, most of whose
// threads would have nothing to read).
constexpr int REDUCE_FEW = 16;
// Up to here 16 partials at a time, workgroups of 256 threads: most of 1024 would have nothing to read.  Parameter gradients, us (replayed
// from a graph), 64 partials at a time and 16: 32 -> 32, 1k points (32 partials) 7.97 and 7.71, 2k (64) 8.51 and 8.02, 4k (128) 9.13 and
// 9.07; 64 -> 64, 2k (64) 11.15 and 10.85, 4k (128) 13.27 and 13.20; 9 -> 64, 4k 8.57 and 8.55; 64 -> 128, 3k (47) 18.0 and 17.1, 20k (128)
// 33.8 and 33.5; 128 -> 128, 4k (64) 22.95 and 20.74, 24k (128) 37.4 and 37.1; 256 -> 256, 4k (16 blocks of 16 to 32) 43.3 and 32.5.
constexpr int REDUCE_SOME = 128;
__global__ __launch_bounds__(256) void reduce_partials_few_kernel(const float *__restrict__ partials, const ReduceArgs p,
                                                                  float *__restrict__ grad_theta,
                                                                  float *__restrict__ grad_bias)
{
    const int E = 4 * p.DIP * p.DOP, e = 4 * (blockIdx.x * 256 + threadIdx.x);
    if (e >= E) return;
    const float *src = partials + (int64_t)blockIdx.y * p.n_wg * E + e;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int g0 = 0; g0 < p.n_wg; g0 += 4) {
        v4f x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = *reinterpret_cast<const v4f *>(src + (int64_t)min(g0 + u, p.n_wg - 1) * E);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (g0 + u < p.n_wg)
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[i] += (double)x[u][i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) reduce_store(p, blockIdx.y, e + i, sum[i], grad_theta, grad_bias);
}

// grid: (64-element segments of a partial, blocks of the result)
template <int GROUPS>
__global__ __launch_bounds__(16 * GROUPS) void reduce_partials_kernel(const float *__restrict__ partials, const ReduceArgs p,
                                                                      float *__restrict__ grad_theta,
                                                                      float *__restrict__ grad_bias)
{
    __shared__ double s_sum[GROUPS / 4][64];
    reduce_segment<GROUPS>(partials, p, blockIdx.y, blockIdx.x, grad_theta, grad_bias, s_sum);
}

// The same, run only if the one-pass backward handed over (*flag != 0): the second reduction behind its fall-back.
__global__ __launch_bounds__(1024) void reduce_partials_if_kernel(const int *__restrict__ flag,
                                                                  const float *__restrict__ partials,
                                                                  const ReduceArgs p, float *__restrict__ grad_theta,
                                                                  float *__restrict__ grad_bias)
{
    __shared__ double s_sum[16][64];
    if (*flag == 0) return;
    reduce_segment<64>(partials, p, blockIdx.y, blockIdx.x, grad_theta, grad_bias, s_sum);
}

// n_blocks blocks of DIP x DOP channels, n_ho per row of blocks; block b's partials start at partials[b * n_wg].
hipError_t launch_reduce_partials(const float *partials, int n_wg, int DIP, int DOP, int n_blocks, int n_ho, int Din,
                                  int Dout, float *grad_theta, float *grad_bias, hipStream_t s)
{
    const ReduceArgs a{n_wg, DIP, DOP, Din, Dout, n_ho};
    if (n_wg <= REDUCE_FEW)
        hipLaunchKernelGGL(reduce_partials_few_kernel, dim3((4 * DIP * DOP + 1023) / 1024, (unsigned)n_blocks), dim3(256), 0,
                           s, partials, a, grad_theta, grad_bias);
    else if (n_wg <= REDUCE_SOME)
        hipLaunchKernelGGL(reduce_partials_kernel<16>, dim3(4 * DIP * DOP / 64, (unsigned)n_blocks), dim3(256), 0, s, partials,
                           a, grad_theta, grad_bias);
    else
        hipLaunchKernelGGL(reduce_partials_kernel<64>, dim3(4 * DIP * DOP / 64, (unsigned)n_blocks), dim3(1024), 0, s, partials,
                           a, grad_theta, grad_bias);
    return hipGetLastError();
}

hipError_t launch_reduce_partials_if(const int *flag, const float *partials, int n_wg, int DIP, int DOP, int Din,
                                     int Dout, float *grad_theta, float *grad_bias, hipStream_t s)
{
    hipLaunchKernelGGL(reduce_partials_if_kernel, dim3(4 * DIP * DOP / 64, 1), dim3(1024), 0, s, flag, partials,
                       ReduceArgs{n_wg, DIP, DOP, Din, Dout, 1}, grad_theta, grad_bias);
    return hipGetLastError();
}

// The first reduction of the one-pass backward (64 -> 64).  It leaves what the check of the result needs
// (fused_result_resolved): every workgroup its row's sum of squares, and one more workgroup Q_c from the workgroups'
// records; as doubles at FUSED_ROW_INT of record kd and FUSED_Q_INT of record c.
__global__ __launch_bounds__(1024) void reduce_partials_fused_kernel(const float *__restrict__ partials,
                                                                     const ReduceArgs p, int *__restrict__ control,
                                                                     float *__restrict__ grad_theta,
                                                                     float *__restrict__ grad_bias)
{
    __shared__ double s_sum[16][64];
    if (blockIdx.x + 1 < gridDim.x) {
        double v = reduce_segment<64>(partials, p, 0, blockIdx.x, grad_theta, grad_bias, s_sum);    // row kd = blockIdx.x
        if (threadIdx.x < 64) {
            v = (double)(float)v;
            v *= v;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d, 64);
            if (threadIdx.x == 0)
                *reinterpret_cast<double *>(control + FUSED_FLAG_INTS + (int64_t)blockIdx.x * FUSED_RECORD_INTS + FUSED_ROW_INT) = v;
        }
        return;
    }
    const int c = threadIdx.x & 63, part = threadIdx.x >> 6;
    double q = 0.0;
    constexpr int UN = 16;                           // records requested together
    for (int g0 = part; g0 < p.n_wg; g0 += 16 * UN) {
        int e[UN], n[UN], ce[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int g = min(g0 + u * 16, p.n_wg - 1);
            const int *rec = control + FUSED_FLAG_INTS + (int64_t)g * FUSED_RECORD_INTS;
            e[u] = rec[0]; n[u] = (g0 + u * 16 < p.n_wg) ? rec[1] : 0; ce[u] = rec[2 + c];
        }
#pragma unroll
        for (int u = 0; u < UN; ++u)
            if (n[u] > 0) q += __builtin_ldexp((double)n[u], -20 - 2 * (e[u] + ce[u]));
    }
    s_sum[part][c] = q;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    q = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) q += s_sum[w][c];
    *reinterpret_cast<double *>(control + FUSED_FLAG_INTS + (int64_t)c * FUSED_RECORD_INTS + FUSED_Q_INT) = q;
}

hipError_t launch_reduce_partials_fused(const float *partials, int n_wg, int *control, int Din, int Dout,
                                        float *grad_theta, float *grad_bias, hipStream_t s)
{
    if (n_wg > FUSED_MAX_WG) return hipErrorInvalidValue;
    hipLaunchKernelGGL(reduce_partials_fused_kernel, dim3(4 * 64 * 64 / 64 + 1), dim3(1024), 0, s, partials,
                       ReduceArgs{n_wg, 64, 64, Din, Dout, 1}, control, grad_theta, grad_bias);
    return hipGetLastError();
}

// ---- range check and zero fill --------------------------------------------------
__global__ void count_bad_kernel(const int32_t *__restrict__ nbr, int64_t count, int N,
                                 int32_t *__restrict__ bad)
{
    int local = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int v = nbr[i];
        local += (v < 0 || v >= N);
    }
    if (local) atomicAdd(bad, local);
}

hipError_t launch_count_bad(const int32_t *nbr, int64_t count, int N, int32_t *bad, hipStream_t s)
{
    hipError_t e = launch_fill_zero(bad, sizeof(int32_t), s);
    if (e != hipSuccess) return e;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(count_bad_kernel, dim3((unsigned)blocks), dim3(256), 0, s, nbr, count, N, bad);
    return hipGetLastError();
}

__global__ void fill_zero_kernel(uint32_t *__restrict__ p, int64_t words)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// bytes must be a multiple of 4 and ptr 4-byte aligned.
hipError_t launch_fill_zero(void *ptr, size_t bytes, hipStream_t s)
{
    const int64_t words = (int64_t)(bytes / 4);
    if (words == 0) return hipSuccess;
    int64_t blocks = (words + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t *)ptr, words);
    return hipGetLastError();
}

// ---- generic direct-form kernels ------------------------------------------------
// Element (b, c, l) of a [B,C,N] / [B,N,C] tensor.
__device__ __forceinline__ int64_t at(int bnc, int b, int c, int l, int C, int N)
{
    return bnc ? ((int64_t)b * N + l) * C + c : ((int64_t)b * C + c) * N + l;
}

__global__ void generic_fwd_kernel(const float *__restrict__ feat, const float *__restrict__ pos,
                                   const int32_t *__restrict__ nbr, const float *__restrict__ theta,
                                   const float *__restrict__ bias, float *__restrict__ out, int B,
                                   int N, int K, int Din, int Dout, int bnc)
{
    const int64_t total = (int64_t)B * N * Dout;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int o = (int)(i % Dout);
        const int64_t gp = i / Dout;
        const int b = (int)(gp / N), l = (int)(gp % N);
        const float *px = pos + (int64_t)b * 3 * N, *py = px + N, *pz = py + N;
        float acc = 0.f;
        for (int k = 0; k < K; ++k) {
            const int n = nbr[((int64_t)b * K + k) * N + l];
            const float dx = px[n] - px[l], dy = py[n] - py[l], dz = pz[n] - pz[l];
            for (int c = 0; c < Din; ++c) {
                const float w = theta[((int64_t)0 * Din + c) * Dout + o] * dx +
                                theta[((int64_t)1 * Din + c) * Dout + o] * dy +
                                theta[((int64_t)2 * Din + c) * Dout + o] * dz +
                                bias[(int64_t)c * Dout + o];
                acc = fmaf(w, feat[at(bnc, b, c, n, Din, N)], acc);
            }
        }
        out[at(bnc, b, o, l, Dout, N)] = acc;
    }
}

hipError_t launch_generic_fwd(const float *feat, const float *pos, const int32_t *nbr,
                              const float *theta, const float *bias, float *out, int B, int N,
                              int K, int Din, int Dout, int bnc, hipStream_t s)
{
    const int64_t total = (int64_t)B * N * Dout;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(generic_fwd_kernel, dim3((unsigned)blocks), dim3(256), 0, s, feat, pos, nbr,
                       theta, bias, out, B, N, K, Din, Dout, bnc);
    return hipGetLastError();
}

// grad_feat by scatter: one thread per (centre, slot, input channel).
__global__ void generic_grad_feat_kernel(const float *__restrict__ pos,
                                         const int32_t *__restrict__ nbr,
                                         const float *__restrict__ theta,
                                         const float *__restrict__ bias,
                                         const float *__restrict__ grad_out,
                                         float *__restrict__ grad_feat, int B, int N, int K, int Din,
                                         int Dout, int bnc)
{
    const int64_t total = (int64_t)B * N * K * Din;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % Din);
        const int64_t e = i / Din;
        const int k = (int)(e % K);
        const int64_t gp = e / K;
        const int b = (int)(gp / N), l = (int)(gp % N);
        const float *px = pos + (int64_t)b * 3 * N, *py = px + N, *pz = py + N;
        const int n = nbr[((int64_t)b * K + k) * N + l];
        const float dx = px[n] - px[l], dy = py[n] - py[l], dz = pz[n] - pz[l];
        float sum = 0.f;
        for (int o = 0; o < Dout; ++o) {
            const float w = theta[((int64_t)0 * Din + c) * Dout + o] * dx +
                            theta[((int64_t)1 * Din + c) * Dout + o] * dy +
                            theta[((int64_t)2 * Din + c) * Dout + o] * dz +
                            bias[(int64_t)c * Dout + o];
            sum = fmaf(w, grad_out[at(bnc, b, o, l, Dout, N)], sum);
        }
        atomicAdd(&grad_feat[at(bnc, b, c, n, Din, N)], sum);
    }
}

// grad_theta / grad_bias: block = (input channel c, chunk of centres); threads over o.
__global__ __launch_bounds__(256) void generic_grad_theta_kernel(
    const float *__restrict__ feat, const float *__restrict__ pos, const int32_t *__restrict__ nbr,
    const float *__restrict__ grad_out, float *__restrict__ grad_theta,
    float *__restrict__ grad_bias, int B, int N, int K, int Din, int Dout, int bnc,
    int64_t pts_per_chunk)
{
    const int c = blockIdx.x;
    const int64_t BN = (int64_t)B * N;
    const int64_t g0 = (int64_t)blockIdx.y * pts_per_chunk;
    const int64_t g1 = (g0 + pts_per_chunk < BN) ? g0 + pts_per_chunk : BN;
    for (int o0 = 0; o0 < Dout; o0 += 256) {
        const int o = o0 + threadIdx.x;
        float ax = 0.f, ay = 0.f, az = 0.f, ab = 0.f;
        for (int64_t gp = g0; gp < g1; ++gp) {
            const int b = (int)(gp / N), l = (int)(gp % N);
            const float *px = pos + (int64_t)b * 3 * N, *py = px + N, *pz = py + N;
            float sx = 0.f, sy = 0.f, sz = 0.f, sb = 0.f;
            for (int k = 0; k < K; ++k) {
                const int n = nbr[((int64_t)b * K + k) * N + l];
                const float f = feat[at(bnc, b, c, n, Din, N)];
                sx = fmaf(px[n] - px[l], f, sx);
                sy = fmaf(py[n] - py[l], f, sy);
                sz = fmaf(pz[n] - pz[l], f, sz);
                sb += f;
            }
            if (o < Dout) {
                const float g = grad_out[at(bnc, b, o, l, Dout, N)];
                ax = fmaf(sx, g, ax); ay = fmaf(sy, g, ay); az = fmaf(sz, g, az); ab = fmaf(sb, g, ab);
            }
        }
        if (o < Dout) {
            atomicAdd(&grad_theta[((int64_t)0 * Din + c) * Dout + o], ax);
            atomicAdd(&grad_theta[((int64_t)1 * Din + c) * Dout + o], ay);
            atomicAdd(&grad_theta[((int64_t)2 * Din + c) * Dout + o], az);
            atomicAdd(&grad_bias[(int64_t)c * Dout + o], ab);
        }
    }
}

hipError_t launch_generic_bwd(const float *feat, const float *pos, const int32_t *nbr,
                              const float *theta, const float *bias, const float *grad_out,
                              float *grad_feat, float *grad_theta, float *grad_bias, int B, int N,
                              int K, int Din, int Dout, int bnc, hipStream_t s)
{
    hipError_t e;
    if (grad_feat) {
        e = launch_fill_zero(grad_feat, sizeof(float) * (size_t)B * N * Din, s);
        if (e != hipSuccess) return e;
        const int64_t total = (int64_t)B * N * K * Din;
        int64_t blocks = (total + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(generic_grad_feat_kernel, dim3((unsigned)blocks), dim3(256), 0, s, pos, nbr,
                           theta, bias, grad_out, grad_feat, B, N, K, Din, Dout, bnc);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (grad_theta && grad_bias) {
        e = launch_fill_zero(grad_theta, sizeof(float) * (size_t)3 * Din * Dout, s);
        if (e != hipSuccess) return e;
        e = launch_fill_zero(grad_bias, sizeof(float) * (size_t)Din * Dout, s);
        if (e != hipSuccess) return e;
        const int64_t BN = (int64_t)B * N;
        int64_t chunks = (BN + 255) / 256;
        if (chunks > 1024) chunks = 1024;
        const int64_t per = (BN + chunks - 1) / chunks;
        chunks = (BN + per - 1) / per;
        hipLaunchKernelGGL(generic_grad_theta_kernel, dim3(Din, (unsigned)chunks), dim3(256), 0, s,
                           feat, pos, nbr, grad_out, grad_theta, grad_bias, B, N, K, Din, Dout, bnc, per);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---- location gradient, direct form (any shape) -------------------------------------
// one thread per edge (b, l, k): s_d = sum_{c,o} theta[d,c,o] feat[c,n] g[o,l]; +s_d to n, -s_d to l
__global__ __launch_bounds__(256) void generic_bwd_pos_kernel(const float *__restrict__ feat,
                                                              const int32_t *__restrict__ nbr,
                                                              const float *__restrict__ theta,
                                                              const float *__restrict__ grad_out,
                                                              float *__restrict__ grad_pos, int B, int N, int K,
                                                              int Din, int Dout, int bnc)
{
    const int64_t total = (int64_t)B * K * N;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int l = (int)(i % N);
        const int64_t bk = i / N;
        const int b = (int)(bk / K);
        const int n = nbr[i];
        if (n == l) continue;                       // a self edge adds and subtracts the same value
        float s[3] = {0.f, 0.f, 0.f};
        for (int c = 0; c < Din; ++c) {
            const float f = feat[at(bnc, b, c, n, Din, N)];
            float t0 = 0.f, t1 = 0.f, t2 = 0.f;
            for (int o = 0; o < Dout; ++o) {
                const float g = grad_out[at(bnc, b, o, l, Dout, N)];
                t0 = fmaf(theta[((int64_t)0 * Din + c) * Dout + o], g, t0);
                t1 = fmaf(theta[((int64_t)1 * Din + c) * Dout + o], g, t1);
                t2 = fmaf(theta[((int64_t)2 * Din + c) * Dout + o], g, t2);
            }
            s[0] = fmaf(f, t0, s[0]); s[1] = fmaf(f, t1, s[1]); s[2] = fmaf(f, t2, s[2]);
        }
        for (int d = 0; d < 3; ++d) {
            atomicAdd(&grad_pos[((int64_t)b * 3 + d) * N + n], s[d]);
            atomicAdd(&grad_pos[((int64_t)b * 3 + d) * N + l], -s[d]);
        }
    }
}

hipError_t launch_generic_bwd_pos(const float *feat, const int32_t *nbr, const float *theta,
                                  const float *grad_out, float *grad_pos, int B, int N, int K, int Din,
                                  int Dout, int bnc, hipStream_t s)
{
    hipError_t e = launch_fill_zero(grad_pos, sizeof(float) * (size_t)B * 3 * N, s);
    if (e != hipSuccess) return e;
    const int64_t total = (int64_t)B * K * N;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(generic_bwd_pos_kernel, dim3((unsigned)blocks), dim3(256), 0, s, feat, nbr, theta,
                       grad_out, grad_pos, B, N, K, Din, Dout, bnc);
    return hipGetLastError();
}

// ---- 1x1 convolution composed into the flex-convolution parameters (Sec. 4.3 block) ----------
// P = [theta; bias] as four [D x Dout] slabs j = 0..3.  Parameter-sized work, but cubic in the width (4 * 1024^3
// multiply-adds for a 1024-wide layer), so it runs as small LDS-tiled matrix products accumulated in double.  Layers that
// are wide enough to fill the device that way (256 workgroups of the 64 x 64 form) take 64 x 64 tiles, 4 x 4 results per
// thread, depth in steps of 16; the others, where a call is one workgroup's serial chain of loads, take 16 x 16 tiles
// with a result per thread, depth in steps of 64 requested a step ahead, and the four slabs side by side in the four
// 256-thread quarters of a workgroup (width 64: 14 -> 6 us forward, 47 -> 5 us back).
__device__ __forceinline__ const float *slab(const float *theta, const float *bias, int j, int D, int Dout)
{
    return j < 3 ? theta + (int64_t)j * D * Dout : bias;
}

// acc[i][jn] += sum_k A(m0 + ty*4 + i, k) * B(k, n0 + tx*4 + jn), A(m,k) = A[m*sam + k*sak], B(k,n) = B[k*sbk + n*sbn];
// elements outside M x K / K x N read as zero.  All 256 threads of the block must call it together.
__device__ __forceinline__ void tile_product(double (&acc)[4][4], const float *__restrict__ A, int64_t sam, int64_t sak,
                                             const float *__restrict__ B, int64_t sbk, int64_t sbn, int M, int N, int K,
                                             int m0, int n0, float (&As)[16][65], float (&Bs)[16][65])
{
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int idx = tid + 256 * e;
            // the unit-stride index runs fastest over the threads
            const int am = sam == 1 ? idx & 63 : idx >> 4, ak = sam == 1 ? idx >> 6 : idx & 15;
            const int bn = sbn == 1 ? idx & 63 : idx >> 4, bk = sbn == 1 ? idx >> 6 : idx & 15;
            As[ak][am] = (m0 + am < M && k0 + ak < K) ? A[(int64_t)(m0 + am) * sam + (int64_t)(k0 + ak) * sak] : 0.f;
            Bs[bk][bn] = (n0 + bn < N && k0 + bk < K) ? B[(int64_t)(k0 + bk) * sbk + (int64_t)(n0 + bn) * sbn] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            double a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = (double)As[k][ty * 4 + i]; b[i] = (double)Bs[k][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int jn = 0; jn < 4; ++jn) acc[i][jn] += a[i] * b[jn];
        }
        __syncthreads();
    }
}

__device__ __forceinline__ void tile_store(const double (&acc)[4][4], float *__restrict__ C, int64_t ldc, int M, int N,
                                           int m0, int n0)
{
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jn = 0; jn < 4; ++jn) {
            const int m = m0 + ty * 4 + i, n = n0 + tx * 4 + jn;
            if (m < M && n < N) C[(int64_t)m * ldc + n] = (float)acc[i][jn];
        }
}

// Pc[j][c0][o] = sum_c W[c][c0] * P[j][c][o]; grid (tiles over c0, tiles over o, 4 slabs)
__global__ __launch_bounds__(256) void compose_1x1_kernel(const float *__restrict__ W, const float *__restrict__ theta,
                                                          const float *__restrict__ bias, float *__restrict__ theta_c,
                                                          float *__restrict__ bias_c, int Din0, int Dmid, int Dout)
{
    __shared__ float As[16][65], Bs[16][65];
    const int j = blockIdx.z, m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    double acc[4][4] = {};
    tile_product(acc, W, 1, Din0, slab(theta, bias, j, Dmid, Dout), Dout, 1, Din0, Dout, Dmid, m0, n0, As, Bs);
    tile_store(acc, j < 3 ? theta_c + (int64_t)j * Din0 * Dout : bias_c, Dout, Din0, Dout, m0, n0);
}

// blockIdx.z < 4: gP[j][c][o] = sum_c0 W[c][c0] * gPc[j][c0][o], j = blockIdx.z (tiles over c and o);
// blockIdx.z == 4: gW[c][c0] = sum_{j,o} P[j][c][o] * gPc[j][c0][o] (tiles over c and c0).
__global__ __launch_bounds__(256) void compose_1x1_bwd_kernel(const float *__restrict__ W, const float *__restrict__ theta,
                                                              const float *__restrict__ bias,
                                                              const float *__restrict__ gtheta_c,
                                                              const float *__restrict__ gbias_c, float *__restrict__ gW,
                                                              float *__restrict__ gtheta, float *__restrict__ gbias,
                                                              int Din0, int Dmid, int Dout)
{
    __shared__ float As[16][65], Bs[16][65];
    const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    double acc[4][4] = {};
    if (blockIdx.z < 4) {
        const int j = blockIdx.z;
        if (m0 >= Dmid || n0 >= Dout) return;          // the grid covers the larger of the two tilings
        tile_product(acc, W, Din0, 1, slab(gtheta_c, gbias_c, j, Din0, Dout), Dout, 1, Dmid, Dout, Din0, m0, n0, As, Bs);
        tile_store(acc, j < 3 ? gtheta + (int64_t)j * Dmid * Dout : gbias, Dout, Dmid, Dout, m0, n0);
    } else {
        if (m0 >= Dmid || n0 >= Din0) return;
        for (int j = 0; j < 4; ++j)
            tile_product(acc, slab(theta, bias, j, Dmid, Dout), Dout, 1, slab(gtheta_c, gbias_c, j, Din0, Dout), 1, Dout,
                         Dmid, Din0, Dout, m0, n0, As, Bs);
        tile_store(acc, gW, Din0, Dmid, Din0, m0, n0);
    }
}

// ---- 16 x 16 tiles: quarter j of the workgroup computes slab j's product, a result per thread ----
constexpr int SMALL_T = 16, SMALL_K = 64;
struct SmallTiles { float A[4][SMALL_K][SMALL_T + 1], B[4][SMALL_K][SMALL_T + 1]; };

// sum_k A(m0 + ty, k) * B(k, n0 + tx) of this quarter's operands; every thread of the workgroup must call it
__device__ __forceinline__ double small_product(SmallTiles &sm, const float *__restrict__ A, int sam, int sak,
                                                const float *__restrict__ B, int sbk, int sbn, int M, int N, int K, int m0, int n0)
{
    const int j = threadIdx.x >> 8, tid = threadIdx.x & 255, tx = tid & 15, ty = tid >> 4;
    constexpr int E = SMALL_T * SMALL_K / 256;
    float a[E], b[E];
    int am[E], ak[E], bn[E], bk[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int idx = tid + 256 * e;
        // the unit-stride index runs fastest over the threads
        am[e] = sam == 1 ? idx & 15 : idx >> 6; ak[e] = sam == 1 ? idx >> 4 : idx & 63;
        bn[e] = sbn == 1 ? idx & 15 : idx >> 6; bk[e] = sbn == 1 ? idx >> 4 : idx & 63;
    }
    auto request = [&](int k0) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            a[e] = (m0 + am[e] < M && k0 + ak[e] < K) ? A[(int64_t)(m0 + am[e]) * sam + (int64_t)(k0 + ak[e]) * sak] : 0.f;
            b[e] = (n0 + bn[e] < N && k0 + bk[e] < K) ? B[(int64_t)(k0 + bk[e]) * sbk + (int64_t)(n0 + bn[e]) * sbn] : 0.f;
        }
    };
    request(0);
    double acc = 0.0;
    for (int k0 = 0; k0 < K; k0 += SMALL_K) {
#pragma unroll
        for (int e = 0; e < E; ++e) { sm.A[j][ak[e]][am[e]] = a[e]; sm.B[j][bk[e]][bn[e]] = b[e]; }
        __syncthreads();
        if (k0 + SMALL_K < K) request(k0 + SMALL_K);
#pragma unroll 16
        for (int k = 0; k < SMALL_K; ++k) acc += (double)sm.A[j][k][ty] * (double)sm.B[j][k][tx];
        __syncthreads();
    }
    return acc;
}

// as compose_1x1_kernel; grid (tiles over c0, tiles over o)
__global__ __launch_bounds__(1024) void compose_1x1_small_kernel(const float *__restrict__ W, const float *__restrict__ theta,
                                                                 const float *__restrict__ bias, float *__restrict__ theta_c,
                                                                 float *__restrict__ bias_c, int Din0, int Dmid, int Dout)
{
    __shared__ SmallTiles sm;
    const int j = threadIdx.x >> 8, m0 = blockIdx.x * SMALL_T, n0 = blockIdx.y * SMALL_T;
    const double v = small_product(sm, W, 1, Din0, slab(theta, bias, j, Dmid, Dout), Dout, 1, Din0, Dout, Dmid, m0, n0);
    const int m = m0 + ((threadIdx.x & 255) >> 4), n = n0 + (threadIdx.x & 15);
    float *C = j < 3 ? theta_c + (int64_t)j * Din0 * Dout : bias_c;
    if (m < Din0 && n < Dout) C[(int64_t)m * Dout + n] = (float)v;
}

// as compose_1x1_bwd_kernel; blockIdx.z 0: gP (tiles over c and o), 1: gW (tiles over c and c0, the quarters' sums added)
__global__ __launch_bounds__(1024) void compose_1x1_bwd_small_kernel(const float *__restrict__ W, const float *__restrict__ theta,
                                                                     const float *__restrict__ bias,
                                                                     const float *__restrict__ gtheta_c,
                                                                     const float *__restrict__ gbias_c, float *__restrict__ gW,
                                                                     float *__restrict__ gtheta, float *__restrict__ gbias,
                                                                     int Din0, int Dmid, int Dout)
{
    __shared__ SmallTiles sm;
    __shared__ double part[3][256];
    const int j = threadIdx.x >> 8, tid = threadIdx.x & 255, m0 = blockIdx.x * SMALL_T, n0 = blockIdx.y * SMALL_T;
    const int m = m0 + (tid >> 4), n = n0 + (tid & 15);
    const float *gPc = slab(gtheta_c, gbias_c, j, Din0, Dout);
    if (blockIdx.z == 0) {
        if (m0 >= Dmid || n0 >= Dout) return;          // the grid covers the larger of the two tilings
        const double v = small_product(sm, W, Din0, 1, gPc, Dout, 1, Dmid, Dout, Din0, m0, n0);
        float *C = j < 3 ? gtheta + (int64_t)j * Dmid * Dout : gbias;
        if (m < Dmid && n < Dout) C[(int64_t)m * Dout + n] = (float)v;
    } else {
        if (m0 >= Dmid || n0 >= Din0) return;
        const double v = small_product(sm, slab(theta, bias, j, Dmid, Dout), Dout, 1, gPc, 1, Dout, Dmid, Din0, Dout, m0, n0);
        if (j > 0) part[j - 1][tid] = v;
        __syncthreads();
        if (j == 0 && m < Dmid && n < Din0) gW[(int64_t)m * Din0 + n] = (float)(((v + part[0][tid]) + part[1][tid]) + part[2][tid]);
    }
}

// 64 x 64 tiles where those alone are a workgroup per CU; below, their few workgroups' serial chains decide
static bool compose_wide(int M, int N) { return (int64_t)((M + 63) / 64) * ((N + 63) / 64) * 4 >= 256; }

hipError_t launch_compose_1x1(const float *W, const float *theta, const float *bias, float *theta_c, float *bias_c,
                              int Din0, int Dmid, int Dout, hipStream_t s)
{
    if (!compose_wide(Din0, Dout)) {
        hipLaunchKernelGGL(compose_1x1_small_kernel, dim3((Din0 + SMALL_T - 1) / SMALL_T, (Dout + SMALL_T - 1) / SMALL_T), dim3(1024),
                           0, s, W, theta, bias, theta_c, bias_c, Din0, Dmid, Dout);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(compose_1x1_kernel, dim3((Din0 + 63) / 64, (Dout + 63) / 64, 4), dim3(256), 0, s, W, theta, bias,
                       theta_c, bias_c, Din0, Dmid, Dout);
    return hipGetLastError();
}

hipError_t launch_compose_1x1_bwd(const float *W, const float *theta, const float *bias, const float *gtheta_c,
                                  const float *gbias_c, float *gW, float *gtheta, float *gbias, int Din0, int Dmid,
                                  int Dout, hipStream_t s)
{
    const int n_max = Dout > Din0 ? Dout : Din0;
    if (!compose_wide(Dmid, n_max)) {
        hipLaunchKernelGGL(compose_1x1_bwd_small_kernel, dim3((Dmid + SMALL_T - 1) / SMALL_T, (n_max + SMALL_T - 1) / SMALL_T, 2),
                           dim3(1024), 0, s, W, theta, bias, gtheta_c, gbias_c, gW, gtheta, gbias, Din0, Dmid, Dout);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(compose_1x1_bwd_kernel, dim3((Dmid + 63) / 64, (n_max + 63) / 64, 5), dim3(256), 0, s, W, theta,
                       bias, gtheta_c, gbias_c, gW, gtheta, gbias, Din0, Dmid, Dout);
    return hipGetLastError();
}

}  // namespace flex
