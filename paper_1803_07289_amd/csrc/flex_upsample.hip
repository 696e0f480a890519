// Flex-upsampling (Sec. 4.1): the smaller layer's features are copied to their points in the
// larger layer, every other point counts as zero, and flex-max-pooling runs over the larger
// layer's neighbourhoods.  The zero-filled tensor is never written: an inverse map
// inv[b*Nf + m] = j (or -1) is built in the workspace and the pooling gather reads row
// inv[n] of the smaller layer, or takes 0.  Same tie rule as the pooling layer.
#include <climits>
#include "flex_common.hpp"

namespace flex {

// (value desc, point index asc): the winner among equal values is the lowest index.
__device__ __forceinline__ void take_up(float v, int n, float &bv, int &bn)
{
    // as selects (measured faster here than the short-circuit `if`, which compiles to exec-mask code; the plain
    // pooling kernel is the other way round and keeps the `if`)
    const bool better = (v > bv) | ((v == bv) & (n < bn));
    bv = better ? v : bv;
    bn = better ? n : bn;
}

__device__ __forceinline__ int64_t xcd_tile_up(int64_t total_tiles)
{
    const int64_t per_xcd = (total_tiles + 7) >> 3;
    const int64_t slot = blockIdx.x >> 3;
    const int64_t tile = (int64_t)(blockIdx.x & 7) * per_xcd + slot;
    return (slot < per_xcd && tile < total_tiles) ? tile : -1;
}
static inline unsigned xcd_grid_up(int64_t total_tiles) { return (unsigned)(((total_tiles + 7) >> 3) << 3); }

__global__ __launch_bounds__(256) void upsample_inv_fill_kernel(int32_t *__restrict__ inv, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        inv[i] = -1;
}

// inv[b*Nf + sel[b,j]] = j; entries of sel outside [0,Nf) are skipped (flex_validate_selection counts them)
__global__ __launch_bounds__(256) void upsample_inv_scatter_kernel(const int32_t *__restrict__ sel,
                                                                   int32_t *__restrict__ inv, int B, int Ns,
                                                                   int Nf)
{
    const int64_t total = (int64_t)B * Ns;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = i / Ns;
        const int m = sel[i];
        if (m >= 0 && m < Nf) inv[b * Nf + m] = (int)(i - b * Ns);
    }
}

// Point-major, C >= 4 (ODD: no multiple of four): a workgroup takes `points` consecutive points of the larger layer.  First eight lanes per point
// sort its neighbours out: those with a row in the smaller layer go to the point's list in LDS, all the zero-filled ones
// together are one candidate, the value 0 with the lowest of their indices.  Then a thread per (point, 4 channels) compares
// the rows of the list and that candidate.  What bounds it is the vector ALU and the chain neighbour -> inverse map -> row:
// compared one by one, the three quarters of the neighbours that are zero-filled cost as much as the others, and every lane
// of a point loaded the same ids and map entries (437.5k points x 128, K = 8, a quarter kept: 215 -> 138 us, of which the outputs alone are 72).
// K * points entries of LDS; points: a power of two, at most 32.  (C = 113, 500k points, a quarter kept: an element per thread 716 us
// and 377 backward, here 151 and 118.)
template <bool ODD>
__global__ __launch_bounds__(256) void upsample_fwd_bnc4_kernel(const float *__restrict__ feat_small,
                                                                const int32_t *__restrict__ inv,
                                                                const int32_t *__restrict__ nbr,
                                                                float *__restrict__ out,
                                                                int32_t *__restrict__ argmax, int64_t BN,
                                                                int Ns, int Nf, int K, int C, int points,
                                                                int64_t total_tiles)
{
    constexpr int U = 4;
    extern __shared__ int2 s_list[];               // [points][K]: (index in the larger layer, row of the smaller one)
    __shared__ int2 s_head[32];                    // (entries | first neighbour has a row << 30, lowest zero-filled index)
    const int64_t tile = xcd_tile_up(total_tiles);
    if (tile < 0) return;
    {
        const int slot = threadIdx.x & 7, p = threadIdx.x >> 3;
        const int64_t gp = tile * points + p;
        if (p < points && gp < BN) {               // whole groups of eight lanes take either side
            const int b = (int)(gp / Nf), l = (int)(gp % Nf);
            const int32_t *nb = nbr + (int64_t)b * K * Nf + l;
            const int32_t *iv = inv + (int64_t)b * Nf;
            int entries = 0, zero = INT_MAX, first = 0;
            for (int k0 = 0; k0 < K; k0 += 8) {
                const int k = k0 + slot;
                const int n = nb[(int64_t)min(k, K - 1) * Nf];
                const int j = iv[n];
                const bool has = k < K && j >= 0;
                zero = (k < K && j < 0) ? min(zero, n) : zero;
                const unsigned mask = (unsigned)(__ballot(has) >> (threadIdx.x & 56)) & 0xffu;
                if (has) s_list[p * K + entries + __popc(mask & ((1u << slot) - 1))] = make_int2(n, j);
                if (k0 == 0) first = mask & 1;
                entries += __popc(mask);
            }
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) zero = min(zero, __shfl_xor(zero, d, 64));
            if (slot == 0) s_head[p] = make_int2(entries | first << 30, zero);
        }
    }
    __syncthreads();
    const int C4 = ODD ? (C + 3) / 4 : C / 4;
    for (int i = threadIdx.x; i < points * C4; i += 256) {
        const int p = i / C4, c4 = i - p * C4;
        const int64_t gp = tile * points + p;
        if (gp >= BN) break;
        const int c0 = RowChunk<float, ODD>::first(c4, C);
        const float *rows = feat_small + gp / Nf * Ns * C + c0;
        const int2 head = s_head[p];
        const int entries = head.x & 0x3fffffff, zero = head.y;
        const int2 *list = s_list + p * K;
        // the first neighbour is what the others are compared with
        float v0 = 0.f, v1 = 0.f, v2 = 0.f, v3 = 0.f;
        int b0 = zero, b1 = zero, b2 = zero, b3 = zero;
        for (int e0 = 0; e0 < entries; e0 += U) {
            int2 en[U];
            v4f v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) en[u] = list[min(e0 + u, entries - 1)];        // past the end: the last entry again
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = RowChunk<float, ODD>::load(rows + (int64_t)en[u].y * C);
            if (e0 == 0 && head.x >> 30) {
                v0 = v[0].x; v1 = v[0].y; v2 = v[0].z; v3 = v[0].w;
                b0 = b1 = b2 = b3 = en[0].x;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                take_up(v[u].x, en[u].x, v0, b0);
                take_up(v[u].y, en[u].x, v1, b1);
                take_up(v[u].z, en[u].x, v2, b2);
                take_up(v[u].w, en[u].x, v3, b3);
            }
        }
        if (zero != INT_MAX) {
            take_up(0.f, zero, v0, b0);
            take_up(0.f, zero, v1, b1);
            take_up(0.f, zero, v2, b2);
            take_up(0.f, zero, v3, b3);
        }
        const v4f bv = {v0, v1, v2, v3};
        typedef int i4v __attribute__((ext_vector_type(4)));
        RowChunk<float, ODD>::store(out + gp * C + c0, c4, C, bv);
        const i4v bi = {b0, b1, b2, b3};
        RowChunk<int, ODD>::store(argmax + gp * C + c0, c4, C, bi);
    }
}

// Channel-major.  A workgroup owns 64 consecutive points of the larger layer: lane = point, so ids, outputs and winners move
// as whole 256-byte rows, and the four waves split the channels in chunks of CH.  First they sort the neighbours out as above,
// a quarter of the slots each: entries in slot order, lane by lane, in LDS.  Then a wave compares the entries of its points,
// CH x U four-byte values in flight per lane.  (An element per thread asked for every id and map entry once a channel: 235k points x
// 128, K = 16, 744 us, here 158; 1.46M x 64, K = 6, 1158 and 343; 26k x 128, K = 12, 72 and 31; 4k x 33 18.1 and 17.1.)
// Dynamic LDS: K * 64 entries.
template <int CH>
__global__ __launch_bounds__(256) void upsample_fwd_bcn_kernel(const float *__restrict__ feat_small, const int32_t *__restrict__ inv,
                                                               const int32_t *__restrict__ nbr, float *__restrict__ out,
                                                               int32_t *__restrict__ argmax, int Ns, int Nf, int K, int C,
                                                               int tiles_per_cloud, int64_t total_tiles)
{
    constexpr int U = 4;
    extern __shared__ int2 s_list[];               // [K][64]: (index in the larger layer, row of the smaller one)
    __shared__ int s_count[4][64], s_zero[4][64];  // per quarter of the slots: entries, lowest zero-filled index
    const int64_t tile = xcd_tile_up(total_tiles);
    if (tile < 0) return;
    const int64_t b = tile / tiles_per_cloud;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: channel rows get scalar base addresses
    const int l = (int)(tile - b * tiles_per_cloud) * 64 + lane, lc = min(l, Nf - 1);
    const int32_t *nb = nbr + b * K * Nf + lc, *iv = inv + b * Nf;
    const int per = (K + 3) / 4, k_from = w * per, k_to = min(K, k_from + per);
    int mine = 0, zero = INT_MAX;
    for (int k = k_from; k < k_to; ++k) {
        const int n = nb[(int64_t)k * Nf];
        const bool has = iv[n] >= 0;
        mine += has;
        zero = has ? zero : min(zero, n);
    }
    s_count[w][lane] = mine;
    s_zero[w][lane] = zero;
    __syncthreads();
    int entries = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q == w) mine = entries;                // where this wave's begin
        entries += s_count[q][lane];
        zero = min(zero, s_zero[q][lane]);
    }
    for (int k = k_from; k < k_to; ++k) {
        const int n = nb[(int64_t)k * Nf], j = iv[n];
        if (j >= 0) s_list[64 * mine++ + lane] = make_int2(n, j);
    }
    __syncthreads();
    // the first neighbour is what the others are compared with
    const bool first = iv[nb[0]] >= 0;
    int most = entries;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) most = max(most, __shfl_xor(most, d, 64));
    most = __builtin_amdgcn_readfirstlane(most);
    const int last = max(entries - 1, 0);
    for (int c0 = (blockIdx.y * 4 + w) * CH; c0 < C; c0 += 4 * CH * gridDim.y) {
        const char *row[CH];
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) row[ch] = reinterpret_cast<const char *>(feat_small + (b * C + min(c0 + ch, C - 1)) * Ns);
        float bv[CH];
        int bn[CH];
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) { bv[ch] = 0.f; bn[ch] = zero; }
        for (int e0 = 0; e0 < most; e0 += U) {
            int2 en[U];
            float v[CH][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {          // past the end: the last entry again; no entry: row 0, not looked at
                en[u] = s_list[64 * min(e0 + u, last) + lane];
                en[u].y = entries > 0 ? en[u].y : 0;
            }
#pragma unroll
            for (int ch = 0; ch < CH; ++ch)
#pragma unroll
                for (int u = 0; u < U; ++u) v[ch][u] = *reinterpret_cast<const float *>(row[ch] + 4u * (unsigned)en[u].y);
            if (entries > 0) {
#pragma unroll
                for (int ch = 0; ch < CH; ++ch) {
                    if (e0 == 0 && first) { bv[ch] = v[ch][0]; bn[ch] = en[0].x; }
#pragma unroll
                    for (int u = 0; u < U; ++u) take_up(v[ch][u], en[u].x, bv[ch], bn[ch]);
                }
            }
        }
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            if (zero != INT_MAX) take_up(0.f, zero, bv[ch], bn[ch]);
            if (l < Nf && c0 + ch < C) {
                const int64_t at = (b * C + c0 + ch) * Nf + l;
                __builtin_nontemporal_store(bv[ch], &out[at]);
                __builtin_nontemporal_store(bn[ch], &argmax[at]);
            }
        }
    }
}

// Any C, either layout: one thread per output element.
__global__ __launch_bounds__(256) void upsample_fwd_generic_kernel(const float *__restrict__ feat_small,
                                                                   const int32_t *__restrict__ inv,
                                                                   const int32_t *__restrict__ nbr,
                                                                   float *__restrict__ out,
                                                                   int32_t *__restrict__ argmax, int B, int Ns,
                                                                   int Nf, int K, int C, int bnc)
{
    const int64_t total = (int64_t)B * Nf * C;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        int b, c, l;
        if (bnc) { c = (int)(i % C); const int64_t gp = i / C; b = (int)(gp / Nf); l = (int)(gp % Nf); }
        else     { l = (int)(i % Nf); const int64_t bc = i / Nf; b = (int)(bc / C); c = (int)(bc % C); }
        const int32_t *nb = nbr + (int64_t)b * K * Nf + l;
        const int32_t *iv = inv + (int64_t)b * Nf;
        auto value = [&](int n) {
            const int j = iv[n];
            if (j < 0) return 0.f;
            return bnc ? feat_small[((int64_t)b * Ns + j) * C + c] : feat_small[((int64_t)b * C + c) * Ns + j];
        };
        int bn = nb[0];
        float bv = value(bn);
        for (int k = 1; k < K; ++k) {
            const int n = nb[(int64_t)k * Nf];
            take_up(value(n), n, bv, bn);
        }
        out[i] = bv;
        argmax[i] = bn;
    }
}

// Backward as a gather over the in-edge lists of the larger layer (sorted, repeats adjacent):
//   grad_small[j][c] = sum over centres l that list m = sel[j] of (argmax[l][c] == m ? grad_out[l][c] : 0)
template <bool ODD>
__global__ __launch_bounds__(256) void upsample_bwd_bnc4_kernel(
    const float *__restrict__ grad_out, const int32_t *__restrict__ argmax, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ in_off, const int32_t *__restrict__ in_src, float *__restrict__ grad_small,
    int64_t BNs, int Ns, int Nf, int C, int PT, int64_t total_tiles)
{
    constexpr int U = 4;
    typedef int i4v __attribute__((ext_vector_type(4)));
    const int C4 = ODD ? (C + 3) / 4 : C / 4;
    const int64_t tile = xcd_tile_up(total_tiles);
    if (tile < 0) return;
    for (int i = threadIdx.x; i < PT * C4; i += 256) {
        const int c4 = i % C4;
        const int64_t gj = tile * PT + i / C4;
        if (gj >= BNs) break;
        const int64_t b = gj / Ns;
        const int m = sel[gj];
        const int c0 = RowChunk<float, ODD>::first(c4, C);
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        if (m >= 0 && m < Nf) {
            const float *g_rows = grad_out + b * Nf * C + c0;
            const int32_t *a_rows = argmax + b * Nf * C + c0;
            const int64_t gp = b * Nf + m;
            const int e0 = in_off[gp], e1 = in_off[gp + 1];
            int prev = -1;
            for (int e = e0; e < e1; e += U) {
                int l[U];
                i4v a[U];
                v4f g[U];
#pragma unroll
                for (int u = 0; u < U; ++u) l[u] = in_src[min(e + u, e1 - 1)];     // past the end: the last entry again
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    a[u] = RowChunk<int, ODD>::load(a_rows + (int64_t)l[u] * C);
                    g[u] = RowChunk<float, ODD>::load(g_rows + (int64_t)l[u] * C);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool fresh = l[u] != prev;   // a centre that lists m twice routes one gradient
                    prev = l[u];
                    acc.x += (fresh && a[u].x == m) ? g[u].x : 0.f;
                    acc.y += (fresh && a[u].y == m) ? g[u].y : 0.f;
                    acc.z += (fresh && a[u].z == m) ? g[u].z : 0.f;
                    acc.w += (fresh && a[u].w == m) ? g[u].w : 0.f;
                }
            }
        }
        RowChunk<float, ODD>::template store<false>(grad_small + gj * C + c0, c4, C, acc);
    }
}

__global__ __launch_bounds__(256) void upsample_bwd_generic_kernel(
    const float *__restrict__ grad_out, const int32_t *__restrict__ argmax, const int32_t *__restrict__ sel,
    const int32_t *__restrict__ in_off, const int32_t *__restrict__ in_src, float *__restrict__ grad_small,
    int B, int Ns, int Nf, int C, int bnc)
{
    const int64_t total = (int64_t)B * Ns * C;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        int64_t b; int c, j;
        if (bnc) { c = (int)(i % C); const int64_t gj = i / C; b = gj / Ns; j = (int)(gj % Ns); }
        else     { j = (int)(i % Ns); const int64_t bc = i / Ns; b = bc / C; c = (int)(bc % C); }
        const int m = sel[b * Ns + j];
        float acc = 0.f;
        if (m >= 0 && m < Nf) {
            const int64_t gp = b * Nf + m;
            const int e1 = in_off[gp + 1];
            int prev = -1;
            for (int e = in_off[gp]; e < e1; ++e) {
                const int64_t l = in_src[e];
                if ((int)l == prev) continue;
                prev = (int)l;
                const int64_t at = bnc ? (b * Nf + l) * C + c : (b * C + c) * Nf + l;
                if (argmax[at] == m) acc += grad_out[at];
            }
        }
        grad_small[i] = acc;
    }
}

// number of sel entries outside [0,Nf) plus the number that repeat an earlier entry of their cloud
// (inv must hold the map built from the same sel)
__global__ __launch_bounds__(256) void upsample_check_sel_kernel(const int32_t *__restrict__ sel,
                                                                 const int32_t *__restrict__ inv, int B, int Ns,
                                                                 int Nf, int32_t *__restrict__ bad)
{
    const int64_t total = (int64_t)B * Ns;
    int mine = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = i / Ns;
        const int m = sel[i];
        if (m < 0 || m >= Nf) ++mine;
        else if (inv[b * Nf + m] != (int)(i - b * Ns)) ++mine;   // another entry of the cloud claimed m
    }
    if (mine) atomicAdd(bad, mine);
}

static unsigned capped_blocks(int64_t items, int64_t cap)
{
    int64_t blocks = (items + 255) / 256;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (unsigned)blocks;
}

hipError_t launch_upsample_inv(const int32_t *sel, int32_t *inv, int B, int Ns, int Nf, hipStream_t s)
{
    hipLaunchKernelGGL(upsample_inv_fill_kernel, dim3(capped_blocks((int64_t)B * Nf, 8192)), dim3(256), 0, s, inv,
                       (int64_t)B * Nf);
    hipLaunchKernelGGL(upsample_inv_scatter_kernel, dim3(capped_blocks((int64_t)B * Ns, 8192)), dim3(256), 0, s, sel,
                       inv, B, Ns, Nf);
    return hipGetLastError();
}

hipError_t launch_upsample_fwd(const float *feat_small, const int32_t *inv, const int32_t *nbr, float *out,
                               int32_t *argmax, int B, int Ns, int Nf, int K, int C, int bnc, hipStream_t s)
{
    // 32 points a workgroup (eight lanes each) as far as their lists fit 16 KB
    int points = 32;
    while (points > 1 && (int64_t)points * K > 2048) points >>= 1;
    const int64_t BN = (int64_t)B * Nf;
    // Fewer where a workgroup would go over its rows several times and the device is not full: us, 32 points and so, K = 8: 300 points x 113 10.2
    // and 7.5 (an element per thread 7.9), 3k x 113 11.3 and 8.2 (10.0), 3k x 256 14.7 and 8.4, 10k x 150 13.4 and 11.4, 10k x 33 9.0 and 8.6.
    while (bnc && points > 4 && (int64_t)points * C > 1024 && BN / points < 1024) points >>= 1;
    const int64_t tiles = (BN + points - 1) / points;
    if (bnc && C >= 4 && K <= 8192) {          // one point's list of up to 64 KB
        const auto kernel = C % 4 == 0 ? upsample_fwd_bnc4_kernel<false> : upsample_fwd_bnc4_kernel<true>;
        hipLaunchKernelGGL(kernel, dim3(xcd_grid_up(tiles)), dim3(256), sizeof(int2) * points * K, s, feat_small,
                           inv, nbr, out, argmax, BN, Ns, Nf, K, C, points, tiles);
    } else if (!bnc && K <= 64 && Ns < 1 << 30 && (K > 10 || BN * C * K >= 1 << 21)) {
        // Few outputs of few neighbours are sooner compared by a thread each than the neighbours sorted out: us, that and here, K = 8, 300 points x 64
        // 7.9 and 9.1, 1k x 128 8.5 and 9.5, 2k x 128 9.9 and 9.9, 2k x 256 13.0 and 12.1; K = 6, 4k x 64 9.4 and 9.9; K = 4, 8k x 64 10.7 and 9.9;
        // K = 16, 1k x 3 10.1 and 9.0, 1k x 64 10.2 and 10.0.
        const int tpc = (Nf + 63) / 64;
        const int64_t tiles64 = (int64_t)B * tpc;
        hipLaunchKernelGGL(upsample_fwd_bcn_kernel<4>, dim3(xcd_grid_up(tiles64), channel_parts(tiles64, C, 2048)), dim3(256),
                           sizeof(int2) * 64 * K, s, feat_small, inv, nbr, out, argmax, Ns, Nf, K, C, tpc, tiles64);
    } else {
        hipLaunchKernelGGL(upsample_fwd_generic_kernel, dim3(capped_blocks((int64_t)B * Nf * C, 1 << 20)), dim3(256),
                           0, s, feat_small, inv, nbr, out, argmax, B, Ns, Nf, K, C, bnc);
    }
    return hipGetLastError();
}

hipError_t launch_upsample_bwd(const float *grad_out, const int32_t *argmax, const int32_t *sel,
                               const int32_t *in_off, const int32_t *in_src, float *grad_small, int B, int Ns,
                               int Nf, int C, int bnc, hipStream_t s)
{
    if (bnc && C >= 4) {
        const int C4 = (C + 3) / 4;
        const int PT = C4 >= 256 ? 1 : 256 / C4;
        const int64_t BNs = (int64_t)B * Ns, tiles = (BNs + PT - 1) / PT;
        const auto kernel = C % 4 == 0 ? upsample_bwd_bnc4_kernel<false> : upsample_bwd_bnc4_kernel<true>;
        hipLaunchKernelGGL(kernel, dim3(xcd_grid_up(tiles)), dim3(256), 0, s, grad_out, argmax, sel,
                           in_off, in_src, grad_small, BNs, Ns, Nf, C, PT, tiles);
    } else if (!bnc && Nf < 1 << 30 && (int64_t)B * Ns * C * C >= (int64_t)147456 * ((C + 15) / 16 * 16)) {
        // Below that (outputs, with the channels of a workgroup that are missing taken off) an element per thread is all at once and
        // has no lists to set out.  us, it and here, a quarter kept, K = 8, Z-order | as drawn: 4k points x 128 9.4 and 9.4 | 9.7 and 11.3, 20k x 32 11.0 and
        // 10.0 | 12.1 and 12.2, 40k x 13 9.4 and 9.6 | 13.6 and 12.0, 80k x 3 7.8 and 11.9, 10k x 64 10.5 and 9.8 | 17.4 and 13.6; K = 32, 20k x 16 25
        // and 38, 20k x 32 37.5 and 37.3 | 44.9 and 41.1
        return launch_upsample_bwd_bcn(grad_out, argmax, sel, in_off, in_src, grad_small, B, Ns, Nf, C, s);
    } else {
        hipLaunchKernelGGL(upsample_bwd_generic_kernel, dim3(capped_blocks((int64_t)B * Ns * C, 1 << 20)), dim3(256),
                           0, s, grad_out, argmax, sel, in_off, in_src, grad_small, B, Ns, Nf, C, bnc);
    }
    return hipGetLastError();
}

hipError_t launch_upsample_check_sel(const int32_t *sel, const int32_t *inv, int B, int Ns, int Nf, int32_t *bad,
                                     hipStream_t s)
{
    hipError_t e = launch_fill_zero(bad, sizeof(int32_t), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(upsample_check_sel_kernel, dim3(capped_blocks((int64_t)B * Ns, 4096)), dim3(256), 0, s, sel,
                       inv, B, Ns, Nf, bad);
    return hipGetLastError();
}

}  // namespace flex
