// Flex-convolution from rows of at most 16 channels (gfx950, wave64): the forward pass of a network's first layer (colours,
// coordinates) and the feature gradient of its last one (class scores).  Compiled once per list form, -DFLEX_NARROW_CSR=.
//
// A lane is a point.  Its neighbours' rows are 4 * W bytes, so a row has no lanes to spread over: the wide kernels give a
// row sixteen lanes, of which a 9-channel one keeps nine busy, and spend some 300 instructions on four points.  Here a
// lane loads whole rows (eight of them under way), the position difference it weighs them with is its own, and the 4 W
// sums stay in its registers: no exchange between lanes until the sums of the wave's 64 points go through LDS, as
// split-half rows (flex_prep.hip), onto the f16 matrix cores.  Every wave works on tiles of its own, so nothing waits at a
// barrier; two waves per SIMD hide one's loads behind the other's products.
//
// What bounds it: the requests of the row and position loads (every lane its own line), not the bytes: 9 -> 64, 1M points,
// K = 8 in Z-order, 171 us by the sixteen-lane kernels, 136 here, of which the 336 MB touched once would take 54.
#include "flex_tile.hpp"

#if !defined(FLEX_NARROW_CSR)
#error "build with -DFLEX_NARROW_CSR"
#endif

#define FLEX_NARROW_CAT(a, b) a##b
#define FLEX_NARROW_NAME(a, b) FLEX_NARROW_CAT(a, b)

namespace flex {

// W floats at a byte offset of the buffer; zeros past its end
template <int W>
__device__ __forceinline__ void load_narrow(__amdgpu_buffer_rsrc_t rows, unsigned offset, float (&f)[W])
{
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    constexpr int W4 = W / 4 * 4, R = W - W4;
#pragma unroll
    for (int c = 0; c < W4; c += 4) {
        const v4f v = load_row4(rows, offset + 4u * c);
#pragma unroll
        for (int i = 0; i < 4; ++i) f[c + i] = v[i];
    }
    if constexpr (R >= 2) {
        const v2u v = __builtin_amdgcn_raw_buffer_load_b64(rows, (int)(offset + 4u * W4), 0, 0);
        f[W4] = __uint_as_float(v[0]);
        f[W4 + 1] = __uint_as_float(v[1]);
    }
    if constexpr (R & 1) f[W - 1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, (int)(offset + 4u * (W - 1)), 0, 0));
}

template <int W, bool CSR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void narrow_conv_kernel(const TileArgs a)
{
    constexpr int RP = W <= 8 ? 8 : 16, KD = 4 * RP, KS = KD / 32;       // packed rows per component, depth, depth steps
    constexpr int ARS = 4 * KD + 16;                                     // LDS row: [hi: KD halves][lo: KD halves][16 B]
    constexpr int U = CSR || W > 10 ? 4 : 8;                             // rows under way per lane
    constexpr int NS = 4;                                                // 16-channel slices of the output block
    __shared__ __attribute__((aligned(16))) char s_A[64 * ARS];

    const int j = blockIdx.x / a.chunks;
    const TileSchedule sc(a.total, (int)blockIdx.x - j * a.chunks, a.chunks);
    if (!(sc.first < sc.end)) return;
    const int lane = threadIdx.x, q = lane >> 4, r16 = lane & 15;
    const char *blk = a.theta + (int64_t)j * a.blk_bytes;
    const float *rscale = reinterpret_cast<const float *>(blk + a.rs_off);
    h8 tH[NS][KS], tL[NS][KS];
    v4i ec[NS];
#pragma unroll
    for (int n = 0; n < NS; ++n) {
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            tH[n][st] = *reinterpret_cast<const h8 *>(blk + ((n * KS + st) * 64 + lane) * 16);
            tL[n][st] = *reinterpret_cast<const h8 *>(blk + NS * KS * 1024 + ((n * KS + st) * 64 + lane) * 16);
        }
        ec[n] = *reinterpret_cast<const v4i *>(reinterpret_cast<const int *>(blk + a.exp_off) + 16 * n + 4 * q);
    }

    for (int tile = sc.first; tile < sc.end; tile += sc.step) {
        const int b = tile / a.tpc, l0 = (tile - b * a.tpc) * 64, at = min(l0 + lane, a.N - 1);
        const float *pos = a.pos + (int64_t)b * 3 * a.N;
        const auto rows = row_buffer(a.rows + (int64_t)b * a.N * a.rs, (unsigned)a.N * (unsigned)a.rs * 4u);
        const unsigned none = 0u - 4u * (unsigned)a.rs;                  // past the end of the rows: reads zeros
        int point = at, lo = 0, deg = a.K;
        if constexpr (CSR) {
            point = a.order[(int64_t)b * a.N + at];
            lo = a.off[(int64_t)b * a.N + point];
            deg = l0 + lane < a.N ? a.off[(int64_t)b * a.N + point + 1] - lo : 0;
        }
        const int most = CSR ? wave_max(deg) : a.K;
        float c[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) c[x] = pos[(int64_t)x * a.N + point];

        // ---- gather ----
        float acc[4][W];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int i = 0; i < W; ++i) acc[jj][i] = 0.f;
        for (int e0 = 0; e0 < most; e0 += U) {
            int id[U];
            float p[U][3], f[U][W];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = min(e0 + u, (CSR ? deg : a.K) - 1);
                if constexpr (CSR) id[u] = a.src[deg > 0 ? lo + e : 0];  // a list entry is always there (K >= 1)
                else id[u] = a.nbr[((int64_t)b * a.K + e) * a.N + point];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool has = e0 + u < deg;
                const int n = CSR && !has ? point : id[u];
                load_narrow<W>(rows, has ? (unsigned)n * (4u * (unsigned)a.rs) : none, f[u]);
#pragma unroll
                for (int x = 0; x < 3; ++x) p[u][x] = pos[(int64_t)x * a.N + n];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float sg = CSR ? -1.f : 1.f;                       // CSR: point - listing centre
                // a slot without an entry weighs its zeros with zero, wherever the point lies
                const bool has = e0 + u < deg;
                const float d0 = has ? sg * (p[u][0] - c[0]) : 0.f, d1 = has ? sg * (p[u][1] - c[1]) : 0.f,
                            d2 = has ? sg * (p[u][2] - c[2]) : 0.f;
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    acc[0][i] = fmaf(d0, f[u][i], acc[0][i]);
                    acc[1][i] = fmaf(d1, f[u][i], acc[1][i]);
                    acc[2][i] = fmaf(d2, f[u][i], acc[2][i]);
                    acc[3][i] += f[u][i];
                }
            }
        }

        // ---- the point's split-half row ----
        float m = 0.f;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int i = 0; i < W; ++i) {
                acc[jj][i] *= rscale[jj * RP + i];
                m = __builtin_amdgcn_fmed3f(m, __builtin_fabsf(acc[jj][i]), __builtin_inff());
            }
        const int ex = 15 - __builtin_amdgcn_frexp_expf(m);
        wave_lds_sync();                                                 // the rows of the tile before have been read
        char *row = s_A + lane * ARS;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int g = 0; g < RP / 8; ++g) {
                h8 h, l;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float x = 8 * g + i < W ? __builtin_ldexpf(acc[jj][8 * g + i < W ? 8 * g + i : 0], ex) : 0.f;
                    h[i] = (_Float16)x;
                    l[i] = (_Float16)(x - (float)h[i]);
                }
                *reinterpret_cast<h8 *>(row + 2 * (jj * RP + 8 * g)) = h;
                *reinterpret_cast<h8 *>(row + 2 * (KD + jj * RP + 8 * g)) = l;
            }
        wave_lds_sync();

        // ---- contract: 16 points at a time ----
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
            const char *arow = s_A + (16 * mb + r16) * ARS + 16 * q;
            v4f cc[NS];
#pragma unroll
            for (int n = 0; n < NS; ++n) cc[n] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < KS; ++st) {
                const h8 bh = *reinterpret_cast<const h8 *>(arow + 64 * st);
                const h8 bl = *reinterpret_cast<const h8 *>(arow + 64 * st + 2 * KD);
#pragma unroll
                for (int n = 0; n < NS; ++n) cc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tL[n][st], bh, cc[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NS; ++n) cc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tH[n][st], bl, cc[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NS; ++n) cc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tH[n][st], bh, cc[n], 0, 0, 0);
            }
            const int e = __shfl(ex, 16 * mb + r16, 64);
            const int l = CSR ? __shfl(point, 16 * mb + r16, 64) : l0 + 16 * mb + r16;
            if (l0 + 16 * mb + r16 >= a.N) continue;
#pragma unroll
            for (int n = 0; n < NS; ++n) {
                const int o = 64 * j + 16 * n + 4 * q;
                v4f d = cc[n];
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] = __builtin_ldexpf(d[i], -(e + ec[n][i]));
                float *dst = a.out + b * a.out_b + l * a.out_l + o * a.out_c;
                if (a.out_c == 1 && o + 3 < a.w_out) *reinterpret_cast<v4fu *>(dst) = d;
                else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (o + i < a.w_out) dst[i * a.out_c] = d[i];
                }
            }
        }
    }
}

hipError_t FLEX_NARROW_NAME(launch_narrow_, FLEX_NARROW_CSR)(const TileArgs &a, int grid, hipStream_t s)
{
    constexpr bool CSR = FLEX_NARROW_CSR != 0;
    switch (a.w_in) {
#define FLEX_NARROW_CASE(W) \
    case W: hipLaunchKernelGGL((narrow_conv_kernel<W, CSR>), dim3(grid), dim3(64), 0, s, a); break;
        FLEX_NARROW_CASE(1) FLEX_NARROW_CASE(2) FLEX_NARROW_CASE(3) FLEX_NARROW_CASE(4) FLEX_NARROW_CASE(5)
        FLEX_NARROW_CASE(6) FLEX_NARROW_CASE(7) FLEX_NARROW_CASE(8) FLEX_NARROW_CASE(9) FLEX_NARROW_CASE(10)
        FLEX_NARROW_CASE(11) FLEX_NARROW_CASE(12) FLEX_NARROW_CASE(13) FLEX_NARROW_CASE(14) FLEX_NARROW_CASE(15)
        FLEX_NARROW_CASE(16)
#undef FLEX_NARROW_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace flex
