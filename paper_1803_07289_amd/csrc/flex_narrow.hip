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

// A wave packs the parameters of an output block for itself, as pack_slice does (flex_prep.hip): the rows' scales to LDS, the
// fragments and column exponents to registers, the same bits.  What it costs, some 600 instructions a wave, is less than a launch in
// front of the kernel costs a call.  us, with that launch and here, called one after another (replayed from a graph): 9 -> 64, K = 8, 1024
// points 15.2 and 12.3 (10.5 and 9.8), 100k 18.8 and 17.2; 3 -> 32, 300 points 15.2 and 12.2 (9.2 and 5.9), 500k 31.0 and 27.9.
template <int W>
struct OwnParameters {
    static constexpr int RP = W <= 8 ? 8 : 16, KS = W <= 8 ? 1 : 2, NS = 4;
    float y[NS][KS][8];
    // a.theta, a.bias: the tensors; output block j
    __device__ __forceinline__ void request(const TileArgs &a, int j)
    {
        const int lane = threadIdx.x, q = lane >> 4, r16 = lane & 15;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            // eight rows of one component: kd = 32 * st + 8 * q ..
            const int jj = (32 * st + 8 * q) / RP, r0 = 8 * q % RP;
            const float *rows = jj < 3 ? reinterpret_cast<const float *>(a.theta) + (int64_t)jj * W * a.w_out : a.bias;
#pragma unroll
            for (int n = 0; n < NS; ++n) {
                const int col = 64 * j + 16 * n + r16;
                const float *at = rows + min(col, a.w_out - 1);
#pragma unroll
                for (int e = 0; e < 8; ++e) y[n][st][e] = at[min(r0 + e, W - 1) * a.w_out];      // past the tensor: a place inside it
            }
        }
        // all of them are asked for before any is looked at
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int n = 0; n < NS; ++n)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    asm volatile("" : "+v"(y[n][st][e]));
                    if (!(8 * q % RP + e < W && 64 * j + 16 * n + r16 < a.w_out)) y[n][st][e] = 0.f;
                }
    }
    __device__ __forceinline__ void pack(h8 (&tH)[NS][KS], h8 (&tL)[NS][KS], v4i (&ec)[NS], float *s_rs)
    {
        const int lane = threadIdx.x, q = lane >> 4, r16 = lane & 15;
        auto finite = [](float m, float x) {             // non-finite entries do not count
            const float v = __builtin_fabsf(x);
            return v < __builtin_inff() && v > m ? v : m;
        };
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float m = 0.f;
#pragma unroll
                for (int n = 0; n < NS; ++n) m = finite(m, y[n][st][e]);
                m = group_max<16>(m);
                const int er = m > 0.f ? min(max(-__builtin_amdgcn_frexp_expf(m), -60), 60) : 0;
#pragma unroll
                for (int n = 0; n < NS; ++n) y[n][st][e] = __builtin_ldexpf(y[n][st][e], er);
                if (r16 == 0) s_rs[32 * st + 8 * q + e] = __builtin_ldexpf(1.f, -er);
            }
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            float m = 0.f;
#pragma unroll
            for (int st = 0; st < KS; ++st)
#pragma unroll
                for (int e = 0; e < 8; ++e) m = finite(m, y[n][st][e]);
            m = fmaxf(m, __shfl_xor(m, 16, 64));
            m = fmaxf(m, __shfl_xor(m, 32, 64));
            const int x = m > 0.f ? 15 - __builtin_amdgcn_frexp_expf(m) : 0;
#pragma unroll
            for (int st = 0; st < KS; ++st)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = __builtin_ldexpf(y[n][st][e], x);
                    tH[n][st][e] = (_Float16)v;
                    tL[n][st][e] = (_Float16)(v - (float)tH[n][st][e]);
                }
#pragma unroll
            for (int i = 0; i < 4; ++i) ec[n][i] = __shfl(x, 4 * q + i, 64);
        }
        wave_lds_sync();
    }
};

// RAW: the parameters come as the caller has them (OwnParameters)
template <int W, bool CSR, bool RAW>
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
    __shared__ float s_rs[RAW ? KD : 1];
    h8 tH[NS][KS], tL[NS][KS];
    v4i ec[NS];
    if constexpr (RAW) {
        OwnParameters<W> own;
        own.request(a, j);
        own.pack(tH, tL, ec, s_rs);
    } else
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
                acc[jj][i] *= RAW ? s_rs[jj * RP + i] : rscale[jj * RP + i];
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

// ---- from records -------------------------------------------------------------------------------------------------
// With room in the workspace a point's location and row travel together as a 64-byte record (PrepList::records): four
// quads of floats, quad t = (component t of (x, y, z, 1), channels R t .. R t + 2), the fourth channel of R = 4 in a second
// array.  Four lanes are a point; each loads a quad, so a neighbour is ONE access of the texture path (two with R = 4)
// where a lane's own loads of its row and location are six.  What a lane holds is just what the 4 x 4 x 1 matrix op
// takes: lane t's location difference as the first operand (component t), a channel as the second, so the four lanes'
// sums need R ops a neighbour and no exchange at all.  Sixteen points of a cloud per wave, whose result leaves by whole rows; a
// workgroup's waves may serve several clouds (2048 clouds of 64 points, 9 -> 64, K = 8, the call: 29.3 us with tiles of 128 points
// of one cloud and the preparation likewise, 20.3 here).  The sums run in the order of the kernel above, and the result is the same bits.
//
// A wave serves its sixteen points and ends, and workgroups are dispatched in order, three of eight waves per CU.  What bounds it
// is the latency of what is not in a cache, ids above all, beside the result's stores.  A wave's loads and stores retire in
// the order they were issued, so in a wave that goes on to other points every load waits for the stores before it to reach
// memory, however far ahead it was asked for.  9 -> 64, K = 8, 1M points in Z-order, nothing in a cache: 129 us by the kernel
// above, 102 by three resident waves per SIMD, 96 here, 69 where the preparation has read the ids (make_records); the preparation 25 and 30.
template <int CTRL>
__device__ __forceinline__ unsigned quad_bcast(unsigned x) { return (unsigned)dpp_movi<CTRL>((int)x); }
__device__ __forceinline__ unsigned quad_lane(unsigned x, int slot)          // slot: a constant after unrolling
{
    return slot == 0 ? quad_bcast<0x00>(x) : slot == 1 ? quad_bcast<0x55>(x) : slot == 2 ? quad_bcast<0xAA>(x) : quad_bcast<0xFF>(x);
}

static constexpr int RECORD_NT = 512, RECORD_WAVES = RECORD_NT / 64;         // threads, waves per workgroup

template <int R, bool CSR>
__global__ __launch_bounds__(RECORD_NT) __attribute__((amdgpu_waves_per_eu(6, 6)))
void narrow_record_kernel(const TileArgs a, const float *__restrict__ rec, const float *__restrict__ rec4)
{
    constexpr int RP = R <= 2 ? 8 : 16, KD = 4 * RP, KS = KD / 32, ARS = 4 * KD + 32, NS = 4, U = 8;
    constexpr int ORS = 64 + 4;                                          // floats of a result row in LDS
    constexpr int WB = 16 * (ARS > 4 * ORS ? ARS : 4 * ORS);             // a wave's LDS: its split-half rows, then its result
    constexpr int TH = 2 * NS * KS * 1024;
    __shared__ __attribute__((aligned(16))) char s_th[TH];               // the parameters' fragments: [hi, lo][slice][step][lane]
    __shared__ __attribute__((aligned(16))) char s_w[RECORD_WAVES][WB];
    __shared__ __attribute__((aligned(16))) int s_ec[64];
    __shared__ __attribute__((aligned(16))) float s_rs[KD];

    // workgroup: output block, XCD's share of the workgroups, place in it; wave: cloud and first point (past the last wave's: past
    // the cloud, whose last point it gathers and does not store)
    const int j = blockIdx.x / a.chunks, w = blockIdx.x - j * a.chunks;
    const int wg = (w & 7) * (a.chunks >> 3) + (w >> 3);
    if (wg * RECORD_WAVES >= a.total) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), at_wave = wg * RECORD_WAVES + wave;
    const int b = __builtin_amdgcn_readfirstlane(min(at_wave, a.total - 1) / a.tpc);
    const int l0 = at_wave < a.total ? 16 * (at_wave - b * a.tpc) : a.N;
    const int lane = threadIdx.x & 63, p = lane >> 2, t = lane & 3, q = lane >> 4, r16 = lane & 15;
    const char *blk = a.theta + (int64_t)j * a.blk_bytes;

    // this lane's point (past the cloud's end its last one again) and the ids of its slots of the first batch: lane % 4 and four more
    int self = min(l0 + p, a.N - 1), lo = 0, deg = a.K;
    if constexpr (CSR) {
        self = a.order[(int64_t)b * a.N + self];
        lo = a.off[(int64_t)b * a.N + self];
        deg = a.off[(int64_t)b * a.N + self + 1] - lo;
    }
    auto ids = [&](int (&id)[2], int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = k0 + t + 4 * h;
            if constexpr (CSR) id[h] = a.src[k < deg ? lo + k : 0];      // a list entry is always there (K >= 1)
            else id[h] = a.nbr[((int64_t)b * a.K + min(k, a.K - 1)) * a.N + self];
        }
    };
    const unsigned lane_off = 16u * (unsigned)t, none = 0u - 64u;
    auto records = [&](const float *base, unsigned bytes) {
        return row_buffer(reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + (int64_t)b * a.N * bytes), (unsigned)a.N * bytes);
    };
    const auto rb = records(rec, 64u), rb4 = records(rec4, 16u);
    int id[2];
    ids(id, 0);
    // lane 3's component is the constant 1, in the neighbour's record and in the point's own
    const float own = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (int)((unsigned)self * 64u + lane_off), 0, 0));

    for (int i = threadIdx.x; i < TH / 16; i += RECORD_NT) *reinterpret_cast<v4i *>(s_th + 16 * i) = *reinterpret_cast<const v4i *>(blk + 16 * i);
    if (threadIdx.x < 64) s_ec[threadIdx.x] = reinterpret_cast<const int *>(blk + a.exp_off)[threadIdx.x];
    if (threadIdx.x < KD) s_rs[threadIdx.x] = reinterpret_cast<const float *>(blk + a.rs_off)[threadIdx.x];
    __syncthreads();

    // ---- gather ----
    const int most = CSR ? max(wave_max(deg), 1) : a.K;
    const float cen = t == 3 ? (CSR ? 2.f : 0.f) : own;
    v4f acc[R];                                                          // [channel][component]
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < most; k0 += U) {
        unsigned ro[2];                                                  // a slot without an entry: past the end, reads zeros
#pragma unroll
        for (int h = 0; h < 2; ++h) ro[h] = !CSR || k0 + t + 4 * h < deg ? (unsigned)id[h] * 64u : none;
        v4f f[U];
        float f4[R == 4 ? U : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned o = quad_lane(ro[u >> 2], u & 3) + lane_off;
            f[u] = load_row4(rb, o);
            if constexpr (R == 4) f4[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb4, (int)(o >> 2), 0, 0));
        }
        ids(id, k0 + U);                                                 // (past the last batch: read, not used)
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u < most) {
                float dp = CSR ? cen - f[u][0] : f[u][0] - cen;
                if (CSR) dp = k0 + u < deg ? dp : 0.f;                   // weighs its zeros with zero, wherever the point lies
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_4x4x1f32(dp, r < 3 ? f[u][1 + (r < 3 ? r : 0)] : f4[R == 4 ? u : 0], acc[r], 0, 0, 0);
            }
    }

    // ---- the points' split-half rows ----
    float m = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            acc[r][jj] *= s_rs[jj * RP + R * t + r];
            m = __builtin_amdgcn_fmed3f(m, __builtin_fabsf(acc[r][jj]), __builtin_inff());
        }
    m = group_max<4>(m);
    const int ex = 15 - __builtin_amdgcn_frexp_expf(m);
    char *row = s_w[wave] + p * ARS;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float x = __builtin_ldexpf(acc[r][jj], ex);
            const _Float16 h = (_Float16)x;
            *reinterpret_cast<_Float16 *>(row + 2 * (jj * RP + R * t + r)) = h;
            *reinterpret_cast<_Float16 *>(row + 2 * (KD + jj * RP + R * t + r)) = (_Float16)(x - (float)h);
        }
        if constexpr (4 * R < RP) {                                      // four channels of padding
            *reinterpret_cast<_Float16 *>(row + 2 * (jj * RP + 4 * R + t)) = (_Float16)0.f;
            *reinterpret_cast<_Float16 *>(row + 2 * (KD + jj * RP + 4 * R + t)) = (_Float16)0.f;
        }
    }
    wave_lds_sync();

    // ---- contract ----
    const char *arow = s_w[wave] + r16 * ARS + 16 * q;
    v4f cc[NS];
#pragma unroll
    for (int n = 0; n < NS; ++n) cc[n] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < KS; ++st) {
        const h8 bh = *reinterpret_cast<const h8 *>(arow + 64 * st);
        const h8 bl = *reinterpret_cast<const h8 *>(arow + 64 * st + 2 * KD);
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            const h8 tL = *reinterpret_cast<const h8 *>(s_th + (((NS + n) * KS + st) * 64 + lane) * 16);
            const h8 tH = *reinterpret_cast<const h8 *>(s_th + ((n * KS + st) * 64 + lane) * 16);
            cc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tL, bh, cc[n], 0, 0, 0);
            cc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tH, bl, cc[n], 0, 0, 0);
            cc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tH, bh, cc[n], 0, 0, 0);
        }
    }
    const int e = __shfl(ex, 4 * r16, 64);
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const v4i ec = *reinterpret_cast<const v4i *>(s_ec + 16 * n + 4 * q);
#pragma unroll
        for (int i = 0; i < 4; ++i) cc[n][i] = __builtin_ldexpf(cc[n][i], -(e + ec[i]));
    }
    if (a.out_c == 1) {
        // Point-major: through LDS, so that sixteen lanes write a point's row, 16 accesses a store where lanes of sixteen
        // different points take 64; streaming stores, which leave the records in L2
        float *s_out = reinterpret_cast<float *>(s_w[wave]);
        wave_lds_sync();                                                 // the split-half rows have been read
#pragma unroll
        for (int n = 0; n < NS; ++n) *reinterpret_cast<v4f *>(s_out + r16 * ORS + 16 * n + 4 * q) = cc[n];
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int pt = 4 * i + q, o = 64 * j + 4 * r16;
            const int l = CSR ? __shfl(self, 4 * pt, 64) : l0 + pt;
            const v4f d = *reinterpret_cast<const v4f *>(s_out + pt * ORS + 4 * r16);
            if (l0 + pt < a.N) {
                float *dst = a.out + b * a.out_b + l * a.out_l + o;
                if (o + 3 < a.w_out) __builtin_nontemporal_store(d, reinterpret_cast<v4fu *>(dst));
                else {
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        if (o + x < a.w_out) dst[x] = d[x];
                }
            }
        }
    } else {
        const int at = CSR ? __shfl(self, 4 * r16, 64) : l0 + r16;
        if (l0 + r16 >= a.N) return;
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            const int o = 64 * j + 16 * n + 4 * q;
            float *dst = a.out + b * a.out_b + at * a.out_l + o * a.out_c;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (o + i < a.w_out) dst[i * a.out_c] = cc[n][i];
        }
    }
}

hipError_t FLEX_NARROW_NAME(launch_narrow_records_, FLEX_NARROW_CSR)(const TileArgs &args, const float *rec, const float *rec4,
                                                                     int B, int n_out, hipStream_t s)
{
    constexpr bool CSR = FLEX_NARROW_CSR != 0;
    TileArgs a = args;                                   // tiles of this kernel's own: waves
    a.tpc = (a.N + 15) / 16;
    const int64_t total = (int64_t)B * a.tpc, chunks = (total + 8 * RECORD_WAVES - 1) / (8 * RECORD_WAVES) * 8;
    if (total > NARROW_RECORD_WAVES_MAX || chunks * n_out > 0x7fffffff) return hipErrorInvalidValue;
    a.total = (int)total;
    a.chunks = (int)chunks;
    const dim3 grid((unsigned)(chunks * n_out)), block(RECORD_NT);
    switch (narrow_record_channels(a.w_in)) {
    case 2: hipLaunchKernelGGL((narrow_record_kernel<2, CSR>), grid, block, 0, s, a, rec, rec4); break;
    case 3: hipLaunchKernelGGL((narrow_record_kernel<3, CSR>), grid, block, 0, s, a, rec, rec4); break;
    case 4:                                              // (the forward pass has no use for these)
        if constexpr (CSR) { hipLaunchKernelGGL((narrow_record_kernel<4, CSR>), grid, block, 0, s, a, rec, rec4); break; }
        [[fallthrough]];
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t FLEX_NARROW_NAME(launch_narrow_, FLEX_NARROW_CSR)(const TileArgs &a, int grid, hipStream_t s)
{
    constexpr bool CSR = FLEX_NARROW_CSR != 0;
    switch (a.w_in) {
#define FLEX_NARROW_CASE(W) \
    case W: \
        if constexpr (!CSR) if (a.bias != nullptr) { hipLaunchKernelGGL((narrow_conv_kernel<W, CSR, true>), dim3(grid), dim3(64), 0, s, a); break; } \
        hipLaunchKernelGGL((narrow_conv_kernel<W, CSR, false>), dim3(grid), dim3(64), 0, s, a); \
        break;
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
