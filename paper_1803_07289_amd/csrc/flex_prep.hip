// The steps in front of a call's main kernels -- packing the parameters, the walking order of the in-edge gathers,
// layout and width conversions of the feature tensors, clearing control words -- as jobs of ONE launch.  None of them
// depends on another, each is a few microseconds of latency and little bandwidth, and a launch of its own costs each of
// them about as much again (4 - 5 us); a call collects the ones it needs in a PrepList and every workgroup of the
// launch finds its job by its number.
#include "flex_common.hpp"

namespace flex {

// 512 threads and loops that are unrolled no further than the loads in flight ask for: a launch of a few workgroups is
// over in the time its instructions take to arrive, so the code executed in a straight line counts (256 threads with
// everything unrolled twice as far: 9 us for the packing at 64 x 64).
static constexpr int PREP_NT = 512, PREP_WAVES = PREP_NT / 64;

// ---- parameter packing for the split-half contraction ------------------------------
// The wave-specialised kernels contract on the f16 matrix cores with every fp32
// operand x carried as two halves of a scaled x:  hi = half(x s), lo = half(x s - hi),
// and the three products hi*hi + hi*lo + lo*hi (error ~2^-22 per product, the level
// of fp32 rounding) -- as long as x s stays within f16's normal range, i.e. within
// about 2^17 of the largest scaled magnitude.  Scaling by powers of two is exact, so the
// packing equilibrates the matrix first, in both directions:
//   row kd (a depth index: component j, gathered channel) gets 2^er[kd] so that its largest
//       magnitude is in [1/2, 1); the aggregate's column kd is multiplied by 2^-er[kd]
//       (rscale[kd], applied by the producers before their split), so a gathered channel of
//       small magnitude whose parameters are large (or the other way round) keeps its bits;
//   column o (an output channel) then gets 2^ec[o] so that its largest magnitude is in
//       [2^14, 2^15); the consumers undo it with the per-point exponent.
//   ThetaS[kd][o] = ThetaP[kd][o] * 2^(er[kd] + ec[o]);  out[l][o] = 2^-(e_l + ec[o]) * sum_kd As[l][kd] ThetaS[kd][o],
//   As[l][kd] = A[l][kd] * 2^-er[kd] * 2^e_l  (e_l: the point's own exponent, store_split_rows).
// What is left inside one row and column after that (entries of the SAME channel pair block far
// below their neighbours) contributes to the output in proportion to its size, as in any
// fp32 product.  er is clamped to +-60 so that no scale leaves fp32's normal range.
// Buffer layout (halves), the operand fragments of v_mfma_f32_16x16x32_f16 in the order
// a wave loads them:
//   thetaF[(((part*NS + slice)*KS + step)*64 + lane)*8 + e]
//       = part( ThetaS[32*step + 8*(lane>>4) + e][16*slice + (lane&15)] )
// with NS = CP/16 slices, KS = KDP/32 depth steps, rows >= 4*RP and padding zero; then, at
// byte offset theta_f16_exp_offset(RP, CP): int32 ec[CP], and at theta_f16_rscale_offset(RP, CP):
// float rscale[KDP] (1 for padding rows).
//
// One workgroup per 16-column slice.  The row scales need every column, so each workgroup reads the whole block (64 KB
// at 64 x 64, from L2) for the row maxima; its own columns' maxima and fragments it has to itself.  One workgroup for
// the whole block, which read it once, took 19 us at 64 x 64 and 43 us at 128 x 64 -- a single CU's latency chain and
// its LDS atomics --; the slices take 4 and 5.
struct PackArgs {
    int Din, Dout;        // the real tensor: [3,Din,Dout] and [Din,Dout]; everything outside reads as zero
    int RP, CP, n_i;      // rows per component and columns of a block; blocks along the rows
    int transpose;        // 0: rows = input channels, columns = output channels; 1: the other way round
    int block_bytes, exp_off, rs_off;
};

struct PackBlock {
    const float *theta, *bias;
    int Din, Dout, r0, c0, transpose;
    __device__ __forceinline__ int rows() const { return (transpose ? Dout : Din) - r0; }
    __device__ __forceinline__ int cols() const { return (transpose ? Din : Dout) - c0; }
    // channels (input, output) of (row, column)
    __device__ __forceinline__ int64_t at(int r, int c) const
    {
        return transpose ? (int64_t)(c0 + c) * Dout + r0 + r : (int64_t)(r0 + r) * Dout + c0 + c;
    }
};

// largest finite magnitude, the way the maxima are taken (non-finite entries do not count)
__device__ __forceinline__ float max_finite(float m, float x)
{
    const float a = fabsf(x);
    return (a < __builtin_inff() && a > m) ? a : m;
}

template <int CTRL>
__device__ __forceinline__ float dpp_max(float m)
{
    return fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), CTRL, 0xf, 0xf, true)));
}

// Row maxima of a block into s_er.  The tensor's contiguous index (output channel) runs over the lanes of a 16-lane
// group, four channels each; a group takes one component and every eighth input channel, UN rows requested together
// (addresses clamped instead of branches, so that nothing stands between the requests; a repeat changes no maximum).
// VEC: 16-byte reads.
template <bool VEC, bool TR>
__device__ __forceinline__ void pack_row_maxima(const PackBlock &v, int RP, int nr, int nc, int *s_er)
{
    constexpr int UN = VEC ? 8 : 4, STEP = PREP_NT / 64;
    const int l16 = threadIdx.x & 15, j = (threadIdx.x >> 4) & 3;
    const int ni = TR ? nc : nr, no = TR ? nr : nc;                     // input / output channels of the block
    const float *base = (j < 3 ? v.theta + (int64_t)j * v.Din * v.Dout : v.bias) +
                        (int64_t)(TR ? v.c0 : v.r0) * v.Dout + (TR ? v.r0 : v.c0);
#pragma unroll 1
    for (int o = 4 * l16; o - 4 * l16 < no; o += 64) {
        float mt[4] = {0.f, 0.f, 0.f, 0.f};             // TR: the maxima of rows (j, o .. o+3)
#pragma unroll 1
        for (int r0 = threadIdx.x >> 6; r0 < ni; r0 += STEP * UN) {
            v4f x[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const float *src = base + (int64_t)min(r0 + STEP * u, ni - 1) * v.Dout;
                if constexpr (VEC) x[u] = *reinterpret_cast<const v4f *>(src + min(o, no - 4));
                else x[u] = v4f{src[min(o, no - 1)], src[min(o + 1, no - 1)], src[min(o + 2, no - 1)], src[min(o + 3, no - 1)]};
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                if constexpr (TR) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) mt[i] = max_finite(mt[i], x[u][i]);
                } else {
                    float m = 0.f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) m = max_finite(m, x[u][i]);
                    m = dpp_max<0xB1>(m); m = dpp_max<0x4E>(m); m = dpp_max<0x141>(m); m = dpp_max<0x140>(m);
                    if (l16 == 0) atomicMax(&s_er[j * RP + min(r0 + STEP * u, ni - 1)], __float_as_int(m));
                }
            }
        }
        if constexpr (TR) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (o + i < no) atomicMax(&s_er[j * RP + o + i], __float_as_int(mt[i]));
        }
    }
}

// exponent e with |m| * 2^-e in [1/2, 1); 0 for m == 0
__device__ __forceinline__ int frexp_exp(float m) { return __builtin_amdgcn_frexp_expf(m); }

__device__ void pack_slice(const float *theta, const float *bias, char *thetaF_all, const PackArgs &p, int block,
                           char *lds)
{
    int *s_er = reinterpret_cast<int *>(lds);                   // [PACK_MAX_KD]
    int *s_ec = s_er + PACK_MAX_KD;                             // [16]
    const int NS = p.CP / 16, blk = block / NS, slice = block - blk * NS;
    const int j_blk = blk / p.n_i, i_blk = blk - j_blk * p.n_i;
    const PackBlock v{theta, bias, p.Din, p.Dout, p.RP * i_blk, p.CP * j_blk, p.transpose};
    const int KD = 4 * p.RP, KDP = (KD + 31) / 32 * 32, KS = KDP / 32;
    const int tid = threadIdx.x, l16 = tid & 15;
    const int nr = min(p.RP, v.rows()), nc = min(p.CP, v.cols());       // what exists of the block (may be nothing)
    for (int i = tid; i < PACK_MAX_KD; i += PREP_NT) s_er[i] = 0;
    if (tid < 16) s_ec[tid] = 0;
    __syncthreads();
    if (nr > 0 && nc > 0) {
        const int no = p.transpose ? nr : nc, co0 = p.transpose ? v.r0 : v.c0;
        const bool vec = ((p.Dout | co0 | no) & 3) == 0 &&
                         ((reinterpret_cast<uintptr_t>(theta) | reinterpret_cast<uintptr_t>(bias)) & 15) == 0;
        if (p.transpose) {
            if (vec) pack_row_maxima<true, true>(v, p.RP, nr, nc, s_er);
            else pack_row_maxima<false, true>(v, p.RP, nr, nc, s_er);
        } else {
            if (vec) pack_row_maxima<true, false>(v, p.RP, nr, nc, s_er);
            else pack_row_maxima<false, false>(v, p.RP, nr, nc, s_er);
        }
    }
    // this slice's elements: item = (step, lane), eight depth rows of one column
    constexpr int ITEMS = PACK_MAX_KD / 32 * 64 / PREP_NT;
    float y[ITEMS][8];
    const int col = 16 * slice + l16;
    const int64_t slab = (int64_t)p.Din * p.Dout;
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int item = tid + PREP_NT * t;
        if (item >= KS * 64) break;
        const int kd0 = 32 * (item >> 6) + 8 * ((item >> 4) & 3);
        int j = kd0 / p.RP, r = kd0 - j * p.RP;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool on = j < 4 && r < nr && col < nc;
            const float *src = (j < 3 ? theta + min(j, 2) * slab : bias) + (on ? v.at(r, col) : 0);
            const float x = *src;
            y[t][e] = on ? x : 0.f;
            if (++r == p.RP) { r = 0; ++j; }
        }
    }
    __syncthreads();
    _Float16 *thetaF = reinterpret_cast<_Float16 *>(thetaF_all + (size_t)blk * p.block_bytes);
    for (int kd = tid; kd < KDP; kd += PREP_NT) {
        const float m = __int_as_float(s_er[kd]);
        int er = m > 0.f ? -frexp_exp(m) : 0;
        er = er < -60 ? -60 : (er > 60 ? 60 : er);
        s_er[kd] = er;
        if (slice == 0)
            reinterpret_cast<float *>(reinterpret_cast<char *>(thetaF) + p.rs_off)[kd] = __builtin_ldexpf(1.f, -er);
    }
    __syncthreads();
    float mc = 0.f;
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int item = tid + PREP_NT * t;
        if (item >= KS * 64) break;
        const int kd0 = 32 * (item >> 6) + 8 * ((item >> 4) & 3);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            y[t][e] = __builtin_ldexpf(y[t][e], s_er[kd0 + e]);
            mc = max_finite(mc, y[t][e]);
        }
    }
    mc = fmaxf(mc, __shfl_xor(mc, 16, 64));
    mc = fmaxf(mc, __shfl_xor(mc, 32, 64));
    if ((tid & 63) < 16) atomicMax(&s_ec[l16], __float_as_int(mc));
    __syncthreads();
    const float m = __int_as_float(s_ec[l16]);
    const int ec = m > 0.f ? 15 - frexp_exp(m) : 0;
    if (tid < 16) reinterpret_cast<int *>(reinterpret_cast<char *>(thetaF) + p.exp_off)[col] = ec;
    const int per_part = NS * KS * 64 * 8;
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int item = tid + PREP_NT * t;
        if (item >= KS * 64) break;
        h8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float vs = __builtin_ldexpf(y[t][e], ec);
            hi[e] = (_Float16)vs;
            lo[e] = (_Float16)(vs - (float)hi[e]);
        }
        const int64_t at = ((int64_t)slice * KS * 64 + item) * 8;
        *reinterpret_cast<h8 *>(thetaF + at) = hi;
        *reinterpret_cast<h8 *>(thetaF + per_part + at) = lo;
    }
}

size_t theta_f16_exp_offset(int RP, int CP)
{
    const int KDP = (4 * RP + 31) / 32 * 32;
    return align256(sizeof(_Float16) * (size_t)2 * CP * KDP);
}
size_t theta_f16_rscale_offset(int RP, int CP) { return theta_f16_exp_offset(RP, CP) + align256(sizeof(int) * (size_t)CP); }
size_t theta_f16_bytes(int RP, int CP)
{
    const int KDP = (4 * RP + 31) / 32 * 32;
    return theta_f16_rscale_offset(RP, CP) + align256(sizeof(float) * (size_t)KDP);
}

// ---- theta fragments for the location-gradient kernel --------------------------------
// Theta_d = theta[d] (transpose == 0: depth = input channel, columns = output channel) or its
// transpose (transpose == 1), d = x, y, z, split-half with one exponent for all three:
//   thetaF[((((2*d + part)*NS + slice)*KS + step)*64 + lane)*8 + e]
//       = part( Theta_d[32*step + 8*(lane>>4) + e][16*slice + (lane&15)] * 2^e_theta ),
// NS = CP/16, KS = KDP/32, zero outside the matrix; int32 e_theta at theta_pos_exp_offset(KDP, CP).
// (r0, c0) / (nr, nc): the block of theta's input / output channels that is packed; entries outside theta are zero.
// One workgroup per (d, slice); the exponent needs every entry, so each workgroup reads the block once for it.
struct PackPosArgs {
    int Din, Dout, ci0, co0, KDP, CP, transpose, exp_off;
};

__device__ void pack_pos_slice(const float *theta, _Float16 *thetaF, const PackPosArgs &p, int block, char *lds)
{
    float *s_max = reinterpret_cast<float *>(lds);
    const int NS = p.CP / 16, KS = p.KDP / 32, d = block / NS, slice = block - d * NS;
    const int depth = p.transpose ? p.Dout - p.co0 : p.Din - p.ci0, cols = p.transpose ? p.Din - p.ci0 : p.Dout - p.co0;
    const int ni = min(p.transpose ? cols : depth, p.transpose ? p.CP : p.KDP);
    const int no = min(p.transpose ? depth : cols, p.transpose ? p.KDP : p.CP);
    const int tid = threadIdx.x;
    float m = 0.f;
    for (int o = tid & 63; o < no; o += 64)
        for (int r0 = tid >> 6; r0 < 3 * ni; r0 += PREP_WAVES * 8) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int row = min(r0 + PREP_WAVES * u, 3 * ni - 1), j = (row >= ni) + (row >= 2 * ni);   // repeats change no maximum
                x[u] = theta[((int64_t)j * p.Din + p.ci0 + row - j * ni) * p.Dout + p.co0 + o];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) m = fmaxf(m, fabsf(x[u]));
        }
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) m = fmaxf(m, __shfl_xor(m, w, 64));
    if ((tid & 63) == 0) s_max[tid >> 6] = m;
    __syncthreads();
    for (int w = 0; w < PREP_WAVES; ++w) m = fmaxf(m, s_max[w]);
    int ex = 0;
    if (m > 0.f && m < __builtin_inff()) ex = 15 - frexp_exp(m);
    if (block == 0 && tid == 0) *reinterpret_cast<int *>(reinterpret_cast<char *>(thetaF) + p.exp_off) = ex;
    const int per_part = NS * KS * 64 * 8;
    for (int item = tid; item < KS * 64; item += PREP_NT) {
        const int kd0 = 32 * (item >> 6) + 8 * ((item >> 4) & 3), col = 16 * slice + (item & 15);
        h8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int kd = kd0 + e, ci = p.ci0 + (p.transpose ? col : kd), co = p.co0 + (p.transpose ? kd : col);
            const bool on = ci < p.Din && co < p.Dout;
            const float x = theta[on ? ((int64_t)d * p.Din + ci) * p.Dout + co : 0];
            const float vs = __builtin_ldexpf(on ? x : 0.f, ex);
            hi[e] = (_Float16)vs;
            lo[e] = (_Float16)(vs - (float)hi[e]);
        }
        const int64_t at = ((int64_t)slice * KS * 64 + item) * 8;
        *reinterpret_cast<h8 *>(thetaF + (int64_t)(2 * d) * per_part + at) = hi;
        *reinterpret_cast<h8 *>(thetaF + (int64_t)(2 * d + 1) * per_part + at) = lo;
    }
}

size_t theta_pos_exp_offset(int KDP, int CP) { return align256(sizeof(_Float16) * (size_t)6 * CP * KDP); }
size_t theta_pos_bytes(int KDP, int CP) { return theta_pos_exp_offset(KDP, CP) + 256; }

// ---- walking order for the gathers over in-edge lists -----------------------------------------
// order[b*N + p] = the point that stands at position p of cloud b: inside every window of ORDER_WINDOW consecutive
// positions the window's points, sorted by the length of their in-edge list (lengths past 31 count as 31), points
// of equal length in index order.  A wave of the gather kernels takes four consecutive positions and a tile a few
// dozen, so their lists have (nearly) one length: no slot of a batch stays empty and no wave waits for a longer
// list at the tile's barrier, while a window is small enough for its gathered rows to stay in the caches.
// Four waves per window: lengths -> per (length, 64-point chunk) counts by ballots -> running sum in
// (length, chunk) order -> every point's place.
// The window is 13 tiles of 48 points: the persistent kernels deal tiles to workgroups with a stride that is a
// power of two, and a window of a power-of-two number of tiles would hand a workgroup the same place in every
// window, i.e. always the short or always the long lists.
static constexpr int ORDER_WINDOW = 624;
static constexpr int ORDER_CHUNKS = (ORDER_WINDOW + 63) / 64;  // 64-point chunks of a window
static constexpr int ORDER_NT = 256, ORDER_WAVES = ORDER_NT / 64;       // threads per window
static constexpr int ORDER_PER_BLOCK = PREP_NT / ORDER_NT;              // windows per workgroup
static constexpr int ORDER_ROUNDS = (ORDER_CHUNKS + ORDER_WAVES - 1) / ORDER_WAVES;    // chunks per wave
static constexpr int ORDER_BUCKETS = 32;
static_assert((ORDER_BUCKETS * ORDER_CHUNKS) % 64 == 0, "order: whole entries per lane in the running sum");

__device__ void order_window(const int32_t *__restrict__ off, int32_t *__restrict__ order, int N, int windows_per_cloud,
                             int windows, int block, char *lds)
{
    const int part = threadIdx.x / ORDER_NT, tid = threadIdx.x % ORDER_NT;      // window of the workgroup, thread in it
    int *s_cnt = reinterpret_cast<int *>(lds) + part * (ORDER_BUCKETS * ORDER_CHUNKS + ORDER_WINDOW);
    int *s_ord = s_cnt + ORDER_BUCKETS * ORDER_CHUNKS;         // [ORDER_WINDOW]; s_cnt: [length][chunk], then its exclusive running sum
    const int win = block * ORDER_PER_BLOCK + part;
    const int b = win / windows_per_cloud, w = win - b * windows_per_cloud;
    const int p0 = w * ORDER_WINDOW, n = win < windows ? min(ORDER_WINDOW, N - p0) : 0;
    const int lane = tid & 63, wave = tid >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    int len[ORDER_ROUNDS], rank[ORDER_ROUNDS];
#pragma unroll
    for (int r = 0; r < ORDER_ROUNDS; ++r) {
        const int chunk = r * ORDER_WAVES + wave, i = chunk * 64 + lane;
        len[r] = -1;
        if (i < n) {
            const int64_t g = (int64_t)b * N + p0 + i;
            len[r] = min(off[g + 1] - off[g], ORDER_BUCKETS - 1);
        }
        rank[r] = 0;
    }
    for (int i = tid; i < ORDER_BUCKETS * ORDER_CHUNKS; i += ORDER_NT) s_cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ORDER_ROUNDS; ++r) {
        const int chunk = r * ORDER_WAVES + wave;
        // one round per length that occurs in the chunk (about ten of the 32)
        uint64_t todo = __ballot(len[r] >= 0);
        while (todo) {
            const int d = __shfl(len[r], __ffsll((long long)todo) - 1, 64);     // wave-uniform
            const uint64_t m = __ballot(len[r] == d);
            if (len[r] == d) rank[r] = __popcll(m & lt);
            if (lane == 0) s_cnt[d * ORDER_CHUNKS + chunk] = __popcll(m);
            todo &= ~m;
        }
    }
    __syncthreads();
    if (wave == 0) {
        // exclusive running sum of the ORDER_BUCKETS * ORDER_CHUNKS counts: PER consecutive entries per lane
        constexpr int PER = ORDER_BUCKETS * ORDER_CHUNKS / 64;
        int v[PER], sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) { v[i] = s_cnt[lane * PER + i]; sum += v[i]; }
        int x = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        int run = x - sum;
#pragma unroll
        for (int i = 0; i < PER; ++i) { s_cnt[lane * PER + i] = run; run += v[i]; }
    }
    __syncthreads();
    // every point's place, through LDS so that the window leaves as one contiguous write
#pragma unroll
    for (int r = 0; r < ORDER_ROUNDS; ++r) {
        const int chunk = r * ORDER_WAVES + wave, i = chunk * 64 + lane;
        if (i < n) s_ord[s_cnt[len[r] * ORDER_CHUNKS + chunk] + rank[r]] = p0 + i;
    }
    __syncthreads();
    for (int i = tid; i < n; i += ORDER_NT) order[(int64_t)b * N + p0 + i] = s_ord[i];
}

size_t inedges_order_bytes(int64_t BN) { return align256(sizeof(int32_t) * (size_t)BN); }

// ---- copies between feature tensors of different layouts and widths ------------------------------
// dst[b, n, c] = src[b, n, c_off + c] where that channel exists, else 0, for c < Cd (so it transposes, pads with zero
// channels, keeps the leading ones, or cuts a column block out).  *_bcn: that tensor is channel-major.
// 64 points x 64 channels per workgroup through LDS, so that both sides are touched in their own contiguous
// direction (a thread per destination element, whatever the source's direction, took 103 us where this takes 9:
// 100 000 points, 64 point-major channels to channel-major).  vec: 16-byte accesses on both sides.
struct CopyArgs {
    int N, Cs, Cd, c_off, src_bcn, dst_bcn, tiles_n, tiles_c, vec;
};

__device__ void copy_tile(const float *__restrict__ src, float *__restrict__ dst, const CopyArgs &p, int64_t block,
                          char *lds)
{
    float (*tile)[65] = reinterpret_cast<float (*)[65]>(lds);   // [channel][point]
    const int tc = (int)(block % p.tiles_c);
    const int64_t bt = block / p.tiles_c;
    const int tn = (int)(bt % p.tiles_n);
    const int64_t b = bt / p.tiles_n;
    const int n0 = 64 * tn, c0 = 64 * tc;
    const float *s = src + b * (int64_t)p.N * p.Cs;
    float *d = dst + b * (int64_t)p.N * p.Cd;
    if (p.vec) {
        const int x = 4 * (threadIdx.x & 15), y = threadIdx.x >> 4;
        v4f v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int yy = y + 32 * i;
            v[i] = v4f{0.f, 0.f, 0.f, 0.f};
            if (p.src_bcn) {
                const int c = p.c_off + c0 + yy;
                if (c < p.Cs && n0 + x < p.N) v[i] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(s + (int64_t)c * p.N + n0 + x));
            } else {
                const int c = p.c_off + c0 + x;
                if (c < p.Cs && n0 + yy < p.N) v[i] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(s + (int64_t)(n0 + yy) * p.Cs + c));
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (p.src_bcn) tile[y + 32 * i][x + e] = v[i][e];
                else tile[x + e][y + 32 * i] = v[i][e];
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int yy = y + 32 * i;
            if (p.dst_bcn) {
                if (c0 + yy < p.Cd && n0 + x < p.N)
                    *reinterpret_cast<v4f *>(d + (int64_t)(c0 + yy) * p.N + n0 + x) =
                        v4f{tile[yy][x], tile[yy][x + 1], tile[yy][x + 2], tile[yy][x + 3]};
            } else {
                if (c0 + x < p.Cd && n0 + yy < p.N)
                    *reinterpret_cast<v4f *>(d + (int64_t)(n0 + yy) * p.Cd + c0 + x) =
                        v4f{tile[x][yy], tile[x + 1][yy], tile[x + 2][yy], tile[x + 3][yy]};
            }
        }
        return;
    }
    const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int yy = y + 8 * i;
        const int c = p.c_off + c0 + (p.src_bcn ? yy : x), n = n0 + (p.src_bcn ? x : yy);
        v[i] = (c < p.Cs && n < p.N) ? __builtin_nontemporal_load(p.src_bcn ? s + (int64_t)c * p.N + n : s + (int64_t)n * p.Cs + c) : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (p.src_bcn) tile[y + 8 * i][x] = v[i];
        else tile[x][y + 8 * i] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int yy = y + 8 * i;
        if (p.dst_bcn) {
            if (c0 + yy < p.Cd && n0 + x < p.N) d[(int64_t)(c0 + yy) * p.N + n0 + x] = tile[yy][x];
        } else {
            if (c0 + x < p.Cd && n0 + yy < p.N) d[(int64_t)(n0 + yy) * p.Cd + c0 + x] = tile[x][yy];
        }
    }
}

// ---- point locations as records ---------------------------------------------------------------------
// pos4[b*N + n] = (x, y, z, 0).  A gather asks the texture path for a cache line per quarter wave and component out of
// [B,3,N], for one per point out of these.
// Threads run over the points of all clouds (total: B * N), here and below.  In blocks of one cloud each, 16384 clouds of 16
// points, K = 8: 64 -> 64 forward 145 us, 130 here; 9 -> 64 from the records below 150 and 30.
static constexpr int POINTS_PER_THREAD = 4;

__device__ __forceinline__ unsigned cloud_of(unsigned g, int N, int total) { return total == N ? 0u : g / (unsigned)N; }

__device__ void pack_points(const float *__restrict__ pos, float *__restrict__ pos4, int N, int total, int block)
{
    const unsigned g0 = (unsigned)block * (PREP_NT * POINTS_PER_THREAD) + threadIdx.x;
    v4f *dst = reinterpret_cast<v4f *>(pos4);
    float x[POINTS_PER_THREAD][3];
#pragma unroll
    for (int i = 0; i < POINTS_PER_THREAD; ++i) {
        const unsigned g = min(g0 + PREP_NT * i, (unsigned)total - 1), b = cloud_of(g, N, total);
        const float *p = pos + (int64_t)b * 3 * N + (g - b * (unsigned)N);
#pragma unroll
        for (int d = 0; d < 3; ++d) x[i][d] = p[(int64_t)d * N];
    }
#pragma unroll
    for (int i = 0; i < POINTS_PER_THREAD; ++i)
        if (g0 + PREP_NT * i < (unsigned)total) dst[g0 + PREP_NT * i] = v4f{x[i][0], x[i][1], x[i][2], 0.f};
}

// ---- rows of at most 16 channels with their locations, as records -----------------------------------------------------
// rec[(b*N + n)*16 + 4 t ..] = (component t of (x, y, z, 1), channels R t .. R t + 2), rec4[(b*N + n)*4 + t] = channel 4 t + 3 (R = 4);
// channels past the row's end are zero.  A thread makes a quad: what a wave writes is contiguous.
// nbr: the neighbour tensor that the records are gathered by, read and dropped here, so that it stands in the memory-side cache
// (256 MB) when the gather waits for it; null where it is too large to stay there, or lists are walked.
struct RecordArgs {
    int N, total, W, bcn, K;             // total: B * N
    float *rec4;
    const int32_t *nbr;
};
static constexpr int RECORDS_PER_THREAD = 2;

__device__ void make_records(const float *__restrict__ pos, const float *__restrict__ feat, float *__restrict__ rec,
                             const RecordArgs &p, int block)
{
    constexpr int PER_BLOCK = PREP_NT / 4 * RECORDS_PER_THREAD;
    const int t = threadIdx.x & 3, R = narrow_record_channels(p.W);
    const unsigned first = (unsigned)block * PER_BLOCK;                  // below total
    const int64_t sn = p.bcn ? 1 : p.W, sc = p.bcn ? p.N : 1;
#pragma unroll
    for (int i = 0; i < RECORDS_PER_THREAD; ++i) {
        const unsigned n = first + (threadIdx.x >> 2) + PREP_NT / 4 * i, g = min(n, (unsigned)p.total - 1), b = cloud_of(g, p.N, p.total);
        const int64_t at = g - b * (unsigned)p.N;
        const float *f = feat + (int64_t)b * p.N * p.W;
        const float x = pos[((int64_t)b * 3 + min(t, 2)) * p.N + at];
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = R * t + r;
            v[r] = 0.f;
            if (r < R) {
                const float y = f[at * sn + min(c, p.W - 1) * sc];
                v[r] = c < p.W ? y : 0.f;
            }
        }
        if (n < (unsigned)p.total) {
            reinterpret_cast<v4f *>(rec)[(int64_t)n * 4 + t] = v4f{t < 3 ? x : 1.f, v[0], v[1], v[2]};
            if (R == 4) p.rec4[(int64_t)n * 4 + t] = v[3];
        }
    }
    if (p.nbr != nullptr) {
        const unsigned g = min(first + threadIdx.x % PER_BLOCK, (unsigned)p.total - 1), b = cloud_of(g, p.N, p.total);
        const int32_t *ids = p.nbr + (int64_t)b * p.K * p.N + (g - b * (unsigned)p.N);
        for (int k = threadIdx.x / PER_BLOCK; k < p.K; k += 4 * (PREP_NT / PER_BLOCK)) {
            int x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = ids[(int64_t)min(k + u * (PREP_NT / PER_BLOCK), p.K - 1) * p.N];
#pragma unroll
            for (int u = 0; u < 4; ++u) asm volatile("" : : "v"(x[u]));
        }
    }
}

// ---- the launch ----------------------------------------------------------------------------------
struct PrepJob {
    int kind, blocks;
    const void *a, *b;
    void *dst;
    union {
        PackArgs pack;
        PackPosArgs pos;
        CopyArgs copy;
        struct { int N, wpc, windows; } order;
        struct { int N, total; } points;
        RecordArgs records;
        struct { int words; } clear;
    };
};
enum { PREP_PACK, PREP_PACK_POS, PREP_ORDER, PREP_COPY, PREP_POINTS, PREP_RECORDS, PREP_CLEAR };
static_assert(sizeof(PrepJob) <= PREP_JOB_BYTES, "PrepList's storage");
struct PrepJobs {
    PrepJob job[PREP_MAX_JOBS];
};

__global__ __launch_bounds__(PREP_NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void prep_kernel(const PrepJobs jobs)
{
    __shared__ __attribute__((aligned(16))) char lds[64 * 65 * sizeof(float)];
    static_assert(sizeof(lds) >= sizeof(int) * (PACK_MAX_KD + 16) &&
                  sizeof(lds) >= sizeof(int) * ORDER_PER_BLOCK * (ORDER_BUCKETS * ORDER_CHUNKS + ORDER_WINDOW), "LDS of every job");
    int block = blockIdx.x, i = 0;
    while (block >= jobs.job[i].blocks) { block -= jobs.job[i].blocks; ++i; }     // the grid is the sum of the blocks
    const PrepJob &j = jobs.job[i];
    switch (j.kind) {
    case PREP_PACK:
        pack_slice((const float *)j.a, (const float *)j.b, (char *)j.dst, j.pack, block, lds);
        break;
    case PREP_PACK_POS:
        pack_pos_slice((const float *)j.a, (_Float16 *)j.dst, j.pos, block, lds);
        break;
    case PREP_ORDER:
        order_window((const int32_t *)j.a, (int32_t *)j.dst, j.order.N, j.order.wpc, j.order.windows, block, lds);
        break;
    case PREP_COPY:
        copy_tile((const float *)j.a, (float *)j.dst, j.copy, block, lds);
        break;
    case PREP_POINTS:
        pack_points((const float *)j.a, (float *)j.dst, j.points.N, j.points.total, block);
        break;
    case PREP_RECORDS:
        make_records((const float *)j.a, (const float *)j.b, (float *)j.dst, j.records, block);
        break;
    default:
        for (int w = threadIdx.x; w < j.clear.words; w += PREP_NT) ((uint32_t *)j.dst)[w] = 0u;
    }
}

static PrepJob *next_job(PrepList &l, int kind, int64_t blocks, const void *a, const void *b, void *dst)
{
    if (l.n >= PREP_MAX_JOBS || blocks <= 0 || blocks > 0x7fffffff) { l.bad = true; return nullptr; }
    PrepJob *j = reinterpret_cast<PrepJob *>(l.storage) + l.n++;
    *j = PrepJob{};
    j->kind = kind; j->blocks = (int)blocks; j->a = a; j->b = b; j->dst = dst;
    return j;
}

void PrepList::pack_theta(const float *theta, const float *bias, void *thetaF, int Din, int Dout, int RP, int CP,
                          int n_i, int n_j, int transpose)
{
    if (4 * RP > PACK_MAX_KD || CP % 16 != 0) { bad = true; return; }
    if (PrepJob *j = next_job(*this, PREP_PACK, (int64_t)n_i * n_j * (CP / 16), theta, bias, thetaF))
        j->pack = PackArgs{Din, Dout, RP, CP, n_i, transpose, (int)theta_f16_bytes(RP, CP),
                           (int)theta_f16_exp_offset(RP, CP), (int)theta_f16_rscale_offset(RP, CP)};
}

void PrepList::pack_theta_pos(const float *theta, void *thetaF, int Din, int Dout, int ci0, int co0, int KDP, int CP,
                              int transpose)
{
    if (PrepJob *j = next_job(*this, PREP_PACK_POS, 3 * (CP / 16), theta, nullptr, thetaF))
        j->pos = PackPosArgs{Din, Dout, ci0, co0, KDP, CP, transpose, (int)theta_pos_exp_offset(KDP, CP)};
}

void PrepList::order(const int32_t *in_off, int B, int N, int32_t *order)
{
    const int wpc = (N + ORDER_WINDOW - 1) / ORDER_WINDOW;
    const int64_t windows = (int64_t)B * wpc;
    if (PrepJob *j = next_job(*this, PREP_ORDER, (windows + ORDER_PER_BLOCK - 1) / ORDER_PER_BLOCK, in_off, nullptr, order)) {
        j->order.N = N; j->order.wpc = wpc; j->order.windows = (int)windows;
    }
}

void PrepList::copy(const float *src, float *dst, int B, int N, int Cs, int Cd, int src_bcn, int dst_bcn, int c_off)
{
    const int tn = (N + 63) / 64, tc = (Cd + 63) / 64;
    if (PrepJob *j = next_job(*this, PREP_COPY, (int64_t)B * tn * tc, src, nullptr, dst)) {
        const bool al = ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0;
        const bool vec = al && (src_bcn ? N % 4 == 0 : (Cs | c_off) % 4 == 0) && (dst_bcn ? N % 4 == 0 : Cd % 4 == 0);
        j->copy = CopyArgs{N, Cs, Cd, c_off, src_bcn, dst_bcn, tn, tc, vec};
    }
}

void PrepList::pack_pos(const float *pos, float *pos4, int B, int N)
{
    constexpr int PER_BLOCK = PREP_NT * POINTS_PER_THREAD;
    const int64_t total = (int64_t)B * N;
    if (PrepJob *j = next_job(*this, PREP_POINTS, (total + PER_BLOCK - 1) / PER_BLOCK, pos, nullptr, pos4)) {
        j->points.N = N; j->points.total = (int)total;
    }
}

void PrepList::records(const float *pos, const float *feat, float *rec, float *rec4, int B, int N, int W, int bcn, const int32_t *nbr, int K)
{
    constexpr int PER_BLOCK = PREP_NT / 4 * RECORDS_PER_THREAD;
    const int64_t total = (int64_t)B * N;
    if (PrepJob *j = next_job(*this, PREP_RECORDS, (total + PER_BLOCK - 1) / PER_BLOCK, pos, feat, rec))
        j->records = RecordArgs{N, (int)total, W, bcn, K, rec4, nbr};
}

void PrepList::clear(void *dst, int words)
{
    if (PrepJob *j = next_job(*this, PREP_CLEAR, 1, nullptr, nullptr, dst)) j->clear.words = words;
}

hipError_t PrepList::launch(hipStream_t s)
{
    if (bad) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    PrepJobs a{};
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        a.job[i] = reinterpret_cast<const PrepJob *>(storage)[i];
        blocks += a.job[i].blocks;
    }
    n = 0;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(prep_kernel, dim3((unsigned)blocks), dim3(PREP_NT), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_copy_rows(const float *src, float *dst, int B, int N, int Cs, int Cd, int src_bcn, int dst_bcn,
                            hipStream_t s, int c_off)
{
    PrepList l;
    l.copy(src, dst, B, N, Cs, Cd, src_bcn, dst_bcn, c_off);
    return l.launch(s);
}

}  // namespace flex
