// Flex-convolution on tiles of 64 points (gfx950, wave64): the forward pass (fixed-K neighbour tensor) and the feature
// gradient (in-edge lists) of layers of any width.
//
// A workgroup of sixteen waves, one per CU.  Eight GATHER waves sum the rows of a tile's neighbours in registers,
//     A[l][j*64 + c] = sum_k dp_j(l,k) row[n_k(l)][c]      (dp_3 = 1; a block of 64 input channels)
// and park the result in LDS as split-half rows (flex_prep.hip: f16 hi + lo of the scaled value); eight CONTRACT waves
// multiply the tile before with the packed parameters on the f16 matrix cores (hi*hi + hi*lo + lo*hi).  Two tile
// buffers, one barrier per tile.  A layer wider than 64 input channels walks its input blocks tile by tile with the
// sums kept in the contracting waves' registers, so a row is gathered once per OUTW output channels (up to 256) and
// nothing but the result leaves the chip.
//
// The kernels of flex_ws.hpp keep their parameters in registers whatever the width: a wide layer would walk the whole
// cloud with them once per 64 input channels, adding to the output in memory, on 32-point tiles; their gathering waves
// spend some 540 instructions on four points.  Here parameters of more than one input block stream from L2, 64 points to a pass, and
// what a lane needs to gather a row -- the position difference and the row's offset -- is prepared one entry per lane
// (eight slots of the wave's eight points: a step) and a step ahead, through LDS: 300 instructions per four points.
// Both matter because a wave issues at most one instruction per five clocks.
#pragma once
#include "flex_ws.hpp"

namespace flex {

template <int WM_, int NSW_>
struct TileGeom {
    static constexpr int IC = 64;                        // input channels per block
    static constexpr int WM = WM_, WN = 8 / WM_;         // contracting waves along the points / the output channels
    static constexpr int NSW = NSW_;                     // 16-channel slices per contracting wave
    static constexpr int NT = 1024, T = 64;
    static constexpr int LPR = IC / 4, G = 64 / LPR;     // lanes per row, points a wave gathers at a time
    static constexpr int PASSES = 8 / G;
    static constexpr int KD = 4 * IC, KS = KD / 32;      // depth, depth steps of the matrix op
    static constexpr int ARS = 4 * KD + 32;              // tile row: [hi: KD halves][lo: KD halves][32 B], = 32 mod 256 (WsGeom)
    static constexpr int MB = 4 / WM;                    // 16-point blocks per contracting wave
    static constexpr int OUTW = 16 * WN * NSW;
};

// Rows are read through a buffer descriptor of the cloud's tensor: a slot without an entry carries an offset past its
// end (the last row that 32-bit offsets reach, which the host keeps free), for which the load returns zeros without touching memory.  So every slot's load is issued unconditionally, which
// is what keeps eight of them in flight: the compiler waits for a load by counting the younger ones, and where those
// may or may not have been issued it has to wait for all of them (branches around them: 13 000 clocks a tile).
typedef unsigned v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const float *rows, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(rows), 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ v4f load_row4(__amdgpu_buffer_rsrc_t rows, unsigned offset)
{
    return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)offset, 0, 0));
}

typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));

// maximum over the wave, in every lane
__device__ __forceinline__ int wave_max(int v)
{
    v = max(v, dpp_movi<0xB1>(v));
    v = max(v, dpp_movi<0x4E>(v));
    v = max(v, dpp_movi<0x141>(v));
    v = max(v, dpp_movi<0x140>(v));
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// One step of a gathering wave: eight list slots of its eight points of a tile, for one input block (all wave-uniform).
struct TileStep {
    int b, ib;
    int n0, n1;          // slots that some point of the first / second four has
    bool last;           // last step of (tile, input block)
};

// Walks a gathering wave's steps.  lane = 8 * slot + point.
template <bool CSR>
struct StepWalk {
    TileWalk tw;
    int ib, c;                       // input block, step inside the lists
    int nc;                          // steps per input block
    // CSR: this lane's point and list in the current tile and in the next, its point in the one after
    int pid, lo, deg, pid1, lo1, hi1, pid2;
    TileWalk tw1, tw2;

    __device__ __forceinline__ int position(const TileWalk &w, int first) const { return w.tic * 64 + first + (threadIdx.x & 7); }
    __device__ __forceinline__ int point_at(const TileArgs &a, const TileWalk &w, int first) const
    {
        return a.order[(int64_t)w.b * a.N + min(position(w, first), a.N - 1)];
    }
    __device__ __forceinline__ void bounds(const TileArgs &a)
    {
        const int64_t gp = (int64_t)tw1.b * a.N + pid1;
        lo1 = a.off[gp];
        hi1 = a.off[gp + 1];
    }
    __device__ __forceinline__ void enter(const TileArgs &a, int first)
    {
        // the walk `tw1` stands on the tile that becomes current
        tw = tw1;
        pid = pid1; lo = lo1;
        deg = position(tw, first) < a.N ? hi1 - lo1 : 0;         // positions past the cloud have no list
        nc = max(1, (wave_max(deg) + 7) >> 3);
        tw1.next_clamped();
        pid1 = pid2;
        tw2.next_clamped();
        pid2 = point_at(a, tw2, first);
        bounds(a);
    }
    // first: the wave's first point inside a tile
    __device__ __forceinline__ StepWalk(const TileArgs &a, const TileSchedule &sc, int first)
        : tw(sc, a.tpc), tw1(sc, a.tpc), tw2(sc, a.tpc)
    {
        ib = c = 0;
        if constexpr (CSR) {
            pid1 = point_at(a, tw1, first);
            tw2.next_clamped();
            pid2 = point_at(a, tw2, first);
            bounds(a);
            enter(a, first);
        } else {
            nc = (a.K + 7) >> 3;
        }
    }
    // The step's descriptor and this lane's entry of it: the id and the point it belongs to, has: whether it exists.  Then
    // moves on; past the workgroup's last tile it repeats that tile.
    __device__ __forceinline__ TileStep fetch(const TileArgs &a, int first, int &id, int &point, bool &has)
    {
        TileStep d;
        d.b = tw.b; d.ib = ib;
        d.last = c == nc - 1;
        const int slot = 8 * c + ((threadIdx.x >> 3) & 7);
        if constexpr (CSR) {
            point = pid;
            has = slot < deg;
            id = a.src[has ? lo + slot : 0];                     // a list entry is always there (K >= 1)
            id = has ? id : pid;
            auto most = [&](int l) {
                return max(max(__builtin_amdgcn_readlane(deg, l), __builtin_amdgcn_readlane(deg, l + 1)),
                           max(__builtin_amdgcn_readlane(deg, l + 2), __builtin_amdgcn_readlane(deg, l + 3))) - 8 * c;
            };
            d.n0 = most(0); d.n1 = most(4);
        } else {
            d.n0 = d.n1 = a.K - 8 * c;
            const int at = position(tw, first);
            point = min(at, a.N - 1);
            has = slot < a.K && at < a.N;                        // positions past the cloud have no slots
            id = a.nbr[((int64_t)d.b * a.K + min(slot, a.K - 1)) * a.N + point];
        }
        if (++c == nc) {
            c = 0;
            if (++ib == a.n_in) {
                ib = 0;
                if constexpr (CSR) enter(a, first);
                else tw.next_clamped();
            }
        }
        return d;
    }
};

// Lane's channels of a row in input block ib: past the row's end the last four again, put right after the sums.
__device__ __forceinline__ int tile_lane_channel(const TileArgs &a, int ib) { return min(ib * 64 + 4 * ((int)threadIdx.x & 15), a.w_in - 4); }

// Four channels (X: numbers, or sums of several components) that were read `shift` places early, back in their own places: what lies
// past the row's end becomes zero.
template <class X>
__device__ __forceinline__ void put_channels_right(X &&c, int shift)
{
    typedef std::remove_reference_t<decltype(c[0])> E;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        E x = E{};
#pragma unroll
        for (int w = v; w < 4; ++w)
            if (w - v == shift) x = c[w];
        c[v] = x;
    }
}

// What a gathering wave does: the sums of its eight points (from `first` of every tile) over input blocks ib0 .. ib0 + n_in - 1,
// acc[pass][channel][component]; park(acc, ib, point) takes them when a (tile, input block) is complete, HALVES: park(acc[pass], pass)
// those of the first four points and of the second four as each is.
// Eight rows are in flight at all times.
//
// How a slot's row is weighed with its (dx, dy, dz, 1).  MX: by outer products on the matrix cores (outer_slot): an entry is
// then needed once per wave, in the layout lane = 16 * point + 4 * slot + component, and its row's offset, the fourth
// component, reaches the address by a DPP add.  Else by fused multiply-adds, every lane reading its point's entry from LDS,
// 16 bytes a slot.  The 4 x 4 x 1 op holds the matrix cores for 8 clocks and the vector ALU with them, the sixteen
// multiply-adds that four of them replace hold the vector ALU for 40, the reads LDS for as long.  512 -> 512, 109k points, us: forward 796
// by multiply-adds, 778 by outer products, feature gradient 852 and 836; the parameter gradient, whose contraction
// already fills the matrix cores twice as far, 1681 and 1728.
template <bool CSR, bool MX, bool HALVES, class Park>
__device__ __forceinline__ void gather_steps(const TileArgs &a, const TileSchedule &sc, int tiles, int first, int ib0,
                                             float (*ent)[64][4], Park &&park)
{
    const int lane = threadIdx.x & 63, grp = lane / 16;
    StepWalk<CSR> walk(a, sc, first);
    struct Positions { float n[3], c[3]; };
    auto request = [&](const TileStep &d, int id, int point, Positions &p) {
        const char *pb = reinterpret_cast<const char *>(a.pos + (int64_t)d.b * 3 * a.N);
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            p.n[x] = *reinterpret_cast<const float *>(pb + 4u * ((unsigned)(x * a.N) + (unsigned)id));
            p.c[x] = *reinterpret_cast<const float *>(pb + 4u * ((unsigned)(x * a.N) + (unsigned)point));
        }
    };
    auto publish = [&](int buf, int id, bool has, const Positions &p) {
        const float sg = CSR ? -1.f : 1.f;          // CSR: point - listing centre
        // a slot without an entry weighs its zeros with zero, wherever the point lies (it may lie at infinity or nowhere)
        *reinterpret_cast<v4f *>(ent[buf][lane]) =
            v4f{has ? sg * (p.n[0] - p.c[0]) : 0.f, has ? sg * (p.n[1] - p.c[1]) : 0.f, has ? sg * (p.n[2] - p.c[2]) : 0.f,
                __uint_as_float(has ? (unsigned)id * (4u * (unsigned)a.rs) : 0u - 4u * (unsigned)a.rs)};
        wave_lds_sync();
    };
    auto lane_channel = [&](int ib) { return tile_lane_channel(a, ib0 + ib); };
    auto rows_of = [&](const TileStep &d) {
        return row_buffer(a.rows + (int64_t)d.b * a.N * a.rs, (unsigned)a.N * (unsigned)a.rs * 4u);
    };

    // MX: the entries of four slots of a pass's four points, slots 4 * half ..
    const float *my_ent = &ent[0][8 * ((lane >> 2) & 3) + grp][lane & 3];
    struct Entries { float v[2][2]; };              // [pass][half]
    auto entries = [&](int buf) {
        Entries e;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h) e.v[p][h] = my_ent[buf * 256 + 128 * h + 16 * p];
        return e;
    };
    const bool is_weight = (lane & 3) == 3;
    auto row_offset = [&](float e, int slot) { return (unsigned)row_bcast_offset(__float_as_int(e), slot); };

    TileStep d0, d1, d2;
    int id1, id2, pt1, pt2, pt0;                    // this lane's entries of the next two steps
    bool has1, has2;
    Positions p1;
    Entries e0;
    v4f f[8];                                       // rows in flight
    // how far ahead of its use LDS is read, as the registers allow: the differences EA slots, the offsets of four
    // points from slot to slot over the four points before (fixed lists) or at once in front of them
    constexpr int EA = CSR ? 2 : 4;
    constexpr bool OFF_AHEAD = !CSR;
    unsigned off[MX ? 1 : 8];
    {
        int id0;
        bool has0;
        Positions p0;
        d0 = walk.fetch(a, first, id0, pt0, has0);
        d1 = walk.fetch(a, first, id1, pt1, has1);
        request(d0, id0, pt0, p0);
        d2 = walk.fetch(a, first, id2, pt2, has2);
        publish(0, id0, has0, p0);
        request(d1, id1, pt1, p1);
        if constexpr (MX) e0 = entries(0);
        const auto rows = rows_of(d0);
        const unsigned lane_off = 4u * (unsigned)lane_channel(d0.ib);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if constexpr (MX) f[u] = load_row4(rows, row_offset(e0.v[0][u >> 2], u & 3) + lane_off);
            else f[u] = load_row4(rows, __float_as_uint(ent[0][8 * u + grp][3]) + lane_off);
        }
        if constexpr (OFF_AHEAD && !MX) {
#pragma unroll
            for (int u = 0; u < 8; ++u) off[u] = __float_as_uint(ent[0][8 * u + 4 + grp][3]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    v4f acc[2][4];                                  // [pass][channel][component]
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[p][v] = v4f{0.f, 0.f, 0.f, 0.f};
    };
    clear();

    for (int s = 0, k = 0; k < tiles; ++s) {
        const int buf = s & 1;
        publish(buf ^ 1, id1, has1, p1);            // the next step's entries
        Entries e1;
        if constexpr (MX) e1 = entries(buf ^ 1);
        request(d2, id2, pt2, p1);                  // positions of the step after it, entries of the one after that
        int id3, pt3;
        bool has3;
        const TileStep d3 = walk.fetch(a, first, id3, pt3, has3);

        // Eight rows are in flight at all times: the registers of a slot that has been summed take the same slot of
        // the next four points at once, of the next step's after the second four.
        const auto rows0 = rows_of(d0), rows1 = rows_of(d1);
        const unsigned lane_off0 = 4u * (unsigned)lane_channel(d0.ib), lane_off1 = 4u * (unsigned)lane_channel(d1.ib);
        v4f e[EA + 1];
        if constexpr (!MX) {
#pragma unroll
            for (int u = 0; u < EA; ++u) e[u] = *reinterpret_cast<const v4f *>(ent[buf][8 * u + grp]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            float w[2];                             // MX: the slots' weights
            if constexpr (MX) {
                w[0] = is_weight ? 1.f : e0.v[p][0];
                w[1] = is_weight ? 1.f : e0.v[p][1];
            } else if constexpr (!OFF_AHEAD) {
#pragma unroll
                for (int u = 0; u < 8; ++u) off[u] = __float_as_uint(p == 0 ? ent[buf][8 * u + 4 + grp][3] : ent[buf ^ 1][8 * u + grp][3]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                constexpr int R = EA + 1;
                const int i = 8 * p + u;
                if constexpr (!MX)
                    if (i + EA < 16) e[(i + EA) % R] = *reinterpret_cast<const v4f *>(ent[buf][8 * ((i + EA) & 7) + 4 * ((i + EA) >> 3) + grp]);
                if (u < (p == 0 ? d0.n0 : d0.n1)) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if constexpr (MX) {
                            acc[p][v] = outer_slot(w[u >> 2], f[u][v], acc[p][v], u & 3);
                            continue;
                        }
                        const v4f d = e[i % R];
                        acc[p][v][0] = fmaf(d[0], f[u][v], acc[p][v][0]);
                        acc[p][v][1] = fmaf(d[1], f[u][v], acc[p][v][1]);
                        acc[p][v][2] = fmaf(d[2], f[u][v], acc[p][v][2]);
                        acc[p][v][3] += f[u][v];
                    }
                }
                if constexpr (MX) {
                    f[u] = p == 0 ? load_row4(rows0, row_offset(e0.v[1][u >> 2], u & 3) + lane_off0)
                                  : load_row4(rows1, row_offset(e1.v[0][u >> 2], u & 3) + lane_off1);
                } else {
                    f[u] = p == 0 ? load_row4(rows0, off[u] + lane_off0) : load_row4(rows1, off[u] + lane_off1);
                }
                if constexpr (OFF_AHEAD && !MX) off[u] = __float_as_uint(ent[buf ^ 1][8 * u + 4 * p + grp][3]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (HALVES) {
                if (d0.last) {
                    park(acc[p], p);
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[p][v] = v4f{0.f, 0.f, 0.f, 0.f};
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (d0.last) {
            if constexpr (!HALVES) {
                park(acc, d0.ib, pt0);
                clear();
            }
            ++k;
        }
        if constexpr (MX) e0 = e1;
        d0 = d1; d1 = d2; d2 = d3;
        pt0 = pt1; pt1 = pt2; pt2 = pt3;
        id1 = id2; id2 = id3;
        has1 = has2; has2 = has3;
    }
}

template <int WM, int NSW, bool CSR, bool MULTI>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
void tile_conv_kernel(const TileArgs a)
{
    using P = TileGeom<WM, NSW>;
    constexpr int IC = P::IC;
    __shared__ __attribute__((aligned(16))) char s_A[2][P::T * P::ARS];
    __shared__ __attribute__((aligned(16))) float s_ent[8][2][64][4];     // per gathering wave: (dx, dy, dz, row byte offset) of entry 8 * slot + point
    __shared__ int s_P[2][P::T];                                          // CSR: the point in every tile row
    __shared__ int s_E[2][P::T];                                          // exponents of the tile rows
    constexpr int RS_BLOCKS = MULTI ? 8 : 1;
    __shared__ __attribute__((aligned(16))) float s_rs[RS_BLOCKS][4 * IC];   // depth scales of the first input blocks' parameters

    const int j = blockIdx.x / a.chunks;
    const TileSchedule sc(a.total, (int)blockIdx.x - j * a.chunks, a.chunks);
    if (!(sc.first < sc.end)) return;
    const int tiles = (sc.end - sc.first + sc.step - 1) / sc.step * a.n_in;   // (tile, input block) pairs of this workgroup
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const char *theta_j = a.theta + (int64_t)j * a.n_in * a.blk_bytes;

    for (int i = threadIdx.x; i < min(a.n_in, RS_BLOCKS) * 4 * IC; i += P::NT)
        s_rs[i / (4 * IC)][i % (4 * IC)] =
            reinterpret_cast<const float *>(theta_j + (int64_t)(i / (4 * IC)) * a.blk_bytes + a.rs_off)[i % (4 * IC)];
    __syncthreads();

    if (wave < 8) {
        // ---- gather ----
        static_assert(P::PASSES == 2 && P::G == 4, "two passes of four points");
        const int t = lane % P::LPR, grp = lane / P::LPR, first = 8 * wave;
        const bool ragged = a.w_in % IC != 0;
        int m_buf = 0;                                  // tile buffer of the tile being gathered
        gather_steps<CSR, true, false>(a, sc, tiles, first, 0, s_ent[wave], [&](v4f (&acc)[2][4], int step_ib, int point) __attribute__((always_inline)) {
            // ---- park ----
            const int ib = MULTI ? step_ib : 0;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int shift = ib * IC + 4 * t - tile_lane_channel(a, ib);
                if (ragged && shift > 0) put_channels_right(acc[p], shift);
                float m = 0.f;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const float *rs = ib < RS_BLOCKS ? &s_rs[ib][jj * IC + 4 * t]
                        : reinterpret_cast<const float *>(theta_j + (int64_t)ib * a.blk_bytes + a.rs_off) + jj * IC + 4 * t;
                    const v4f r = *reinterpret_cast<const v4f *>(rs);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        acc[p][v][jj] *= r[v];
                        m = __builtin_amdgcn_fmed3f(m, __builtin_fabsf(acc[p][v][jj]), __builtin_inff());
                    }
                }
                m = group_max<P::LPR>(m);
                const int ex = 15 - __builtin_amdgcn_frexp_expf(m);
                const int pt = first + 4 * p + grp;
                char *row = s_A[m_buf] + pt * P::ARS + 8 * t;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    typedef float f2 __attribute__((ext_vector_type(2)));
                    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
                    h2 h[2], l[2];
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        const f2 x = {__builtin_ldexpf(acc[p][2 * w][jj], ex), __builtin_ldexpf(acc[p][2 * w + 1][jj], ex)};
                        h[w] = __builtin_convertvector(x, h2);
                        const f2 back = __builtin_convertvector(h[w], f2);
                        l[w] = __builtin_convertvector(x - back, h2);
                    }
                    *reinterpret_cast<h4 *>(row + 2 * jj * IC) = h4{h[0][0], h[0][1], h[1][0], h[1][1]};
                    *reinterpret_cast<h4 *>(row + 2 * (P::KD + jj * IC)) = h4{l[0][0], l[0][1], l[1][0], l[1][1]};
                }
                if (t == 0) s_E[m_buf][pt] = ex;
                __builtin_amdgcn_sched_barrier(0);
            }
            if (CSR && lane < 8) s_P[m_buf][first + lane] = point;
            m_buf ^= 1;
            __syncthreads();               // the tile is complete
        });
        return;
    }

    // ---- contract ----
    // An input block's product stands by itself: its own exponents per point and column, and two chains per accumulator
    // block, hi*hi and the cross terms.  What is added up over the input blocks is the unscaled fp32 result, on the vector
    // ALU, which rounds to nearest.  (The matrix op rounds every partial sum down: one chain over all products and blocks
    // was 1.2e-7 off at one input block, 2.2e-7 at two, 3.3e-7 at four and 4.8e-7 at eight, where this is 1.1e-7 to
    // 1.3e-7, in the same time but for 512 -> 512, 4 percent; and one scale for all blocks costs a block its bits next to
    // a larger one.)
    constexpr bool RESIDENT = !MULTI && WM == 2;        // parameters of one block, 64 registers: kept
    const int cw = wave - 8, q = lane >> 4, r16 = lane & 15;
    const int wm = cw % WM, wn = cw / WM;
    constexpr int PART = (P::OUTW / 16) * P::KS * 64 * 16;
    constexpr int STEPS = NSW * P::KS;                  // (slice, depth step) pairs of a tile and input block
    constexpr int AHEAD = RESIDENT ? STEPS : MULTI && NSW == 2 ? 2 : 4;     // pairs whose parameters are held, as the registers allow
    h8 tH[AHEAD], tL[AHEAD];
    v4f sum[P::MB][NSW];                                // MULTI: the result over the input blocks so far
#pragma unroll
    for (int m = 0; m < P::MB; ++m)
#pragma unroll
        for (int n = 0; n < NSW; ++n) sum[m][n] = v4f{0.f, 0.f, 0.f, 0.f};
    const char *blk = theta_j;
    unsigned th_off = (unsigned)((wn * NSW) * P::KS * 64 + lane) * 16u;
    auto load_theta = [&](int i) __attribute__((always_inline)) {       // slice i / KS, depth step i % KS
        tH[i % AHEAD] = *reinterpret_cast<const h8 *>(blk + i * 1024 + th_off);
        tL[i % AHEAD] = *reinterpret_cast<const h8 *>(blk + PART + i * 1024 + th_off);
    };
    if constexpr (RESIDENT) {
#pragma unroll
        for (int i = 0; i < STEPS; ++i) load_theta(i);
    }
    TileWalk tw(sc, a.tpc);
    int ib = 0;
    for (int k = 0; k < tiles; ++k) {
        __syncthreads();                   // the tile is complete
        const int m_buf = k & 1, b = tw.b, l0 = tw.tic * 64;
        // (the lane's offsets are formed anew for every tile: the compiler would otherwise read the parameters once
        // and for all before the loop, and spill them)
        unsigned a_off = (unsigned)((wm * P::MB * 16 + r16) * P::ARS + 16 * q);
        int o_lane = wn * NSW * 16 + 4 * q, l_lane = wm * P::MB * 16 + r16;
        asm volatile("" : "+v"(th_off), "+v"(a_off), "+v"(o_lane), "+v"(l_lane));
        if constexpr (!RESIDENT) {
            blk = theta_j + (int64_t)(MULTI ? ib : 0) * a.blk_bytes;
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) load_theta(i);
        }
        const int *ecol = reinterpret_cast<const int *>(blk + a.exp_off) + o_lane;
        const char *arow = s_A[m_buf] + a_off;
        auto store = [&](int m, int n, const v4f &d) __attribute__((always_inline)) {
            const int o = j * P::OUTW + 16 * n + o_lane, pt = m * 16 + l_lane;
            if (l0 + pt >= a.N) return;
            const int l = CSR ? s_P[m_buf][pt] : l0 + pt;
            float *dst = a.out + b * a.out_b + l * a.out_l + o * a.out_c;
            if (a.out_c == 1 && o + 3 < a.w_out) *reinterpret_cast<v4fu *>(dst) = d;
            else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (o + i < a.w_out) dst[i * a.out_c] = d[i];
            }
        };
        // One 16-channel slice after the other, two point blocks at a time, a depth step after the other; the fragments of
        // the next two point blocks are read while the matrix ops of the current ones run.
        constexpr int MH = (MULTI && NSW == 2) ? 1 : 2, HALVES = P::MB / MH, ITEMS = P::KS * HALVES;
        h8 bh[2][MH], bl[2][MH];
        auto load_b = [&](int item) __attribute__((always_inline)) {
            const int st = item / HALVES % P::KS, m0 = item % HALVES * MH;
#pragma unroll
            for (int m = 0; m < MH; ++m) {
                bh[item & 1][m] = *reinterpret_cast<const h8 *>(arow + (m0 + m) * 16 * P::ARS + 64 * st);
                bl[item & 1][m] = *reinterpret_cast<const h8 *>(arow + (m0 + m) * 16 * P::ARS + 64 * st + 2 * P::KD);
            }
        };
        load_b(0);
#pragma unroll
        for (int n = 0; n < NSW; ++n) {
            v4f main[P::MB], cross[P::MB];
#pragma unroll
            for (int m = 0; m < P::MB; ++m) main[m] = cross[m] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const int item = n * ITEMS + i, at = n * P::KS + i / HALVES, m0 = i % HALVES * MH;
                if (item + 1 < NSW * ITEMS) load_b(item + 1);
                __builtin_amdgcn_sched_barrier(0);
                const h8 H = tH[at % AHEAD], L = tL[at % AHEAD];
#pragma unroll
                for (int m = 0; m < MH; ++m) main[m0 + m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(H, bh[item & 1][m], main[m0 + m], 0, 0, 0);
#pragma unroll
                for (int m = 0; m < MH; ++m) cross[m0 + m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(L, bh[item & 1][m], cross[m0 + m], 0, 0, 0);
#pragma unroll
                for (int m = 0; m < MH; ++m) cross[m0 + m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(H, bl[item & 1][m], cross[m0 + m], 0, 0, 0);
                if constexpr (!RESIDENT)
                    if (m0 + MH == P::MB && at + AHEAD < STEPS) load_theta(at + AHEAD);     // into the registers just read
                __builtin_amdgcn_sched_barrier(0);
            }
            const v4i ec = *reinterpret_cast<const v4i *>(ecol + 16 * n);
#pragma unroll
            for (int m = 0; m < P::MB; ++m) {
                const int e = s_E[m_buf][m * 16 + l_lane];
                v4f d = main[m] + cross[m];
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] = __builtin_ldexpf(d[i], -(e + ec[i]));
                if constexpr (MULTI) sum[m][n] += d;
                else store(m, n, d);
            }
        }
        if constexpr (MULTI) {
            if (++ib < a.n_in) continue;
            ib = 0;
#pragma unroll
            for (int n = 0; n < NSW; ++n)
#pragma unroll
                for (int m = 0; m < P::MB; ++m) {
                    store(m, n, sum[m][n]);
                    sum[m][n] = v4f{0.f, 0.f, 0.f, 0.f};
                }
        }
        tw.next();
    }
}

#if defined(FLEX_TILE_CSR) && FLEX_TILE_CSR == 0     // one object holds it
// ---------------------------------------------------------------------------
// Parameter gradients of wide layers on 64-point tiles: partial[kd][o] = sum over the workgroup's points of A[pt][kd] g[pt][o]
// for one block of 64 feature channels (kd = j*64 + c) and 64 output channels.
//
// Workgroup x serves block p = x / chunks = (hi, ho) = (p / n_ho, p % n_ho) as share x % chunks: a deep, low-resolution
// layer has many blocks and few points, so a workgroup walks all points for one block instead of all of them walking a few
// tiles each for every block.
//
// The sums over points: every value as three bf16 pieces (split_bf3), six products on the bf16 matrix cores, operands read
// transposed out of point-major LDS tiles.  The matrix op rounds every partial sum down, a bias of one sign whatever the
// sum's own, so the upstream gradient of the second 32 points of a tile goes in negated and their sums come off the total:
// the biases cancel.  Totals are fp32 in registers, added (to nearest) once per 32 points and moved to the partial every
// FLUSH tiles, because what such a chain of sums loses grows with its length.  2-norm error against 64 bits, chains of
// eight steps flushed into register totals -> this: 128 -> 128 at 2k, 30k and 1M points 1.8e-7, 2.7e-7, 8.4e-7 ->
// 1.0e-7, 1.2e-7, 2.3e-7; 512 -> 512 at 109k 4.0e-7 -> 2.3e-7.  (The moves are 2 percent of the time at 512 -> 512.)
// The gathering waves are those of the convolution above, and the contracting waves fetch the
// upstream gradient.  One tile buffer (100 KB of LDS): the gathering waves sum the next tile in registers while this one is
// contracted, and park it between two barriers.
// What bounds it is the vector ALU (at 4 clocks an instruction 81 percent of its time at 128 -> 128 and 1M points, 83 at 512 -> 512
// and 109k; the matrix cores 41 and 42, no bank conflicts).  Clouds of more than a few tiles a workgroup run tile_grad_theta128_kernel
// below; the rule and both sides' times are beside tile_grad_plan (flex_api.hip).
//
// F32: products and sums on the fp32 matrix op, which rounds to nearest and takes infinities as they are.  In the pieces above an
// infinity becomes no number, terms of up to 2^-21 of a product (2^-24.7 on average) are dropped, and sums of few points carry the matrix
// op's one-sided rounding: 64 -> 128, one point 7.4e-8 where products rounded once leave 2.5e-8, eight points of 4096 with a gradient 9.1e-8
// and 6.8e-8.  A tile's points are summed eight at a time and those sums in pairs: 2-norm error 64 -> 128 at 64, 4k, 30k and 200k points
// 0.9e-7, 0.9e-7, 1.0e-7, 1.3e-7 (chains over a workgroup's points: 1.2e-7, 1.2e-7, 2.0e-7, 5.0e-7).  The fp32 op holds the vector ALU
// with the matrix cores (8192 clocks a tile), so that gathering and contracting add up: 300k points 236 us, 128 -> 64 233.
// SOME: contracting waves whose channels all lie past the rows' ends have no sums (the reduction drops their part of the partial) and
// leave the vector ALU to the others; the launch says from where on.
// ---------------------------------------------------------------------------
template <bool F32, bool SOME>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
void tile_grad_theta_kernel(const TileArgs a, const float *__restrict__ g_rows, int n_ho, float *__restrict__ partials)
{
    constexpr int IC = 64, KD = 4 * IC, OC = 64, T = 64;
    // bytes of a row: 16 mod 64 words, so that the four rows of a read lie in banks of their own
    constexpr int AS = F32 ? 4 * KD + 64 : bf3_stride(KD), GS = F32 ? 4 * OC + 64 : bf3_stride(OC);
    __shared__ __attribute__((aligned(16))) char s_A[T * AS];
    __shared__ __attribute__((aligned(16))) char s_G[T * GS];
    __shared__ __attribute__((aligned(16))) float s_ent[8][2][64][4];

    const int p = blockIdx.x / a.chunks, hi = p / n_ho, ho = p - hi * n_ho;
    const TileSchedule sc(a.total, (int)blockIdx.x - p * a.chunks, a.chunks);
    const int tiles = sc.first < sc.end ? (sc.end - sc.first + sc.step - 1) / sc.step : 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    if (wave < 8) {
        // ---- gather ----
        if (tiles == 0) return;
        const int t = lane & 15, grp = lane >> 4, first = 8 * wave;
        gather_steps<false, false, false>(a, sc, tiles, first, hi, s_ent[wave], [&](v4f (&acc)[2][4], int, int) __attribute__((always_inline)) {
            const int shift = 64 * hi + 4 * t - tile_lane_channel(a, hi);        // channels past the row's end: not in the result
            __syncthreads();               // the tile before is contracted
#pragma unroll
            for (int ps = 0; ps < 2; ++ps) {
                if (a.w_in % 4 != 0) put_channels_right(acc[ps], shift);
                char *row = s_A + (first + 4 * ps + grp) * AS;
                const int swap = bf3_swap(first);            // of all eight points of the wave
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    if constexpr (F32) {
                        *reinterpret_cast<v4f *>(row + 4 * (jj * IC + 4 * t)) = v4f{acc[ps][0][jj], acc[ps][1][jj], acc[ps][2][jj], acc[ps][3][jj]};
                        continue;
                    }
                    unsigned h0, m0, l0, h1, m1, l1;
                    split_bf3(acc[ps][0][jj], acc[ps][1][jj], h0, m0, l0);
                    split_bf3(acc[ps][2][jj], acc[ps][3][jj], h1, m1, l1);
                    char *d = row + bf3_at(8 * t, 2 * jj * IC, swap);
                    *reinterpret_cast<uint2 *>(d) = make_uint2(h0, h1);
                    *reinterpret_cast<uint2 *>(d + 2 * KD) = make_uint2(m0, m1);
                    *reinterpret_cast<uint2 *>(d + 4 * KD) = make_uint2(l0, l1);
                }
            }
            __syncthreads();               // the tile is complete
        });
        return;
    }

    // ---- contract: four 16-row blocks x two 16-column blocks of the partial per wave ----
    constexpr int MBW = 4, NBW = 2, FLUSH = 64;
    const int cw = wave - 8, q = lane >> 4, r16 = lane & 15, wn = cw & 1, wm = cw >> 1, ctid = threadIdx.x - 512;
    v4f tot[MBW][NBW];                     // the sums since the last move to the partial
#pragma unroll
    for (int c = 0; c < MBW; ++c)
#pragma unroll
        for (int n = 0; n < NBW; ++n) tot[c][n] = v4f{0.f, 0.f, 0.f, 0.f};

    float *dst = partials + (int64_t)blockIdx.x * KD * OC;
    auto flush = [&](bool add) __attribute__((always_inline)) {
        unsigned at = (unsigned)((wm * 16 + 4 * q) * OC + wn * 16 + r16);
        asm volatile("" : "+v"(at));       // addresses are formed here, not kept through the loop
        auto place = [&](int c, int n, int i) { return dst + (at + (4 * c * 16 + i) * OC + 2 * n * 16); };
#pragma unroll
        for (int c = 0; c < MBW; ++c) {
            v4f old[NBW];
#pragma unroll
            for (int n = 0; n < NBW; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) old[n][i] = add ? *place(c, n, i) : 0.f;
#pragma unroll
            for (int n = 0; n < NBW; ++n) {
#pragma unroll
                for (int i = 0; i < 4; ++i) *place(c, n, i) = old[n][i] + tot[c][n][i];
                tot[c][n] = v4f{0.f, 0.f, 0.f, 0.f};
            }
        }
    };

    const bool idle = SOME && __builtin_amdgcn_readfirstlane(IC * hi + 16 * wm >= a.w_in || OC * ho + 16 * wn >= a.w_out);

    TileWalk tw(sc, a.tpc);
    v4f gv[2];                             // upstream gradient of a tile: two four-float chunks per thread
    const int g_col = OC * ho + 4 * (ctid & 15), g_at = min(g_col, a.w_out - 4);      // past the row's end the last four again
    auto load_g = [&]() {
        const auto g = row_buffer(g_rows + (int64_t)tw.b * a.N * a.w_out, 4u * (unsigned)a.N * (unsigned)a.w_out);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            // the row behind the cloud's last reads as zeros: points past the cloud contribute nothing
            const int l = min(tw.tic * T + (ctid >> 4) + 32 * c, a.N);
            gv[c] = load_row4(g, 4u * ((unsigned)l * (unsigned)a.w_out + (unsigned)g_at));
        }
    };
    if (tiles > 0) load_g();
    for (int k = 0; k < tiles; ++k) {
        __syncthreads();                   // the tile before is contracted
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            char *row = s_G + ((ctid >> 4) + 32 * c) * GS;
            const int swap = bf3_swap(ctid >> 4), v = 8 * (ctid & 15);
            unsigned h0, m0, l0, h1, m1, l1;
            if (a.w_out % 4 != 0) put_channels_right(gv[c], g_col - g_at);
            if constexpr (F32) {
                *reinterpret_cast<v4f *>(row + 16 * (ctid & 15)) = gv[c];
                continue;
            }
            const v4f g = c == 0 ? gv[c] : -gv[c];                 // (the second 32 points: see above)
            split_bf3(g[0], g[1], h0, m0, l0);
            split_bf3(g[2], g[3], h1, m1, l1);
            *reinterpret_cast<uint2 *>(row + bf3_at(v, 0, swap)) = make_uint2(h0, h1);
            *reinterpret_cast<uint2 *>(row + bf3_at(v, 2 * OC, swap)) = make_uint2(m0, m1);
            *reinterpret_cast<uint2 *>(row + bf3_at(v, 4 * OC, swap)) = make_uint2(l0, l1);
        }
        tw.next_clamped();
        load_g();
        if (k % FLUSH == 0 && k > 0) flush(k > FLUSH);
        __syncthreads();                   // the tile is complete
        if constexpr (F32) {
            if (idle) continue;
            // Sixteen points of a row block at a time, as two chains of eight; what they leave is added, in pairs over the tile, while
            // the next ones run.
            constexpr int SETS = T / 16;
            const float *sA = reinterpret_cast<const float *>(s_A) + q * (AS / 4) + 16 * wm + r16;
            const float *sG = reinterpret_cast<const float *>(s_G) + q * (GS / 4) + 16 * wn + r16;
            float fa[2][4], fg[2][4][NBW];
            v4f x[2][2][NBW], y[NBW], z[NBW];
            auto fetch = [&](int j) __attribute__((always_inline)) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int row = 16 * (j % SETS) + 4 * s;
                    fa[j & 1][s] = sA[row * (AS / 4) + 64 * (j / SETS)];
#pragma unroll
                    for (int n = 0; n < NBW; ++n) fg[j & 1][s][n] = sG[row * (GS / 4) + 32 * n];
                }
            };
            fetch(0);
#pragma unroll
            for (int j = 0; j <= SETS * MBW; ++j) {
                if (j < SETS * MBW) {
                    if (j + 1 < SETS * MBW) fetch(j + 1);
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int n = 0; n < NBW; ++n)
                            x[j & 1][s & 1][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                fa[j & 1][(s & 1) * 2 + s / 2], fg[j & 1][(s & 1) * 2 + s / 2][n], s < 2 ? v4f{0.f, 0.f, 0.f, 0.f} : x[j & 1][s & 1][n], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (j == 0) continue;
                const int i = (j - 1) % SETS, c = (j - 1) / SETS;
#pragma unroll
                for (int n = 0; n < NBW; ++n) {
                    v4f sum = x[(j - 1) & 1][0][n] + x[(j - 1) & 1][1][n];
                    if (i % 2 == 1) sum = y[n] + sum;
                    if (i % 2 == 0) y[n] = sum;
                    else if (i == 1) z[n] = sum;
                    else tot[c][n] += z[n] + sum;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            continue;
        }
#pragma unroll
        for (int st = 0; st < T / 32; ++st) {
            bf8 gH[NBW], gM[NBW], gL[NBW];
#pragma unroll
            for (int n = 0; n < NBW; ++n) {
                gH[n] = read_bf3_frag(s_G, GS, 32 * st + 8 * q, 32 * wn, 64 * n, r16);
                gM[n] = read_bf3_frag(s_G, GS, 32 * st + 8 * q, 32 * wn, 64 * n + 2 * OC, r16);
                gL[n] = read_bf3_frag(s_G, GS, 32 * st + 8 * q, 32 * wn, 64 * n + 4 * OC, r16);
            }
#pragma unroll
            for (int c = 0; c < MBW; ++c) {
                const bf8 aH = read_bf3_frag(s_A, AS, 32 * st + 8 * q, 32 * wm, 128 * c, r16);
                const bf8 aM = read_bf3_frag(s_A, AS, 32 * st + 8 * q, 32 * wm, 128 * c + 2 * KD, r16);
                const bf8 aL = read_bf3_frag(s_A, AS, 32 * st + 8 * q, 32 * wm, 128 * c + 4 * KD, r16);
                v4f acc[NBW];
#pragma unroll
                for (int n = 0; n < NBW; ++n) acc[n] = v4f{0.f, 0.f, 0.f, 0.f};
#define FLEX_BF_MFMA(X, Y)                                                                         \
    _Pragma("unroll") for (int n = 0; n < NBW; ++n)                                               \
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(X, Y[n], acc[n], 0, 0, 0)
                FLEX_BF_MFMA(aL, gH);   // small terms first
                FLEX_BF_MFMA(aH, gL);
                FLEX_BF_MFMA(aM, gM);
                FLEX_BF_MFMA(aM, gH);
                FLEX_BF_MFMA(aH, gM);
                FLEX_BF_MFMA(aH, gH);
#undef FLEX_BF_MFMA
#pragma unroll
                for (int n = 0; n < NBW; ++n) tot[c][n] = st == 0 ? tot[c][n] + acc[n] : tot[c][n] - acc[n];
            }
        }
    }

    if (idle) return;                      // (their part of the partial is read and dropped)
    flush(tiles > FLUSH);                  // a workgroup without tiles still writes its (zero) partial
}

// ---------------------------------------------------------------------------
// The same for blocks of 128 output channels: rows are gathered and weighed half as often (at 64 channels that is what the vector ALU
// does most of the time).  The 256 x 128 sums fill half of a contracting wave's registers, and the tiles all of LDS: 160 KB.
//
// A tile goes through in halves of 32 points -- the first four of every gathering wave's eight, then the others --, one depth
// step of the matrix op each, in two buffers: a half is parked while the one before it is contracted, and one barrier hands
// both over.  (Whole tiles in one buffer, parked between two barriers: 855 us at 128 -> 128 and 1M points where halves take 780,
// and 759 with the contracting waves' priority raised; blocks of 64 channels in halves lose, 1005 -> 1050.)
// Sums and their rounding are those of the kernel above, and the chains half as long: 2-norm error 128 -> 128 at 30k points 1.2e-7 ->
// 1.1e-7, at 200k 2.0e-7 -> 1.6e-7, at 1M 2.27e-7 -> 2.25e-7.
// What bounds it: no unit alone; at 128 -> 128, 1M points, the matrix cores are busy 51 percent of the time, the vector ALU 74 (four clocks an
// instruction, matrix ops among them), no bank conflicts; the contraction alone would take 520 us of the 759, the gathering alone 415.  us, 64 channels a block -> 128: 128 -> 128, 1M points
// 960 -> 759; 256 -> 256, 250k 918 -> 760; 512 -> 512, 109k 1600 -> 1240; K = 16: 1290 -> 940, 1246 -> 905, 2130 -> 1540.
// ---------------------------------------------------------------------------

// Three-piece bf16 tiles whose rows are whole multiples of 256 bytes: the byte address inside a row XORed with bf3x_swizzle(row).
// A turn of the transposing reads (32 lanes, 64 banks) takes 32 bytes each of rows 0-3 and 8-11 (mod 16), eight places that the
// three bits part; a turn of the 8-byte stores takes 128 bytes each of rows 2i and 2i + 1, which bit 7 parts.
__device__ __forceinline__ int bf3x_swizzle(int row) { return ((row & 1) << 7) | ((row & 2) << 4) | ((row & 8) << 3); }
// byte address v + K inside a row; K: a constant, so that all but its bit 7 is an offset in the instruction.
// v below 128, or K a multiple of 256.
__device__ __forceinline__ int bf3x_at(int v, int K, int swizzle) { return (v ^ swizzle ^ (K & 128)) + (K & ~128); }

static __global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
void tile_grad_theta128_kernel(const TileArgs a, const float *__restrict__ g_rows, int n_ho, float *__restrict__ partials)
{
    constexpr int IC = 64, KD = 4 * IC, OC = 128, T = 64, H = 32;
    constexpr int AS = 6 * KD, GS = 6 * OC;
    static_assert(AS % 256 == 0 && GS % 256 == 0, "rows of whole bank turns");
    __shared__ __attribute__((aligned(16))) char s_A[2][H * AS];
    __shared__ __attribute__((aligned(16))) char s_G[2][H * GS];
    __shared__ __attribute__((aligned(16))) float s_ent[8][2][64][4];

    const int p = blockIdx.x / a.chunks, hi = p / n_ho, ho = p - hi * n_ho;
    const TileSchedule sc(a.total, (int)blockIdx.x - p * a.chunks, a.chunks);
    const int tiles = sc.first < sc.end ? (sc.end - sc.first + sc.step - 1) / sc.step : 0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    if (wave < 8) {
        // ---- gather ----
        if (tiles == 0) return;
        const int lane = threadIdx.x & 63, t = lane & 15, grp = lane >> 4;
        const int row = 4 * wave + grp, swizzle = bf3x_swizzle(row);
        gather_steps<false, false, true>(a, sc, tiles, 8 * wave, hi, s_ent[wave], [&](v4f (&acc)[4], int half) __attribute__((always_inline)) {
            if (a.w_in % 4 != 0) put_channels_right(acc, 64 * hi + 4 * t - tile_lane_channel(a, hi));
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                unsigned h0, m0, l0, h1, m1, l1;
                split_bf3(acc[0][jj], acc[1][jj], h0, m0, l0);
                split_bf3(acc[2][jj], acc[3][jj], h1, m1, l1);
                char *d = s_A[half] + row * AS + bf3x_at(8 * t, 2 * jj * IC, swizzle);
                *reinterpret_cast<uint2 *>(d) = make_uint2(h0, h1);
                *reinterpret_cast<uint2 *>(d + 2 * KD) = make_uint2(m0, m1);
                *reinterpret_cast<uint2 *>(d + 4 * KD) = make_uint2(l0, l1);
            }
            __syncthreads();               // this half is complete, the one before it is contracted
        });
        return;
    }

    // ---- contract: MBW 16-row blocks x two 16-column blocks of the partial per wave ----
    constexpr int NBW = 2, WN = OC / (16 * NBW), WM = 8 / WN, MBW = KD / 16 / WM, FLUSH = 64;
    // a wave's row blocks: half of them in each 256 bytes of a row
    constexpr int MBH = MBW / 2;
    const int cw = wave - 8, wn = cw % WN, wm = cw / WN;
    __builtin_amdgcn_s_setprio(3);         // the matrix cores' chain is the longer one: 780 -> 759 us at 128 -> 128, 1M points
    v4f tot[MBW][NBW];                     // the sums since the last move to the partial

    float *dst = partials + (int64_t)blockIdx.x * KD * OC;
    // What a lane needs of its number is formed where it is used, not kept through the loop: the registers are full.
    auto lane_now = [&]() {
        int l;
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
        return l;
    };
    auto flush = [&](bool add) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < MBW; ++c) {
            const int l = lane_now();
            const unsigned at = 4u * (unsigned)((16 * (MBH * wm + c % MBH + 8 * (c / MBH)) + 4 * (l >> 4)) * OC + 32 * wn + (l & 15));
            auto place = [&](int n, int i) { return reinterpret_cast<float *>(reinterpret_cast<char *>(dst) + (at + 4u * (unsigned)(i * OC + 16 * n))); };
            if (add) {
                v4f old[NBW];
#pragma unroll
                for (int n = 0; n < NBW; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) old[n][i] = *place(n, i);
#pragma unroll
                for (int n = 0; n < NBW; ++n) tot[c][n] = old[n] + tot[c][n];
            }
#pragma unroll
            for (int n = 0; n < NBW; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) *place(n, i) = tot[c][n][i];
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Upstream gradient of a half: row r of its tile is point 8 * (r / 4) + 4 * half + r % 4 of the 64, as the gathering
    // waves have it; CH four-float chunks per thread, ROWS rows apart.
    constexpr int CPR = OC / 4, ROWS = 512 / CPR, CH = H / ROWS;
    TileWalk tw(sc, a.tpc);
    v4f gv[CH];
    auto load_g = [&](int half) __attribute__((always_inline)) {
        const int ctid = 64 * cw + lane_now(), r = ctid / CPR;
        const auto rows = row_buffer(g_rows + (int64_t)tw.b * a.N * a.w_out, 4u * (unsigned)a.N * (unsigned)a.w_out);
        const int col = min(OC * ho + 4 * (ctid % CPR), a.w_out - 4);      // past the row's end the last four again
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            // the row behind the cloud's last reads as zeros
            const int l = min(tw.tic * T + 8 * ((r + ROWS * c) >> 2) + 4 * half + (r & 3), a.N);
            gv[c] = load_row4(rows, 4u * ((unsigned)l * (unsigned)a.w_out + (unsigned)col));
        }
    };
    auto store_g = [&](int half) __attribute__((always_inline)) {
        const int ctid = 64 * cw + lane_now(), r = ctid / CPR, v = 8 * (ctid % CPR);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            char *row = s_G[half] + (r + ROWS * c) * GS;
            const int swizzle = bf3x_swizzle(r + ROWS * c);
            unsigned h0, m0, l0, h1, m1, l1;
            if (a.w_out % 4 != 0) put_channels_right(gv[c], max(0, OC * ho + 4 * (ctid % CPR) - (a.w_out - 4)));
            const v4f g = half == 0 ? gv[c] : -gv[c];              // (the second 32 points: see above)
            split_bf3(g[0], g[1], h0, m0, l0);
            split_bf3(g[2], g[3], h1, m1, l1);
            *reinterpret_cast<uint2 *>(row + bf3x_at(v, 0, swizzle)) = make_uint2(h0, h1);
            *reinterpret_cast<uint2 *>(row + bf3x_at(v, 2 * OC, swizzle)) = make_uint2(m0, m1);
            *reinterpret_cast<uint2 *>(row + bf3x_at(v, 4 * OC, swizzle)) = make_uint2(l0, l1);
        }
    };
    // A row block's three pieces are multiplied one after the other, small terms first, and the next block's take the
    // registers as they fall free.
    auto contract = [&](int half) __attribute__((always_inline)) {
        unsigned a_at[MBH], g_at[NBW];         // byte places of the wave's blocks
        const int l = lane_now(), r = 8 * (l >> 4) + ((l >> 2) & 3), col = 8 * (l & 3);
#pragma unroll
        for (int c = 0; c < MBH; ++c) a_at[c] = (unsigned)(r * AS + bf3x_at(32 * (MBH * wm + c) + col, 0, bf3x_swizzle(r)));
#pragma unroll
        for (int n = 0; n < NBW; ++n) g_at[n] = (unsigned)(r * GS + bf3x_at(64 * wn + 32 * n + col, 0, bf3x_swizzle(r)));
        auto frag_a = [&](int c, int piece) __attribute__((always_inline)) {
            return read_tr_at(s_A[half] + a_at[c % MBH] + (256 * (c / MBH) + 2 * KD * piece), AS);
        };
        auto frag_g = [&](int n, int piece) __attribute__((always_inline)) {
            return read_tr_at(s_G[half] + g_at[n] + 2 * OC * piece, GS);
        };
        bf8 aL = frag_a(0, 2), aM = frag_a(0, 1), aH = frag_a(0, 0), gH[NBW], gM[NBW], gL[NBW];
#pragma unroll
        for (int n = 0; n < NBW; ++n) {
            gH[n] = frag_g(n, 0);
            gM[n] = frag_g(n, 1);
            gL[n] = frag_g(n, 2);
        }
#pragma unroll
        for (int c = 0; c < MBW; ++c) {
            v4f acc[NBW];
#pragma unroll
            for (int n = 0; n < NBW; ++n) acc[n] = v4f{0.f, 0.f, 0.f, 0.f};
            __builtin_amdgcn_sched_barrier(0);
#define FLEX_BF_MFMA(X, Y)                                                                         \
    _Pragma("unroll") for (int n = 0; n < NBW; ++n)                                               \
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(X, Y[n], acc[n], 0, 0, 0)
            FLEX_BF_MFMA(aL, gH);
            if (c + 1 < MBW) aL = frag_a(c + 1, 2);
            __builtin_amdgcn_sched_barrier(0);
            FLEX_BF_MFMA(aM, gM);
            FLEX_BF_MFMA(aM, gH);
            if (c + 1 < MBW) aM = frag_a(c + 1, 1);
            __builtin_amdgcn_sched_barrier(0);
            FLEX_BF_MFMA(aH, gL);
            FLEX_BF_MFMA(aH, gM);
            FLEX_BF_MFMA(aH, gH);
            if (c + 1 < MBW) aH = frag_a(c + 1, 0);
            __builtin_amdgcn_sched_barrier(0);
#undef FLEX_BF_MFMA
#pragma unroll
            for (int n = 0; n < NBW; ++n) {
                tot[c][n] = half == 0 ? tot[c][n] + acc[n] : tot[c][n] - acc[n];
                asm volatile("" : "+v"(tot[c][n]));        // here: put off, the products would wait in registers
            }
        }
    };

    if (tiles > 0) {
        load_g(0);
        store_g(0);
        load_g(1);
        __syncthreads();                   // the first half is complete
    }
    int k = 0;
    do {                                   // (a workgroup without tiles still writes its partial, zeros)
#pragma unroll
        for (int c = 0; c < MBW; ++c)
#pragma unroll
            for (int n = 0; n < NBW; ++n) tot[c][n] = v4f{0.f, 0.f, 0.f, 0.f};
        const int k0 = k, stop = min(tiles, k + FLUSH);
        for (; k < stop; ++k) {
            const bool more = k + 1 < tiles;
            store_g(1);
            tw.next_clamped();
            if (more) load_g(0);
            contract(0);
            __syncthreads();               // the second half is complete
            if (more) {
                store_g(0);
                load_g(1);
            }
            contract(1);
            if (more) __syncthreads();     // the next tile's first half is complete
        }
        flush(k0 > 0);
    } while (k < tiles);
}
#endif

}  // namespace flex
