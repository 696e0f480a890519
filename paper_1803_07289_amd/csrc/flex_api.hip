// C-ABI entry points of libflexconv: validation, workspace carving, dispatch.
#include "flex_common.hpp"
#include <stdlib.h>
#include <algorithm>
#include <mutex>
#include "../../include/flexconv.h"

namespace flex {

// ---- per-shape launchers generated from flex_shapes.def ------------------------
#define FLEX_SHAPE(DI, DO, W, T, OCC, WS)                                                             \
    hipError_t launch_gc_##DI##_##DO(const float *, const float *, const PosRef &, const int32_t *, const int32_t *, \
                                     const int32_t *, const int32_t *, const void *, int, float *, int, int, int, \
                                     int, int, hipStream_t);                                         \
    int theta_format_##DI##_##DO(int, int, int);                                                       \
    int route_##DI##_##DO(int, int, int);                                                              \
    bool gp_ok_##DI##_##DO(int, int);                                                                 \
    hipError_t launch_gp_##DI##_##DO(const float *, const int32_t *, const int32_t *, const int32_t *, \
                                     const void *, const float *, float *, float, int, int, int, int,  \
                                     int, hipStream_t);                                                        \
    hipError_t launch_gt_##DI##_##DO(const float *, const float *, const PosRef &, const int32_t *, const float *, \
                                     float *, int, int, int, int *, hipStream_t);
#include "flex_shapes.def"
#undef FLEX_SHAPE

// 64 -> 64 layers: feature and parameter gradients in one pass over the in-edge lists (flex_tiled_inst.hip, shape 64x64)
bool bwd_fused_ok_64_64(int N, int K);
hipError_t launch_bwd_fused_64_64(const float *g_rows, const float *own_rows, const PosRef &pos, const int32_t *nbr,
                                  const int32_t *off, const int32_t *src, const int32_t *order, const void *thetaP,
                                  float *grad_feat, float *partials, int *control, int B, int N, int K, int out_bcn,
                                  int *n_wg, hipStream_t s);
hipError_t launch_bwd_fused_late_64_64(const float *g_rows, const float *own_rows, const PosRef &pos,
                                       const int32_t *nbr, const void *thetaP, const float *grad_theta,
                                       const float *grad_bias, int Din, int Dout, float *partials, int *control, int B,
                                       int N, int K, hipStream_t s);

// parameter gradients of layers with both widths multiples of 128, block by block (same file, same shape)
hipError_t launch_reduce_partials(const float *partials, int n_wg, int DIP, int DOP, int n_blocks, int n_ho, int Din,
                                  int Dout, float *grad_theta, float *grad_bias, hipStream_t s);

// the 64-point tile kernels over fixed-K neighbour tensors / in-edge lists
hipError_t launch_tile_0(const TileArgs &a, int outw, int grid, hipStream_t s);
hipError_t launch_tile_1(const TileArgs &a, int outw, int grid, hipStream_t s);
hipError_t launch_tile_grad_theta(const TileArgs &a, const float *g_rows, int n_hi, int n_ho, int oc, bool f32, float *partials, hipStream_t s);
// rows of at most 16 channels, one point per lane (flex_narrow.hip)
hipError_t launch_narrow_0(const TileArgs &a, int grid, hipStream_t s);
hipError_t launch_narrow_1(const TileArgs &a, int grid, hipStream_t s);
hipError_t launch_narrow_records_0(const TileArgs &a, const float *rec, const float *rec4, int B, int n_out, hipStream_t s);
hipError_t launch_narrow_records_1(const TileArgs &a, const float *rec, const float *rec4, int B, int n_out, hipStream_t s);

bool gather_contract_supported(int DI, int DO)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS) \
    if (DI == DI_ && DO == DO_) return true;
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return false;
}

hipError_t launch_gather_contract(const float *rows, const float *pos, const PosRef &pr, const int32_t *nbr,
                                  const int32_t *off, const int32_t *src, const int32_t *order, const void *thetaP,
                                  int theta_fmt, float *out, int B, int N, int K, int DI, int DO,
                                  int csr, int out_bcn, hipStream_t s)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS) \
    if (DI == DI_ && DO == DO_)         \
        return launch_gc_##DI_##_##DO_(rows, pos, pr, nbr, off, src, order, thetaP, theta_fmt, out, B, N, K, csr, out_bcn, s);
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return hipErrorNotSupported;
}

int gather_contract_theta_format(int DI, int DO, int N, int K, int csr)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS) \
    if (DI == DI_ && DO == DO_) return theta_format_##DI_##_##DO_(N, K, csr);
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return 0;
}

int gather_contract_route(int DI, int DO, int N, int K, int csr)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS) \
    if (DI == DI_ && DO == DO_) return route_##DI_##_##DO_(N, K, csr);
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return 0;
}

bool grad_pos_supported(int DI, int DO, int N, int K)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS) \
    if (DI == DI_ && DO == DO_) return gp_ok_##DI_##_##DO_(N, K);
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return false;
}

hipError_t launch_grad_pos_term(const float *rows, const int32_t *nbr, const int32_t *off, const int32_t *src,
                                const void *thetaF, const float *dot_rows, float *grad_pos, float sign,
                                int accumulate, int B, int N, int K, int DI, int DO, int csr, hipStream_t s)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS)                                                               \
    if (DI == DI_ && DO == DO_)                                                                           \
        return launch_gp_##DI_##_##DO_(rows, nbr, off, src, thetaF, dot_rows, grad_pos, sign, accumulate, B, N, K, csr, s);
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return hipErrorNotSupported;
}

bool contract_in_fp32()
{
    static const bool f32 = [] {
        const char *v = getenv("FLEX_CONTRACT");
        return v != nullptr && v[0] == 'f' && v[1] == '3' && v[2] == '2' && v[3] == 0;
    }();
    return f32;
}

int lean_producer_mode()
{
    static const int mode = [] {
        const char *v = getenv("FLEX_PRODUCER");
        if (v == nullptr) return 2;
        if (v[0] == 's') return 0;
        if (v[0] == 'l') return 1;
        return 2;
    }();
    return mode;
}

// Wide layers (both widths multiples of 128): the paper's network doubles the feature length at every resolution
// stage while the point count drops by four (Sec. 4.3), so its deeper stages are of this kind.  They run on the 64-point
// tile kernels (FLEX_SPLIT=0 in the environment keeps 128 -> 128 on the single-pass fp32 kernels and the wider ones on the
// direct form, for comparisons).
static bool split_disabled()
{
    static const bool off = [] { const char *v = getenv("FLEX_SPLIT"); return v != nullptr && v[0] == '0'; }();
    return off;
}
// Can the 64-point tile kernels take this gather of w_in wide rows?  32-bit byte offsets inside a cloud, and one more
// row's worth of them for slots without an entry.
static bool tile_ok(int64_t N, int w_in)
{
    return !split_disabled() && !contract_in_fp32() && lean_producer_mode() != 0 && (N + 1) * w_in * 4 <= (1ll << 32) &&
           N * 12 < (1ll << 32);
}
static bool wide_shape(int Din, int Dout)
{
    return !split_disabled() && Din % 128 == 0 && Dout % 128 == 0 &&
           (int64_t)(Din / 64) * (Dout / 64) <= 65535;      // one grid row of the reduction per block
}
static bool wide_ok(int64_t N, int K, int Din, int Dout)
{
    return wide_shape(Din, Dout) && tile_ok(N, Din) && tile_ok(N, Dout) && (int64_t)K * N * 4 < (1ll << 32);
}

// Packed parameters of a wide layer, forward, as 64 x 128 blocks
static size_t wide_packed_bytes(int Din, int Dout) { return (size_t)(Din / 64) * (Dout / 128) * theta_f16_bytes(64, 128); }

// Parameter gradients on the 64-point tile kernels: blocks of [4*64 x oc], `chunks` workgroups each, two launches (partial sums
// per block and workgroup, then their reduction in double).  Rows are read at their own widths; what a block reaches past
// them is dropped by the reduction.
// Blocks of 128 output channels gather half as often, ones of 64 make twice the workgroups for a cloud of few tiles.  Costs in
// tenths of a microsecond, as measured: a tile 3.2 us for 64 channels and 5.0 for 128, whose larger partials take 3 more.
// us, 64 and 128: 128 -> 128, 2k points 15.8 and 17.9, 8k 23.5 and 24.7, 16k 29.8 and 29.6, 60k 66.6 and 60.9, 1M 970 and 782;
// 256 -> 256, 2k 24.6 and 28.5, 12k 59.5 and 52.6; 512 -> 512, 1k 30.6 and 34.6, 2k 43.2 and 43.1, 8k 126 and 109, 109k 1620 and 1270.
// f32: one side of at most 64 channels and the other of 65 to 128.  These widths have no kernel that splits its operands elsewhere (their
// listed ones, 64 -> 128 and 128 -> 64, contract in fp32), and are contracted in fp32 here too, in blocks of 64.
struct TileGradPlan { int oc, n_hi, n_ho, chunks; bool f32; };
static TileGradPlan tile_grad_plan(int64_t B, int64_t N, int Din, int Dout)
{
    const int64_t tiles = B * cdiv64(N, 64), cus = device_cu_count();
    TileGradPlan best{};
    int64_t least = 0;
    const bool f32 = std::min(Din, Dout) <= 64 && std::max(Din, Dout) > 64 && std::max(Din, Dout) <= 128;
    for (const int oc : {64, 128}) {
        if (f32 && oc > 64) break;
        TileGradPlan p{oc, (Din + 63) / 64, (Dout + oc - 1) / oc, 1, f32};
        const int64_t blocks = (int64_t)p.n_hi * p.n_ho;
        p.chunks = (int)std::max<int64_t>(1, std::min(tiles, cus / blocks));
        const int64_t rounds = cdiv64(blocks * p.chunks, cus) * cdiv64(tiles, p.chunks);
        const int64_t cost = oc == 64 ? 32 * rounds : 50 * rounds + 30;
        if (oc == 64 || cost < least) { least = cost; best = p; }
    }
    return best;
}
static size_t tile_grad_partial_bytes(int64_t B, int64_t N, int Din, int Dout)
{
    const TileGradPlan p = tile_grad_plan(B, N, Din, Dout);
    return align256(sizeof(float) * (size_t)p.n_hi * p.n_ho * p.chunks * 4 * 64 * p.oc);
}

// rows [B*N, w_in], g_rows [B*N, w_out]: the tensors, or copies of at least four channels; (Din, Dout): the parameters' widths.
static hipError_t tile_grad_theta(const float *rows, int w_in, const float *pos, const int32_t *nbr, const float *g_rows, int w_out,
                                  float *partials, float *grad_theta, float *grad_bias, int B, int N, int K, int Din, int Dout,
                                  hipStream_t s)
{
    const TileGradPlan p = tile_grad_plan(B, N, Din, Dout);
    TileArgs a{};
    a.rows = rows; a.pos = pos; a.nbr = nbr;
    a.rs = a.w_in = w_in; a.w_out = w_out;
    a.N = N; a.K = K; a.tpc = (N + 63) / 64; a.n_in = 1; a.chunks = p.chunks;
    const int64_t total = (int64_t)B * a.tpc;
    if (total > 0x7fffffff || (int64_t)p.n_hi * p.n_ho * p.chunks > 0x7fffffff) return hipErrorInvalidValue;
    a.total = (int)total;
    hipError_t e = launch_tile_grad_theta(a, g_rows, p.n_hi, p.n_ho, p.oc, p.f32, partials, s);
    if (e != hipSuccess) return e;
    return launch_reduce_partials(partials, p.chunks, 64, p.oc, p.n_hi * p.n_ho, p.n_ho, Din, Dout, grad_theta, grad_bias, s);
}

// Workspace bytes of the packed parameters in either format (rows padded to 4, columns to 16).
static size_t theta_ws_bytes(int rows, int cols)
{
    const int RP = (rows + 3) / 4 * 4, CP = (cols + 15) / 16 * 16;
    const size_t f32 = align256(sizeof(float) * (size_t)4 * RP * CP);
    const size_t f16 = theta_f16_bytes(RP, CP);
    return f32 > f16 ? f32 : f16;
}

static int shape_tile_points(int DI, int DO)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS) \
    if (DI == DI_ && DO == DO_) return T;
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return 0;
}

static int shape_wg_per_cu(int DI, int DO)
{
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS) \
    if (DI == DI_ && DO == DO_) return ((OCC * 4) / W > 0) ? (OCC * 4) / W : 1;
#include "flex_shapes.def"
#undef FLEX_SHAPE
    return 0;
}

static inline int pad4(int x) { return (x + 3) / 4 * 4; }
static inline int pad16(int x) { return (x + 15) / 16 * 16; }

size_t grad_theta_partial_bytes(int64_t B, int64_t N, int Din, int Dout)
{
    const int T = shape_tile_points(Din, Dout);
    if (T == 0) return 0;
    const int64_t tiles = B * ((N + T - 1) / T);
    const int grid = persistent_grid(tiles, shape_wg_per_cu(Din, Dout));
    return align256(sizeof(float) * (size_t)grid * 4 * pad4(Din) * pad16(Dout));
}

// (Dki, Dko): the widths of the rows, which may be padded; (Din, Dout): the parameters'.
static hipError_t launch_grad_theta(const float *rows, const float *pos, const PosRef &pr, const int32_t *nbr, const float *g_rows,
                                    float *partials, float *grad_theta, float *grad_bias, int B, int N, int K, int Dki,
                                    int Dko, int Din, int Dout, hipStream_t s)
{
    int n_wg = 0;
    hipError_t e = hipErrorNotSupported;
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS)                                                    \
    if (Dki == DI_ && Dko == DO_)                                                         \
        e = launch_gt_##DI_##_##DO_(rows, pos, pr, nbr, g_rows, partials, B, N, K, &n_wg, s);
#include "flex_shapes.def"
#undef FLEX_SHAPE
    if (e != hipSuccess) return e;
    return launch_reduce_partials(partials, n_wg, pad4(Dki), pad16(Dko), 1, 1, Din, Dout, grad_theta, grad_bias, s);
}

// ---- the 64-point tile kernels ------------------------------------------------------------
// Do they?  Where the gathered rows are wider than the 64 channels that the wave-specialised kernels hold the parameters
// of in registers (those would walk the cloud once per 64 channels: 128 -> 128, 1M points, forward 819 against 755 us,
// feature gradient 965 against 809; 512 -> 512, 109k points, 1350 against 860 and 1580 against 860), and where those would
// need zero-padded copies of the tensors (K = 8, forward and feature gradient, copies against here: 50 -> 50, 4k points 37
// and 43 against 22 and 20, 100k 88 and 121 against 40 and 58, 1M 600 and 867 against 270 and 407; 64 -> 13 forward, 4k,
// 100k and 1M points 27, 63, 460 against 21, 36, 235; 20 -> 13 forward 27, 52, 323 against 20, 37, 218).
// rs: row stride.
static bool use_tile(int64_t N, int w_in, int rs, bool padded) { return tile_ok(N, rs) && (w_in > 64 || padded); }

struct TilePlan { int outw, n_in, n_out; };
static size_t tile_bytes(const TilePlan &p) { return (size_t)p.n_in * p.n_out * theta_f16_bytes(64, p.outw); }
// How a gather is cut: input blocks of 64 channels, output blocks as wide as pays.  A wider output block gathers its rows
// for more channels; a narrower one makes more jobs for a cloud of few tiles.  The costs of a tile and input block
// (units of 260 clocks) are measured ones.  Packed parameters within `room` bytes go before cheaper ones that are not: wide
// output blocks reach further past the width.
static TilePlan tile_plan(int64_t B, int64_t N, int w_in, int w_out, size_t room)
{
    TilePlan p{};
    p.n_in = (w_in + 63) / 64;
    const int64_t tiles = B * cdiv64(N, 64);
    const int widths[3] = {64, 128, 256}, cost[3] = {50, 55, 75};
    int64_t best = -1;
    bool best_fits = false;
    for (int i = 0; i < 3; ++i) {
        if (i > 0 && widths[i] >= 2 * w_out) break;
        TilePlan q{widths[i], p.n_in, (w_out + widths[i] - 1) / widths[i]};
        const int64_t c = cdiv64(tiles * q.n_out, device_cu_count()) * cost[i];
        const bool fits = tile_bytes(q) <= room;
        if (best < 0 || (fits != best_fits ? fits : c < best)) { best = c; best_fits = fits; p = q; }
    }
    return p;
}

// Workgroups per output block of a persistent grid: as many as there are tiles, at most `most` (what the device holds at
// once), in whole multiples of 8 where that leaves any, so that a share's number tells its XCD.  Never more than the
// device holds: rounded up, three output blocks were 264 workgroups on 256 CUs, and the last eight ran alone for as long as
// all the others before them (128 -> 768, 100k points, three 256-wide blocks: 502 us, 393 in one round).
static int output_block_shares(int64_t tiles, int64_t most)
{
    const int64_t held = most >= 8 ? most / 8 * 8 : std::max<int64_t>(most, 1);
    return (int)std::min((tiles + 7) / 8 * 8, held);
}

// rows [B*N, rs] (w_in channels used) onto out [B, N, w_out] or, out_bcn, [B, w_out, N]
static hipError_t tile_launch(const TilePlan &p, const float *rows, int rs, int w_in, const float *pos,
                               const int32_t *nbr, const int32_t *off, const int32_t *src, const int32_t *order,
                               const void *theta, float *out, int w_out, int out_bcn, int B, int N, int K, hipStream_t s)
{
    TileArgs a{};
    a.rows = rows; a.pos = pos; a.nbr = nbr; a.off = off; a.src = src; a.order = order;
    a.theta = (const char *)theta; a.out = out;
    a.out_c = out_bcn ? N : 1; a.out_l = out_bcn ? 1 : w_out; a.out_b = (int64_t)N * w_out;
    a.rs = rs; a.w_in = w_in; a.w_out = w_out;
    a.blk_bytes = (int)theta_f16_bytes(64, p.outw);
    a.exp_off = (int)theta_f16_exp_offset(64, p.outw);
    a.rs_off = (int)theta_f16_rscale_offset(64, p.outw);
    a.N = N; a.K = K; a.tpc = (N + 63) / 64; a.n_in = p.n_in;
    const int64_t total = (int64_t)B * a.tpc;
    if (total > 0x7fffffff) return hipErrorInvalidValue;
    a.total = (int)total;
    a.chunks = output_block_shares(total, device_cu_count() / p.n_out);
    const int grid = p.n_out * a.chunks;
    return off != nullptr ? launch_tile_1(a, p.outw, grid, s) : launch_tile_0(a, p.outw, grid, s);
}

// ---- rows of at most 16 channels ----------------------------------------------------------
// rs: row stride.  Up to 16 channels, because there a lane per point was never the slower form and beyond it the 4 W sums
// of a point do not fit a lane's registers.  us, forward / feature gradient (the wider sums in the other direction), on the
// kernels that take these layers otherwise -> here.  1M points, K = 8: 9 and 64 (lean) 173 / 332 -> 130 / 175, 3 and 32
// (zero-padded on the lean kernels) 307 / 645 -> 55 / 164, 16 and 64 (tiles) 251 / 348 -> 158 / 278; 100k points, K = 16:
// 9 and 64 39 / 68 -> 26 / 38, 16 and 64 49 / 70 -> 29 / 58; 1k to 16k points, where a call is its launches, 18 / 19
// either way.
static bool use_narrow(int64_t N, int w_in, int rs) { return w_in <= 16 && tile_ok(N, rs); }
static int narrow_rp(int w_in) { return w_in <= 8 ? 8 : 16; }
static int narrow_blocks(int w_out) { return (w_out + 63) / 64; }
static size_t narrow_bytes(int w_in, int w_out) { return (size_t)narrow_blocks(w_out) * theta_f16_bytes(narrow_rp(w_in), 64); }

// theta: packed; bias not null (forward, no records): theta and bias are the tensors, which the kernel's waves pack themselves
// rec (null: none): the rows' records, the fourth channels of four-channel quads behind them
static hipError_t narrow_launch(const float *rows, int rs, int w_in, const float *pos, const float *rec, const int32_t *nbr,
                                const int32_t *off, const int32_t *src, const int32_t *order, const void *theta, const float *bias,
                                float *out, int w_out, int out_bcn, int B, int N, int K, hipStream_t s)
{
    const int rp = narrow_rp(w_in), n_out = narrow_blocks(w_out);
    TileArgs a{};
    a.rows = rows; a.pos = pos; a.nbr = nbr; a.off = off; a.src = src; a.order = order;
    a.theta = (const char *)theta; a.bias = bias; a.out = out;
    a.out_c = out_bcn ? N : 1; a.out_l = out_bcn ? 1 : w_out; a.out_b = (int64_t)N * w_out;
    a.rs = rs; a.w_in = w_in; a.w_out = w_out;
    a.blk_bytes = (int)theta_f16_bytes(rp, 64);
    a.exp_off = (int)theta_f16_exp_offset(rp, 64);
    a.rs_off = (int)theta_f16_rscale_offset(rp, 64);
    a.N = N; a.K = K; a.tpc = (N + 63) / 64; a.n_in = 1;
    const int64_t total = (int64_t)B * a.tpc;
    if (total > 0x7fffffff) return hipErrorInvalidValue;
    a.total = (int)total;
    if (rec != nullptr) {
        const float *rec4 = rec + (int64_t)B * N * 16;
        return off != nullptr ? launch_narrow_records_1(a, rec, rec4, B, n_out, s) : launch_narrow_records_0(a, rec, rec4, B, n_out, s);
    }
    // eight one-wave workgroups per CU are what its registers and LDS hold
    a.chunks = output_block_shares(total, (int64_t)device_cu_count() * 8 / n_out);
    const int grid = n_out * a.chunks;
    return off != nullptr ? launch_narrow_1(a, grid, s) : launch_narrow_0(a, grid, s);
}

// ---- plans -------------------------------------------------------------------------
// The kernels of one gather (the forward pass; the feature gradient over in-edge lists): rows of w_in channels, rs floats
// apart, onto w_out channels; (k_in, k_out): the listed widths that cover them.  Decided here, once, from everything it
// depends on (sizes, environment switches); the entry points dispatch on it, the workspace and the route query follow it.
// room: bytes that the packed parameters should stay within where they can.
struct GatherPlan {
    int route;             // FLEX_ROUTE_NARROW, FLEX_ROUTE_TILE or what gather_contract_route answers
    TilePlan tile;
    int fmt;               // of the packed parameters (listed widths)
    size_t packed;         // bytes of them
    bool own_widths() const { return route == FLEX_ROUTE_NARROW || route == FLEX_ROUTE_TILE; }
};
static GatherPlan plan_gather(int64_t B, int64_t N, int K, int w_in, int w_out, int rs, int k_in, int k_out, bool padded,
                              int csr, size_t room)
{
    GatherPlan g{};
    if (use_narrow(N, w_in, rs)) {
        g.route = FLEX_ROUTE_NARROW;
        g.packed = narrow_bytes(w_in, w_out);
    } else if (use_tile(N, w_in, rs, padded)) {
        g.route = FLEX_ROUTE_TILE;
        g.tile = tile_plan(B, N, w_in, w_out, room);
        g.packed = tile_bytes(g.tile);
    } else {
        g.route = gather_contract_route(k_in, k_out, (int)N, K, csr);
        g.fmt = gather_contract_theta_format(k_in, k_out, (int)N, K, csr);
        g.packed = theta_ws_bytes(k_in, k_out);
    }
    return g;
}

// Packs the parameters the way the planned kernels want them (transpose: the feature gradient's direction).
static hipError_t gather_pack(PrepList &prep, const GatherPlan &g, const float *theta, const float *bias, void *thetaP,
                              int Din, int Dout, int k_in, int k_out, int transpose, hipStream_t s)
{
    const int w_in = transpose ? Dout : Din, w_out = transpose ? Din : Dout;
    if (g.route == FLEX_ROUTE_NARROW)
        prep.pack_theta(theta, bias, thetaP, Din, Dout, narrow_rp(w_in), 64, 1, narrow_blocks(w_out), transpose);
    else if (g.route == FLEX_ROUTE_TILE)
        prep.pack_theta(theta, bias, thetaP, Din, Dout, 64, g.tile.outw, g.tile.n_in, g.tile.n_out, transpose);
    else if (g.fmt)
        prep.pack_theta(theta, bias, thetaP, Din, Dout, pad4(k_in), pad16(k_out), 1, 1, transpose);
    else
        return launch_pack_theta(theta, bias, (float *)thetaP, Din, Dout, pad4(k_in), pad16(k_out), transpose, s);
    return hipSuccess;
}

// Reading the ids ahead pays while they still stand in the memory-side cache (256 MB) when the gather asks for them, beside what the
// preparation reads and writes; beyond that it is a read more.  9 -> 64 in Z-order, nothing in a cache, us without and with: K = 8,
// 500k points (bytes below: 88 MB) 66 and 55, 1M (176) 123 and 99, 1.5M (264) 181 and 172, 1.7M (299) 202 and 203, 3M 366 and 390; K = 16,
// 1M (240) 147 and 123, 1.2M (288) 177 and 182, 2M 288 and 319; 5 -> 64, K = 8, 1.7M (272) 192 and 179.
static bool read_ids_ahead(int64_t points, int K, int w_in) { return points * (64 + 12 + 4 * w_in + 8 * K) <= 272ll << 20; }

// The records that the planned kernels gather instead of the tensors (Packed; packed null: none)
// nbr: what they will be gathered by (null: in-edge lists).
static void pack_points(PrepList &prep, const GatherPlan &g, const float *pos, const float *rows, float *packed, int B, int N,
                        int w_in, int bcn, const int32_t *nbr, int K)
{
    if (packed == nullptr) return;
    if (g.route == FLEX_ROUTE_NARROW)
        prep.records(pos, rows, packed, packed + (int64_t)B * N * 16, B, N, w_in, bcn,
                     read_ids_ahead((int64_t)B * N, K, w_in) ? nbr : nullptr, K);
    else prep.pack_pos(pos, packed, B, N);
}
static PosRef pos_ref(const float *pos, const float *packed, int N) { return packed ? pos_packed(packed, N) : pos_planar(pos, N); }

// rows [B*N, rs] onto out [B, N, w_out] or, out_bcn, [B, w_out, N]; on the listed widths' kernels rs = k_in, w_out = k_out
// packed (null: none): the point locations, on the narrow route the rows with them, as Packed says
static hipError_t gather_launch(const GatherPlan &g, const float *rows, int rs, int w_in, const float *pos, const float *packed,
                                const int32_t *nbr, const int32_t *off, const int32_t *src, const int32_t *order,
                                const void *thetaP, float *out, int w_out, int out_bcn, int B, int N, int K,
                                hipStream_t s)
{
    if (g.route == FLEX_ROUTE_NARROW)
        return narrow_launch(rows, rs, w_in, pos, packed, nbr, off, src, order, thetaP, nullptr, out, w_out, out_bcn, B, N, K, s);
    if (g.route == FLEX_ROUTE_TILE)
        return tile_launch(g.tile, rows, rs, w_in, pos, nbr, off, src, order, thetaP, out, w_out, out_bcn, B, N, K, s);
    return launch_gather_contract(rows, pos, pos_ref(pos, packed, N), nbr, off, src, order, thetaP, g.fmt, out, B, N, K, rs, w_out, off != nullptr,
                                  out_bcn, s);
}

static bool pad_disabled()
{
    static const bool off = [] { const char *v = getenv("FLEX_PAD"); return v != nullptr && v[0] == '0'; }();
    return off;
}

// Widths with neither a tiled nor a wide path of their own (FLEX_PAD=0 in the environment keeps them on the direct-form
// kernels, for comparisons): the nearest listed widths.  Parameter gradients and gathers that the kernels for any width do not
// take run on zero-padded copies at those: extra channels of the features / upstream gradient and
// extra rows / columns of the parameters are zero, so they add nothing, and the results are the leading channels / the
// leading block of what the padded layer returns.
static bool padded_shape(int Din, int Dout, int *DIp, int *DOp)
{
    if (pad_disabled() || wide_shape(Din, Dout)) return false;
    if (gather_contract_supported(Din, Dout) && gather_contract_supported(Dout, Din)) return false;
    if (Din <= 128 && Dout <= 128) {
        int64_t best = -1;
#define FLEX_SHAPE(DI_, DO_, W, T, OCC, WS)                                                         \
        if (DI_ >= Din && DO_ >= Dout && gather_contract_supported(DO_, DI_) &&                         \
            (best < 0 || (int64_t)DI_ * DO_ < best)) {                                                  \
            best = (int64_t)DI_ * DO_; *DIp = DI_; *DOp = DO_;                                          \
        }
#include "flex_shapes.def"
#undef FLEX_SHAPE
        return best > 0;
    }
    *DIp = (Din + 127) / 128 * 128;
    *DOp = (Dout + 127) / 128 * 128;
    return wide_shape(*DIp, *DOp);
}

// Do the parameter gradients run on the 64-point tile kernels, at the tensors' own widths?  (k_in, k_out): the listed widths.
// - Where a side is wider than 64 channels, always: 64 and 128 channels ran a workgroup's points in one chain of sums, other widths on
//   zero-padded copies.  us, K = 8, those and tiles: 64 -> 128, 3k points 23.9 and 17.2, 20k 47 and 33, 300k 378 and 236; 128 -> 64, 300 points
//   14.0 and 14.2, 3k 25.2 and 17.2, 300k 489 and 233; 100 -> 50, 3k 30.3 and 17.3, 300k 556 and 221; 3 -> 100, 300k 439 and 171; 160 -> 160,
//   3k 42 and 22, 300k 1124 and 650.
// - Below that the wave-specialised kernels take fewer points at a time.  Point-major tensors that they need copies of: at 64 x 64 channels
//   from 8k points on (all gradients, copies and tiles: 50 -> 50, 3k 30.8 and 31.1, 20k 45.8 and 44.7, 300k 210 and 165; 33 -> 64, 3k 28.3
//   and 29.2, 20k 43.4 and 42.5, 300k 182 and 159), at fewer where both tensors are copied, from 2^17 points on (20 -> 13, 50k 42.2 and
//   43.5, 300k 128 and 112; 12 -> 60, 50k 55.1 and 53.1, 300k 179 and 154; only the features, 6 -> 64, 300k 149 and 154, 16 -> 32 149 and
//   154).  Channel-major ones are copied either way (64 -> 13, 100k 73 and 82; 50 -> 50 93 and 96).
static bool use_tile_params(int64_t B, int64_t N, int K, int Din, int Dout, int k_in, int k_out, int bcn)
{
    const bool padded = k_in != Din || k_out != Dout;
    if (!tile_ok(N, std::max(Din, 4)) || !tile_ok(N, std::max(Dout, 4)) || (int64_t)K * N * 4 >= (1ll << 32)) return false;
    if ((int64_t)((Din + 63) / 64) * ((Dout + 63) / 64) > 65535) return false;       // one grid row of the reduction per block
    if (Din > 64 || Dout > 64) return true;
    if (!padded || bcn || Din < 4 || Dout < 4) return false;
    if (k_in == 64 && k_out == 64) return B * N >= 8192;
    return k_in != Din && k_out != Dout && B * N >= 1 << 17;
}

static size_t rows_bytes(int64_t B, int64_t N, int width) { return align256(sizeof(float) * (size_t)(B * N) * width); }

// Room for records behind a plan's own bytes: the point locations (PrepList::pack_pos) for the wave-specialised
// kernels, rows of at most 16 channels together with the locations (PrepList::records) for theirs.  A call whose workspace
// has it gathers records, any other the tensors; the results are the same bits.  (The tile kernels read the location tensor
// either way: a lane of theirs reads an entry's three components, the entries of a quarter wave are two slots of eight adjacent points,
// whose neighbours' components lie in a few lines of the tensor and in as many as sixteen of the records.  128 -> 128, 1M points,
// parameter gradient 1020 us, from records 1180; 64 -> 13, 2 x 50 021 points, forward 36 and 42.)  The wave-specialised kernels have
// them at every size: in Z-order they cost nothing beyond what two runs differ by (64 -> 64, K = 8, us without and with: forward, 4k
// points 12.3 and 12.1, 60k 23.6 and 23.3, 1M 225 and 224, all gradients 33, 52, 379 and 33, 52, 376; 32 -> 32 the same), in no order
// they gain from the smallest sizes on (forward, 60k 26.2 and 24.1, 300k 96 and 86; all gradients, 300k 151 and 143).
struct Packed {
    size_t at, best;                     // where they go; the workspace that has room for them (the plan's own: no use for them)
    const float *in(const char *ws, size_t have) const { return at != 0 && have >= best ? (const float *)(ws + at) : nullptr; }
};
// Which rows travel as records.  Shorter ones than 5 channels are not worth 64 bytes (3 -> 32, 500k points: 32 us, from records 44).
// Over in-edge lists all others do (us, K = 8, without and with: 64 -> 5, 256 points 11.6 and 10.0, 20k 16.0 and 12.9, 400k 84 and
// 46; 64 -> 9, 2k 14.1 and 12.7, 200k 40 and 33; 64 -> 16, 50k 27.9 and 17.2; only rows of 9 channels and lists of 3 and fewer
// lose between 100k and 1M points: K = 2, 200k 27 and 30, 1.2M 144 and 113).  The forward pass is decided by clouds in Z-order, nothing in a
// cache; a cloud in no order gains at all of these sizes (K = 4, 9 -> 64, 131k: 29 and 22, 300k 53 and 36):
// - Channel-major tensors are not copied for it then, from 2^17 points on (5 -> 64, K = 4, 131k: 25.9 and 20.4; 12 -> 13, 300k, 38.8 and 35.8).
// - Point-major, up to 32 result channels: their few stores hold up nothing (9 -> 32, K = 4, 1M 88 and 94; 9 -> 13, K = 8, 1M 86 and 95);
//   from K = 12 on (K = 16, 200k 36 and 33, 1M 138 and 117).
// - Wider results, K as long rows need fewer of: 9 -> 64, K = 8, 131k 21.6 and 21.7, 300k 38.8 and 35.5, 1M 142 and 93; 12 -> 64, K = 6,
//   200k 29.1 and 27.6; 6 -> 64, K = 8, 200k 25.9 and 26.1; 5 -> 64, K = 8, 300k 30.6 and 33.6, K = 10, 200k 30.8 and 28.7.
// - Below that K from 2^19 points on: 5 -> 64, K = 8, 400k 38.4 and 41.5, 500k 56 and 48, K = 4, 500k 42 and 47, 600k 64 and 53; 12 -> 64,
//   K = 4, 200k 24.7 and 27.3, 600k 72 and 59.
// A second array is not worth it there (16 -> 64, 400k: 50 and 52).
static bool use_records(int64_t B, int64_t N, int K, int w_in, int w_out, int csr, int bcn)
{
    const int64_t points = B * N;
    if (w_in < 5 || B * ((N + 15) / 16) > NARROW_RECORD_WAVES_MAX) return false;
    if (csr) return true;
    if (w_in > 12 || points < 1 << 17) return false;
    if (bcn) return true;
    if (w_out <= 32) return K >= 12;
    return K >= (w_in >= 8 ? 6 : w_in >= 6 ? 8 : 10) || points >= 1 << 19;
}
static Packed plan_packed(int64_t B, int64_t N, int K, int route, int w_in, int w_out, int csr, int bcn, size_t total)
{
    const int64_t record = use_records(B, N, K, w_in, w_out, csr, bcn) ? 64 + (narrow_record_channels(w_in) == 4 ? 16 : 0) : 0;
    const int64_t per_point = route == FLEX_ROUTE_LEAN ? 16 : route == FLEX_ROUTE_NARROW ? record : 0;
    if (per_point == 0 || N * 64 > (1ll << 32) - 128) return Packed{0, total};       // 32-bit offsets, and one past the end
    const size_t at = align256(total);
    return Packed{at, at + align256((size_t)(B * N) * per_point)};
}

struct FwdPlan {
    bool direct, padded, wide;
    int k_in, k_out;                     // the listed widths: the tensors' own unless padded
    GatherPlan gather;
    bool copy, copy_out;                 // rows are copied (turned round, padded); the result comes from a padded one
    size_t thetaP, rows, out, total;     // byte offsets / total
    Packed packed;
};
struct BwdPlan {
    bool direct, padded, wide;
    int k_in, k_out;
    GatherPlan gather;                   // of the feature gradient
    bool tile_params;                    // the parameter gradients run on the tile kernels
    bool copy_f, copy_g, copy_out;       // features, upstream gradient, result
    int c_in, c_out;                     // widths of the rows that the kernels read, the copies' or the tensors'
    bool fused;      // feature and parameter gradients, when both are asked for, come from the one-pass kernel
    size_t thetaP, featT, gT, gfP, partials, order, flag, in_off, in_src, inedge_ws, total;
    Packed packed;
};

static FwdPlan plan_fwd(int64_t B, int64_t N, int K, int Din, int Dout, int layout)
{
    FwdPlan p{};
    p.k_in = Din; p.k_out = Dout;
    p.padded = padded_shape(Din, Dout, &p.k_in, &p.k_out);
    p.wide = wide_ok(N, K, p.k_in, p.k_out);
    p.direct = !p.wide && !gather_contract_supported(p.k_in, p.k_out);
    // What the listed widths' kernels ask for (copies of features, parameters and result, their own packed parameters) is
    // what a call at padded widths is told to bring, whichever kernels it takes: the size, and with it what the static
    // scratch of flexconv_fwd_noalloc takes, does not change where they hand over to one another.
    const size_t copies = p.padded ? rows_bytes(B, N, p.k_in) + align256(sizeof(float) * (size_t)4 * p.k_in * p.k_out) +
                                         rows_bytes(B, N, p.k_out) : 0;
    p.total = copies + 256;
    p.packed = Packed{0, p.total};
    if (p.direct) return p;
    const bool bcn = layout == FLEX_LAYOUT_BCN;
    // a call whose parameters can be packed into the static scratch beside the turned rows is one that it takes
    const size_t turned = bcn ? rows_bytes(B, N, Din) : 0;
    p.gather = plan_gather(B, N, K, Din, Dout, Din, p.k_in, p.k_out, p.padded, 0,
                           turned < FLEX_NOALLOC_SCRATCH_BYTES ? FLEX_NOALLOC_SCRATCH_BYTES - turned : 0);
    const bool own = p.gather.own_widths();
    p.copy = bcn || (p.padded && !own);
    p.copy_out = p.padded && !own;
    size_t at = p.gather.packed;
    if (p.copy) { p.rows = at; at += rows_bytes(B, N, own ? Din : p.k_in); }
    if (p.copy_out) { p.out = at; at += rows_bytes(B, N, p.k_out); }
    if (p.padded)
        at = std::max(at, copies + (p.wide ? wide_packed_bytes(p.k_in, p.k_out) : theta_ws_bytes(p.k_in, p.k_out)));
    p.total = at;
    p.packed = plan_packed(B, N, K, p.gather.route, Din, Dout, 0, bcn, at);
    return p;
}

static BwdPlan plan_bwd(int64_t B, int64_t N, int K, int Din, int Dout, int layout, bool build)
{
    BwdPlan p{};
    p.k_in = Din; p.k_out = Dout;
    p.padded = padded_shape(Din, Dout, &p.k_in, &p.k_out);
    p.wide = wide_ok(N, K, p.k_in, p.k_out);
    p.direct = !p.wide && !(gather_contract_supported(p.k_in, p.k_out) && gather_contract_supported(p.k_out, p.k_in));
    p.total = 256;
    p.packed = Packed{0, p.total};
    if (p.direct) return p;
    p.gather = plan_gather(B, N, K, Dout, Din, p.k_out, p.k_out, p.k_in, p.padded, 1, SIZE_MAX);
    p.tile_params = (!p.padded || p.gather.own_widths()) &&      // (both then read rows of one stride)
                    use_tile_params(B, N, K, Din, Dout, p.k_in, p.k_out, layout == FLEX_LAYOUT_BCN);
    const bool own = p.gather.own_widths() && (p.tile_params || !p.padded);
    p.c_in = own ? std::max(Din, 4) : p.k_in;
    p.c_out = own ? std::max(Dout, 4) : p.k_out;
    p.copy_f = layout == FLEX_LAYOUT_BCN || p.c_in != Din;
    p.copy_g = layout == FLEX_LAYOUT_BCN || p.c_out != Dout;
    p.copy_out = p.padded && !p.gather.own_widths();
    size_t at = p.gather.packed;
    // (padded: the room for copies at the listed widths stays part of the size that callers are told, as in the forward plan)
    if (p.copy_f || p.padded) { p.featT = at; at += rows_bytes(B, N, std::max(p.c_in, p.k_in)); }
    if (p.copy_g || p.padded) { p.gT = at;    at += rows_bytes(B, N, std::max(p.c_out, p.k_out)); }
    if (p.copy_out) { p.gfP = at; at += rows_bytes(B, N, p.k_in); }
    p.partials = at;
    at += p.tile_params ? tile_grad_partial_bytes(B, N, Din, Dout) : grad_theta_partial_bytes(B, N, p.k_in, p.k_out);
    p.order = at; at += inedges_order_bytes(B * N);          // walking order of the feature gradient's gather
    p.fused = !p.padded && !p.wide && Din == 64 && Dout == 64 && bwd_fused_ok_64_64((int)N, K);
    if (p.fused) { p.flag = at; at += align256(fused_control_bytes()); }   // the one-pass kernel's flag and records
    if (build) {
        p.in_off = at;    at += align256(sizeof(int32_t) * (size_t)(B * N + 1));
        p.in_src = at;    at += align256(sizeof(int32_t) * (size_t)(B * N) * K);
        p.inedge_ws = at; at += inedges_ws_bytes(B * N, K);
    }
    p.total = at;
    p.packed = plan_packed(B, N, K, p.gather.route, Dout, Din, 1, layout == FLEX_LAYOUT_BCN, at);
    return p;
}

struct PosPlan {
    bool lean, blocked;
    size_t thetaC, thetaN, featT, gT, in_off, in_src, inedge_ws, total;
};
static inline int pad32(int x) { return (x + 31) / 32 * 32; }

static PosPlan plan_pos(int64_t B, int64_t N, int K, int Din, int Dout, int layout, bool build)
{
    PosPlan p{};
    p.lean = grad_pos_supported(Din, Dout, (int)N, K) && grad_pos_supported(Dout, Din, (int)N, K);
    size_t at = 0;
    if (p.lean) {
        p.thetaC = at; at += theta_pos_bytes(pad32(pad4(Din)), pad16(Dout));
        p.thetaN = at; at += theta_pos_bytes(pad32(pad4(Dout)), pad16(Din));
        if (layout == FLEX_LAYOUT_BCN) {
            p.featT = at; at += align256(sizeof(float) * (size_t)(B * N) * Din);
            p.gT = at;    at += align256(sizeof(float) * (size_t)(B * N) * Dout);
        }
        if (build) {
            p.in_off = at;    at += align256(sizeof(int32_t) * (size_t)(B * N + 1));
            p.in_src = at;    at += align256(sizeof(int32_t) * (size_t)(B * N) * K);
            p.inedge_ws = at; at += inedges_ws_bytes(B * N, K);
        }
    } else if (!pad_disabled() && grad_pos_supported(64, 64, (int)N, K)) {
        // other widths: the sum over 64 x 64 blocks of the parameters of the 64 -> 64 kernel's result on zero-padded
        // point-major 64-channel column blocks of the two tensors (featT / gT hold those blocks, one after the other)
        p.blocked = true;
        const int n_hi = (Din + 63) / 64, n_ho = (Dout + 63) / 64;
        p.thetaC = at; at += theta_pos_bytes(64, 64);
        p.thetaN = at; at += theta_pos_bytes(64, 64);
        at += align256(sizeof(float) * 3 * 64 * 64);        // not written: part of the size that callers have been told
        p.featT = at;  at += align256(sizeof(float) * (size_t)(B * N) * 64) * n_hi;
        p.gT = at;     at += align256(sizeof(float) * (size_t)(B * N) * 64) * n_ho;
        if (build) {
            p.in_off = at;    at += align256(sizeof(int32_t) * (size_t)(B * N + 1));
            p.in_src = at;    at += align256(sizeof(int32_t) * (size_t)(B * N) * K);
            p.inedge_ws = at; at += inedges_ws_bytes(B * N, K);
        }
    }
    p.total = at > 0 ? at : 256;
    return p;
}

static bool sizes_ok(int64_t B, int64_t N, int64_t K, int64_t Din, int64_t Dout)
{
    if (B <= 0 || N <= 0 || K <= 0 || Din <= 0 || Dout <= 0) return false;
    if (K > N) return false;
    if (B * N >= 0x7fffffffLL) return false;          // global point ids are int32
    if (B * N * K >= 0x7fffffffLL) return false;      // in-edge offsets are int32
    if (Din > 16384 || Dout > 16384) return false;
    return true;
}

// the draw's integer scale needs N <= 2^25 per cloud; one grid row per cloud
static bool idiss_sizes_ok(int64_t B, int64_t N)
{
    return sizes_ok(B, N, 1, 1, 1) && N <= (1 << 25) && B <= 65535;
}

// cell offsets are int32 over all clouds' cells; one grid row per cloud
static bool knn_sizes_ok(int64_t B, int64_t N, int64_t K)
{
    if (!sizes_ok(B, N, K, 1, 1) || B > 65535 || !knn_k_supported((int)K)) return false;
    const int64_t per_cloud = 8 * N < (1ll << 24) ? 8 * N : (1ll << 24);      // the most a cloud's grid may have
    return B * per_cloud < 0x7fffffffLL;
}

static bool ws_ok(const void *ws, size_t have, size_t need)
{
    return ws != nullptr && (((uintptr_t)ws) & 255) == 0 && have >= need;
}

#define FLEX_HIP(expr)                                  \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) return FLEX_ERR_HIP;      \
    } while (0)

}  // namespace flex

using namespace flex;

extern "C" {

const char *flex_status_string(int status)
{
    switch (status) {
    case FLEX_OK: return "ok";
    case FLEX_ERR_NULL: return "null pointer argument";
    case FLEX_ERR_SHAPE: return "bad size, layout or op";
    case FLEX_ERR_UNSUPPORTED: return "unsupported";
    case FLEX_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case FLEX_ERR_HIP: return "HIP launch error";
    case FLEX_ERR_TOO_LARGE: return "call needs more scratch memory than the library's static buffer holds";
    default: return "unknown status";
    }
}

int flexconv_has_fast_path(int Din, int Dout)
{
    int a, b;
    if (gather_contract_supported(Din, Dout) || wide_shape(Din, Dout)) return 1;
    return padded_shape(Din, Dout, &a, &b) ? 2 : 0;
}

// the wide path's name in the route query: 128 -> 128 point-major has one of its own
static int wide_route(int Din, int Dout, int layout)
{
    return Din == 128 && Dout == 128 && layout == FLEX_LAYOUT_BNC ? FLEX_ROUTE_SPLIT128 : FLEX_ROUTE_WIDE;
}

int flexconv_kernel_route(int op, int B, int N, int K, int Din, int Dout, int layout)
{
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return -1;
    if (op != FLEX_OP_CONV_FWD && op != FLEX_OP_CONV_BWD) return -1;
    if (!sizes_ok(B, N, K, Din, Dout)) return -1;
    auto answer = [&](const auto &p) {
        if (p.direct) return (int)FLEX_ROUTE_DIRECT;
        if (p.padded) return (int)(p.gather.own_widths() ? FLEX_ROUTE_PADDED : FLEX_ROUTE_PADDED_COPIES);
        if (p.wide) return wide_route(Din, Dout, layout);
        return p.gather.route;
    };
    if (op == FLEX_OP_CONV_FWD) return answer(plan_fwd(B, N, K, Din, Dout, layout));
    const BwdPlan p = plan_bwd(B, N, K, Din, Dout, layout, false);
    return p.fused ? (int)FLEX_ROUTE_LEAN_FUSED : answer(p);
}

size_t flexconv_workspace_bytes(int op, int B, int N, int K, int Din, int Dout, int layout)
{
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return 0;
    switch (op) {
    case FLEX_OP_CONV_FWD:
    case FLEX_OP_CONV_BWD:
    case FLEX_OP_CONV_BWD_BUILD: {
        if (!sizes_ok(B, N, K, Din, Dout)) return 0;
        if (op == FLEX_OP_CONV_FWD) return plan_fwd(B, N, K, Din, Dout, layout).total;
        return plan_bwd(B, N, K, Din, Dout, layout, op == FLEX_OP_CONV_BWD_BUILD).total;
    }
    case FLEX_OP_INEDGES: return sizes_ok(B, N, K, 1, 1) ? inedges_ws_bytes((int64_t)B * N, K) : 0;
    case FLEX_OP_CONV_BWD_POS: return sizes_ok(B, N, K, Din, Dout) ? plan_pos(B, N, K, Din, Dout, layout, false).total : 0;
    case FLEX_OP_CONV_BWD_POS_BUILD: return sizes_ok(B, N, K, Din, Dout) ? plan_pos(B, N, K, Din, Dout, layout, true).total : 0;
    case FLEX_OP_UPSAMPLE: return sizes_ok(B, N, 1, 1, 1) ? align256(sizeof(int32_t) * (size_t)B * N) : 0;
    case FLEX_OP_IDISS: return idiss_sizes_ok(B, N) ? idiss_ws_bytes(B, N) : 0;
    case FLEX_OP_KNN: return knn_sizes_ok(B, N, K) ? knn_ws_bytes(B, N, K) : 0;
    default: return 0;
    }
}

size_t flexconv_workspace_bytes_best(int op, int B, int N, int K, int Din, int Dout, int layout)
{
    const bool conv = op == FLEX_OP_CONV_FWD || op == FLEX_OP_CONV_BWD || op == FLEX_OP_CONV_BWD_BUILD;
    if (!conv || (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) || !sizes_ok(B, N, K, Din, Dout))
        return flexconv_workspace_bytes(op, B, N, K, Din, Dout, layout);
    if (op == FLEX_OP_CONV_FWD) return plan_fwd(B, N, K, Din, Dout, layout).packed.best;
    return plan_bwd(B, N, K, Din, Dout, layout, op == FLEX_OP_CONV_BWD_BUILD).packed.best;
}

int flexconv_fwd(const float *feat, const float *pos, const int32_t *nbr, const float *theta,
                 const float *bias, float *out, int B, int N, int K, int Din, int Dout, int layout,
                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (!feat || !pos || !nbr || !theta || !bias || !out) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, Din, Dout)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    const int bcn = (layout == FLEX_LAYOUT_BCN);
    const FwdPlan p = plan_fwd(B, N, K, Din, Dout, layout);
    if (!ws_ok(workspace, workspace_bytes, p.total)) return FLEX_ERR_WORKSPACE;
    if (p.direct) {
        FLEX_HIP(launch_generic_fwd(feat, pos, nbr, theta, bias, out, B, N, K, Din, Dout, !bcn, s));
        return FLEX_OK;
    }
    // the kernels for any width take rows as they are; only channel-major ones have to be turned round
    const int w_in = p.gather.own_widths() ? Din : p.k_in, w_out = p.copy_out ? p.k_out : Dout;
    PrepList prep;
    const float *rows = feat, *packed = p.packed.in(ws, workspace_bytes);
    const bool records = packed != nullptr && p.gather.route == FLEX_ROUTE_NARROW;       // made from the tensor as it is
    if (p.copy && !records) {
        prep.copy(feat, (float *)(ws + p.rows), B, N, Din, w_in, bcn, 0);
        rows = (const float *)(ws + p.rows);
    }
    if (p.gather.route == FLEX_ROUTE_NARROW && !records && !p.copy) {       // nothing to prepare but the parameters
        FLEX_HIP(narrow_launch(feat, Din, Din, pos, nullptr, nbr, nullptr, nullptr, nullptr, theta, bias, out, Dout, 0, B, N, K, s));
        return FLEX_OK;
    }
    void *thetaP = ws + p.thetaP;
    FLEX_HIP(gather_pack(prep, p.gather, theta, bias, thetaP, Din, Dout, p.k_in, p.k_out, 0, s));
    pack_points(prep, p.gather, pos, feat, (float *)packed, B, N, Din, bcn, nbr, K);
    FLEX_HIP(prep.launch(s));
    float *dst = p.copy_out ? (float *)(ws + p.out) : out;
    FLEX_HIP(gather_launch(p.gather, rows, w_in, w_in, pos, packed, nbr, nullptr, nullptr, nullptr, thetaP, dst, w_out,
                           bcn && !p.copy_out, B, N, K, s));
    if (p.copy_out) FLEX_HIP(launch_copy_rows(dst, out, B, N, p.k_out, Dout, 0, bcn, s));
    return FLEX_OK;
}

}  // extern "C"

// ---- flexconv_fwd_noalloc: the forward pass with the library's own static scratch memory -------------------
// The scratch (packed parameters; for other layouts / widths also the copies the plan asks for) lives in a
// file-scope device array instead of a caller workspace.  In host code the array's name is only a handle: the
// device address is looked up once per device (with that device current) and kept; every later use goes through
// the kept pointer.  Each GPU holds its own copy of the array at its own address.
static __device__ __align__(256) unsigned char scratch[FLEX_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES];       // device address of `scratch` on each device, nullptr until looked up
std::mutex g_scratch_mutex;

int static_scratch(void **ptr)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return FLEX_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return FLEX_ERR_HIP;
        if ((reinterpret_cast<uintptr_t>(p) & 255) != 0) return FLEX_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return FLEX_OK;
}
}  // namespace

extern "C" {

int flexconv_fwd_noalloc(const float *feat, const float *pos, const int32_t *nbr, const float *theta,
                         const float *bias, float *out, int B, int N, int K, int Din, int Dout, int layout,
                         void *stream)
{
    if (!feat || !pos || !nbr || !theta || !bias || !out) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, Din, Dout)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    const size_t need = flexconv_workspace_bytes(FLEX_OP_CONV_FWD, B, N, K, Din, Dout, layout);
    if (need == 0) return FLEX_ERR_SHAPE;
    if (need > (size_t)FLEX_NOALLOC_SCRATCH_BYTES) return FLEX_ERR_TOO_LARGE;
    void *ws = nullptr;
    const int st = static_scratch(&ws);
    if (st != FLEX_OK) return st;
    // Every byte of the plan that a kernel reads is written earlier in the same call (packed parameters with their
    // padding, exponent tables, turned and padded copies with their zeros), so nothing has to be cleared here.
    return flexconv_fwd(feat, pos, nbr, theta, bias, out, B, N, K, Din, Dout, layout, ws, need, stream);
}

int flex_inedges_build(const int32_t *nbr, int B, int N, int K, int32_t *in_off, int32_t *in_src,
                       void *workspace, size_t workspace_bytes, void *stream)
{
    if (!nbr || !in_off || !in_src) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, 1, 1)) return FLEX_ERR_SHAPE;
    if (!ws_ok(workspace, workspace_bytes, inedges_ws_bytes((int64_t)B * N, K))) return FLEX_ERR_WORKSPACE;
    FLEX_HIP(launch_inedges_build(nbr, B, N, K, in_off, in_src, workspace, (hipStream_t)stream));
    return FLEX_OK;
}

int flexconv_bwd(const float *feat, const float *pos, const int32_t *nbr, const float *theta,
                 const float *bias, const float *grad_out, float *grad_feat, float *grad_theta,
                 float *grad_bias, const int32_t *in_off, const int32_t *in_src, int B, int N, int K,
                 int Din, int Dout, int layout, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!feat || !pos || !nbr || !theta || !bias || !grad_out) return FLEX_ERR_NULL;
    if ((grad_theta == nullptr) != (grad_bias == nullptr)) return FLEX_ERR_NULL;
    if ((in_off == nullptr) != (in_src == nullptr)) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, Din, Dout)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    const bool build = (in_off == nullptr) && (grad_feat != nullptr);
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    const int bcn = (layout == FLEX_LAYOUT_BCN);
    const BwdPlan p = plan_bwd(B, N, K, Din, Dout, layout, build);
    if (!ws_ok(workspace, workspace_bytes, p.total)) return FLEX_ERR_WORKSPACE;
    if (p.direct) {
        FLEX_HIP(launch_generic_bwd(feat, pos, nbr, theta, bias, grad_out, grad_feat, grad_theta,
                                    grad_bias, B, N, K, Din, Dout, !bcn, s));
        return FLEX_OK;
    }
    if (build) {
        int32_t *off = (int32_t *)(ws + p.in_off), *src = (int32_t *)(ws + p.in_src);
        FLEX_HIP(launch_inedges_build(nbr, B, N, K, off, src, ws + p.inedge_ws, s));
        in_off = off;
        in_src = src;
    }
    void *thetaP = ws + p.thetaP;
    float *partials = (float *)(ws + p.partials);
    int32_t *order = (int32_t *)(ws + p.order);
    int *control = (int *)(ws + p.flag);
    const bool fused = p.fused && grad_theta && grad_feat;
    PrepList prep;
    const float *rows = feat, *g_rows = grad_out;
    // The parameter gradients alone have nothing else to prepare unless tensors are copied: the packing would be a launch of its
    // own, which only a cloud in no order earns back.  K = 8, us without and with it: 32 -> 32, 4k points 8.7 and 10.8, 300k 59 and 63,
    // 1M 173 and 180; 64 -> 64, 300k 96 and 100 (in no order 105 and 97).  The tile kernels read the location tensor.
    const float *packed = grad_feat || (!p.tile_params && (p.copy_f || p.copy_g)) ? p.packed.in(ws, workspace_bytes) : nullptr;
    const bool records = packed != nullptr && p.gather.route == FLEX_ROUTE_NARROW;       // made from the tensor as it is
    if (p.copy_g && (grad_theta || !records)) {
        prep.copy(grad_out, (float *)(ws + p.gT), B, N, Dout, p.c_out, bcn, 0);
        g_rows = (const float *)(ws + p.gT);
    }
    if (p.copy_f && grad_theta) {
        prep.copy(feat, (float *)(ws + p.featT), B, N, Din, p.c_in, bcn, 0);
        rows = (const float *)(ws + p.featT);
    }
    if (grad_feat) {
        FLEX_HIP(gather_pack(prep, p.gather, theta, bias, thetaP, Din, Dout, p.k_out, p.k_in, 1, s));
        prep.order(in_off, B, N, order);
    }
    if (fused) prep.clear(control, FUSED_FLAG_INTS);
    if (grad_feat || !records) pack_points(prep, p.gather, pos, grad_out, (float *)packed, B, N, Dout, bcn, nullptr, 0);
    const PosRef pr = pos_ref(pos, records ? nullptr : packed, N);
    FLEX_HIP(prep.launch(s));
    if (fused) {
        int n_wg = 0;
        FLEX_HIP(launch_bwd_fused_64_64(g_rows, rows, pr, nbr, in_off, in_src, order, thetaP, grad_feat, partials, control,
                                        B, N, K, bcn, &n_wg, s));
        FLEX_HIP(launch_reduce_partials_fused(partials, n_wg, control, Din, Dout, grad_theta, grad_bias, s));
        // is the result resolved by the f16 halves, and did no row overflow them?  if not (decided on the device), the
        // stand-alone kernel and a second reduction run; both return at once otherwise
        FLEX_HIP(launch_bwd_fused_late_64_64(g_rows, rows, pr, nbr, thetaP, grad_theta, grad_bias, Din, Dout, partials,
                                             control, B, N, K, s));
        FLEX_HIP(launch_reduce_partials_if(control, partials, n_wg, 64, 64, Din, Dout, grad_theta, grad_bias, s));
        return FLEX_OK;
    }
    if (grad_theta && p.tile_params)
        FLEX_HIP(tile_grad_theta(rows, p.c_in, pos, nbr, g_rows, p.c_out, partials, grad_theta, grad_bias, B, N, K, Din, Dout, s));
    else if (grad_theta)
        FLEX_HIP(launch_grad_theta(rows, pos, pr, nbr, g_rows, partials, grad_theta, grad_bias, B, N, K, p.k_in, p.k_out, Din,
                                   Dout, s));
    if (!grad_feat) return FLEX_OK;
    float *dst = p.copy_out ? (float *)(ws + p.gfP) : grad_feat;
    FLEX_HIP(gather_launch(p.gather, g_rows, p.c_out, p.gather.own_widths() ? Dout : p.k_out, pos, packed, nullptr, in_off, in_src,
                           order, thetaP, dst, p.copy_out ? p.k_in : Din, bcn && !p.copy_out, B, N, K, s));
    if (p.copy_out) FLEX_HIP(launch_copy_rows(dst, grad_feat, B, N, p.k_in, Din, 0, bcn, s));
    return FLEX_OK;
}

int flexpool_fwd(const float *feat, const int32_t *nbr, float *out, int32_t *argmax, int B, int N,
                 int K, int C, int layout, void *stream)
{
    if (!feat || !nbr || !out || !argmax) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, C, 1)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    FLEX_HIP(launch_pool_fwd(feat, nbr, out, argmax, B, N, K, C, layout == FLEX_LAYOUT_BNC,
                             (hipStream_t)stream));
    return FLEX_OK;
}

int flexpool_bwd(const float *grad_out, const int32_t *argmax, float *grad_feat,
                 const int32_t *in_off, const int32_t *in_src, int B, int N, int K, int C, int layout,
                 void *stream)
{
    if (!grad_out || !argmax || !grad_feat) return FLEX_ERR_NULL;
    if ((in_off == nullptr) != (in_src == nullptr)) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, in_off ? K : 1, C, 1)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    if (in_off)
        FLEX_HIP(launch_pool_bwd_gather(grad_out, argmax, in_off, in_src, grad_feat, B, N, C,
                                        layout == FLEX_LAYOUT_BNC, (hipStream_t)stream));
    else
        FLEX_HIP(launch_pool_bwd(grad_out, argmax, grad_feat, B, N, C, layout == FLEX_LAYOUT_BNC,
                                 (hipStream_t)stream));
    return FLEX_OK;
}

// FLEX_POOL_PLAN=1: the planned kernels wherever they can run (any size, any K); =0: never; unset: where they are faster
static int pool_plan_mode()
{
    static const int mode = [] { const char *e = getenv("FLEX_POOL_PLAN"); return !e ? -1 : e[0] == '0' ? 0 : 1; }();
    return mode;
}

size_t flexpool_plan_bytes(int B, int N, int K)
{
    if (!sizes_ok(B, N, K, 1, 1)) return 0;
    return pool_plan_bytes(B, N, K);
}

int flexpool_plan_build(const int32_t *in_off, const int32_t *in_src, int B, int N, int K, void *plan,
                        size_t plan_bytes, void *stream)
{
    if (!in_off || !in_src || !plan) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, 1, 1)) return FLEX_ERR_SHAPE;
    if (plan_bytes < pool_plan_bytes(B, N, K) || (reinterpret_cast<uintptr_t>(plan) & 255)) return FLEX_ERR_WORKSPACE;
    FLEX_HIP(launch_pool_plan_build(in_off, in_src, plan, B, N, K, (hipStream_t)stream));
    return FLEX_OK;
}

int flexpool_bwd_planned(const float *grad_out, const int32_t *argmax, float *grad_feat, const int32_t *in_off,
                         const int32_t *in_src, void *plan, size_t plan_bytes, int B, int N, int K, int C,
                         int layout, void *stream)
{
    if (!grad_out || !argmax || !grad_feat || !in_off || !in_src || !plan) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, C, 1)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    if (plan_bytes < pool_plan_bytes(B, N, K) || (reinterpret_cast<uintptr_t>(plan) & 255)) return FLEX_ERR_WORKSPACE;
    const int mode = pool_plan_mode();
    const bool can = layout == FLEX_LAYOUT_BNC && (C == 64 || C == 128 || C == 256);
    const bool pays = K <= FLEX_POOL_PLAN_MAX_K && (int64_t)B * N >= FLEX_POOL_PLAN_MIN_POINTS;
    if (can && (mode == 1 || (mode == -1 && pays)))
        FLEX_HIP(launch_pool_bwd_planned(grad_out, argmax, in_off, in_src, plan, grad_feat, B, N, K, C,
                                         (hipStream_t)stream));
    else        // widths and layouts the plan has no kernel for, sizes and list lengths it does not pay for: the list form, same sums
        FLEX_HIP(launch_pool_bwd_gather(grad_out, argmax, in_off, in_src, grad_feat, B, N, C,
                                        layout == FLEX_LAYOUT_BNC, (hipStream_t)stream));
    return FLEX_OK;
}

int flexpool_fwd_plan_build(const int32_t *nbr, int B, int N, int K, void *plan, size_t plan_bytes, void *stream)
{
    if (!nbr || !plan) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, 1, 1)) return FLEX_ERR_SHAPE;
    if (plan_bytes < pool_plan_bytes(B, N, K) || (reinterpret_cast<uintptr_t>(plan) & 255)) return FLEX_ERR_WORKSPACE;
    FLEX_HIP(launch_pool_fwd_plan_build(nbr, plan, B, N, K, (hipStream_t)stream));
    return FLEX_OK;
}

int flexpool_fwd_planned(const float *feat, const int32_t *nbr, float *out, int32_t *argmax, void *plan,
                         size_t plan_bytes, int B, int N, int K, int C, int layout, void *stream)
{
    if (!feat || !nbr || !out || !argmax || !plan) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, C, 1)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    if (plan_bytes < pool_plan_bytes(B, N, K) || (reinterpret_cast<uintptr_t>(plan) & 255)) return FLEX_ERR_WORKSPACE;
    const int mode = pool_plan_mode();
    const bool can = layout == FLEX_LAYOUT_BNC && (C == 64 || C == 128 || C == 256);
    const bool pays = K <= FLEX_POOL_PLAN_MAX_K && (int64_t)B * N >= FLEX_POOL_PLAN_MIN_POINTS;
    if (can && (mode == 1 || (mode == -1 && pays)))
        FLEX_HIP(launch_pool_fwd_planned(feat, nbr, plan, out, argmax, B, N, K, C, (hipStream_t)stream));
    else
        FLEX_HIP(launch_pool_fwd(feat, nbr, out, argmax, B, N, K, C, layout == FLEX_LAYOUT_BNC, (hipStream_t)stream));
    return FLEX_OK;
}

int flexconv_compose_1x1(const float *W, const float *theta, const float *bias, float *theta_c, float *bias_c,
                         int Din0, int Dmid, int Dout, void *stream)
{
    if (!W || !theta || !bias || !theta_c || !bias_c) return FLEX_ERR_NULL;
    if (Din0 <= 0 || Dmid <= 0 || Dout <= 0 || Din0 > 16384 || Dmid > 16384 ||
        Dout > 16384)
        return FLEX_ERR_SHAPE;
    FLEX_HIP(launch_compose_1x1(W, theta, bias, theta_c, bias_c, Din0, Dmid, Dout, (hipStream_t)stream));
    return FLEX_OK;
}

int flexconv_compose_1x1_bwd(const float *W, const float *theta, const float *bias, const float *grad_theta_c,
                             const float *grad_bias_c, float *grad_W, float *grad_theta, float *grad_bias,
                             int Din0, int Dmid, int Dout, void *stream)
{
    if (!W || !theta || !bias || !grad_theta_c || !grad_bias_c || !grad_W || !grad_theta || !grad_bias)
        return FLEX_ERR_NULL;
    if (Din0 <= 0 || Dmid <= 0 || Dout <= 0 || Din0 > 16384 || Dmid > 16384 ||
        Dout > 16384)
        return FLEX_ERR_SHAPE;
    FLEX_HIP(launch_compose_1x1_bwd(W, theta, bias, grad_theta_c, grad_bias_c, grad_W, grad_theta, grad_bias, Din0,
                                    Dmid, Dout, (hipStream_t)stream));
    return FLEX_OK;
}

int flex_idiss_phi(const float *pos, const int32_t *nbr, float *phi, int B, int N, int K, void *stream)
{
    return flex_idiss_phi_ws(pos, nbr, phi, B, N, K, nullptr, 0, stream);
}

// Packing is a launch, and pays on clouds in no order from 2^22 neighbours on; which order a cloud has is not known here, and a scan
// comes in its sensor's.  us without and with it, nothing in a cache, a room in the sensor's order | in Z-order: 100k points, K = 8: 13.3,
// 13.5 | 8.2, 11.2; 300k, K = 8: 27.7, 22.1 | 12.0, 14.6; 600k, K = 8: 51.3, 35.6 | 14.7, 20.6; 1M, K = 8: 87.4, 53.7 | 21.6, 25.0; 1M,
// K = 16: 184, 100 | 41.2, 36.9; 2.9M, K = 8 in Z-order 56.3, 55.0.
size_t flex_idiss_phi_workspace_bytes(int B, int N, int K)
{
    if (!sizes_ok(B, N, K, 1, 1) || (int64_t)B * N * K < 1 << 22) return 0;
    return sizeof(float) * 4 * (size_t)B * N;
}

int flex_idiss_phi_ws(const float *pos, const int32_t *nbr, float *phi, int B, int N, int K, void *workspace,
                      size_t workspace_bytes, void *stream)
{
    if (!pos || !nbr || !phi) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, 1, 1)) return FLEX_ERR_SHAPE;
    float *pos4 = ws_ok(workspace, workspace_bytes, sizeof(float) * 4 * (size_t)B * N) ? (float *)workspace : nullptr;
    FLEX_HIP(launch_idiss_phi(pos, nbr, phi, pos4, B, N, K, (hipStream_t)stream));
    return FLEX_OK;
}

int flex_idiss_sample(const float *phi, const uint32_t *u, int32_t *sel, int B, int N, int Ns,
                      void *workspace, size_t workspace_bytes, void *stream)
{
    if (!phi || !u || !sel) return FLEX_ERR_NULL;
    if (!idiss_sizes_ok(B, N) || Ns <= 0 || Ns > N) return FLEX_ERR_SHAPE;
    if (!ws_ok(workspace, workspace_bytes, idiss_ws_bytes(B, N))) return FLEX_ERR_WORKSPACE;
    FLEX_HIP(launch_idiss_sample(phi, u, sel, B, N, Ns, workspace, (hipStream_t)stream));
    return FLEX_OK;
}

int flex_selection_make_distinct(int32_t *sel, int B, int N, int Ns, void *workspace, size_t workspace_bytes,
                                 void *stream)
{
    if (!sel) return FLEX_ERR_NULL;
    if (!idiss_sizes_ok(B, N) || Ns <= 0 || Ns > N) return FLEX_ERR_SHAPE;
    if (!ws_ok(workspace, workspace_bytes, distinct_ws_bytes(B, Ns))) return FLEX_ERR_WORKSPACE;
    FLEX_HIP(launch_selection_make_distinct(sel, B, N, Ns, workspace, (hipStream_t)stream));
    return FLEX_OK;
}

int flex_knn(const float *pos, int32_t *nbr, int B, int N, int K, void *workspace, size_t workspace_bytes,
             void *stream)
{
    if (!pos || !nbr) return FLEX_ERR_NULL;
    if (!knn_sizes_ok(B, N, K)) return FLEX_ERR_SHAPE;
    if (!ws_ok(workspace, workspace_bytes, knn_ws_bytes(B, N, K))) return FLEX_ERR_WORKSPACE;
    FLEX_HIP(launch_knn(pos, nbr, B, N, K, workspace, (hipStream_t)stream));
    return FLEX_OK;
}

int flexpool_sub_fwd(const float *feat, const int32_t *nbr, const int32_t *sel, float *out,
                     int32_t *argmax, int B, int N, int Ns, int K, int C, int layout, void *stream)
{
    if (!feat || !nbr || !sel || !out || !argmax) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, C, 1) || Ns <= 0 || Ns > N) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    FLEX_HIP(launch_pool_sub_fwd(feat, nbr, sel, out, argmax, B, N, Ns, K, C, layout == FLEX_LAYOUT_BNC,
                                 (hipStream_t)stream));
    return FLEX_OK;
}

int flexpool_sub_bwd(const float *grad_out, const int32_t *argmax, const int32_t *in_off,
                     const int32_t *in_src, float *grad_feat, int B, int N, int Ns, int K, int C,
                     int layout, void *stream)
{
    if (!grad_out || !argmax || !grad_feat) return FLEX_ERR_NULL;
    if ((in_off == nullptr) != (in_src == nullptr)) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, in_off ? K : 1, C, 1) || Ns <= 0 || Ns > N) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    hipStream_t s = (hipStream_t)stream;
    const int bnc = layout == FLEX_LAYOUT_BNC;
    if (in_off)
        FLEX_HIP(launch_pool_sub_bwd_gather(grad_out, argmax, in_off, in_src, grad_feat, B, N, Ns, C, bnc, s));
    else
        FLEX_HIP(launch_pool_sub_bwd(grad_out, argmax, grad_feat, B, N, Ns, C, bnc, s));
    return FLEX_OK;
}

int flex_inedges_build_sub(const int32_t *nbr, const int32_t *sel, int B, int N, int Ns, int K,
                           int32_t *in_off, int32_t *in_src, void *workspace, size_t workspace_bytes,
                           void *stream)
{
    if (!nbr || !sel || !in_off || !in_src) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, 1, 1) || Ns <= 0 || Ns > N) return FLEX_ERR_SHAPE;
    if (!ws_ok(workspace, workspace_bytes, inedges_ws_bytes((int64_t)B * N, K))) return FLEX_ERR_WORKSPACE;
    FLEX_HIP(launch_inedges_build_sub(nbr, sel, B, N, Ns, K, in_off, in_src, workspace, (hipStream_t)stream));
    return FLEX_OK;
}

int flexconv_bwd_pos(const float *feat, const int32_t *nbr, const float *theta, const float *grad_out,
                     const int32_t *in_off, const int32_t *in_src, float *grad_pos, int B, int N, int K,
                     int Din, int Dout, int layout, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!feat || !nbr || !theta || !grad_out || !grad_pos) return FLEX_ERR_NULL;
    if ((in_off == nullptr) != (in_src == nullptr)) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, Din, Dout)) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    const bool build = in_off == nullptr;
    const PosPlan p = plan_pos(B, N, K, Din, Dout, layout, build);
    if (!ws_ok(workspace, workspace_bytes, p.total)) return FLEX_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    const int bcn = (layout == FLEX_LAYOUT_BCN);
    if (p.blocked) {
        const int n_hi = (Din + 63) / 64, n_ho = (Dout + 63) / 64;
        const size_t blk_bytes = align256(sizeof(float) * (size_t)B * N * 64);
        PrepList prep;
        for (int i = 0; i < n_hi + n_ho; ++i) {
            if (prep.n == PREP_MAX_JOBS) FLEX_HIP(prep.launch(s));
            if (i < n_hi) prep.copy(feat, (float *)(ws + p.featT + i * blk_bytes), B, N, Din, 64, bcn, 0, 64 * i);
            else prep.copy(grad_out, (float *)(ws + p.gT + (i - n_hi) * blk_bytes), B, N, Dout, 64, bcn, 0, 64 * (i - n_hi));
        }
        FLEX_HIP(prep.launch(s));
        if (build) {
            int32_t *off = (int32_t *)(ws + p.in_off), *src = (int32_t *)(ws + p.in_src);
            FLEX_HIP(launch_inedges_build(nbr, B, N, K, off, src, ws + p.inedge_ws, s));
            in_off = off;
            in_src = src;
        }
        void *thC = ws + p.thetaC, *thN = ws + p.thetaN;
        for (int hi = 0; hi < n_hi; ++hi)
            for (int ho = 0; ho < n_ho; ++ho) {
                const float *f_blk = (const float *)(ws + p.featT + hi * blk_bytes);
                const float *g_blk = (const float *)(ws + p.gT + ho * blk_bytes);
                prep.pack_theta_pos(theta, thC, Din, Dout, 64 * hi, 64 * ho, 64, 64, 0);
                prep.pack_theta_pos(theta, thN, Din, Dout, 64 * hi, 64 * ho, 64, 64, 1);
                FLEX_HIP(prep.launch(s));
                FLEX_HIP(launch_grad_pos_term(f_blk, nbr, nullptr, nullptr, thC, g_blk, grad_pos, -1.f,
                                              (hi | ho) != 0, B, N, K, 64, 64, 0, s));
                FLEX_HIP(launch_grad_pos_term(g_blk, nullptr, in_off, in_src, thN, f_blk, grad_pos, 1.f, 1, B, N, K, 64,
                                              64, 1, s));
            }
        return FLEX_OK;
    }
    if (!p.lean) {
        FLEX_HIP(launch_generic_bwd_pos(feat, nbr, theta, grad_out, grad_pos, B, N, K, Din, Dout, !bcn, s));
        return FLEX_OK;
    }
    const float *rows = feat, *g_rows = grad_out;
    PrepList prep;
    if (bcn) {
        prep.copy(feat, (float *)(ws + p.featT), B, N, Din, Din, 1, 0);
        prep.copy(grad_out, (float *)(ws + p.gT), B, N, Dout, Dout, 1, 0);
        rows = (const float *)(ws + p.featT);
        g_rows = (const float *)(ws + p.gT);
    }
    if (build) {
        int32_t *off = (int32_t *)(ws + p.in_off), *src = (int32_t *)(ws + p.in_src);
        FLEX_HIP(launch_inedges_build(nbr, B, N, K, off, src, ws + p.inedge_ws, s));
        in_off = off;
        in_src = src;
    }
    void *thC = ws + p.thetaC, *thN = ws + p.thetaN;
    prep.pack_theta_pos(theta, thC, Din, Dout, 0, 0, pad32(pad4(Din)), pad16(Dout), 0);
    prep.pack_theta_pos(theta, thN, Din, Dout, 0, 0, pad32(pad4(Dout)), pad16(Din), 1);
    FLEX_HIP(prep.launch(s));
    // centre term: -<(sum_k feat[n_k(x)])^T theta_d, grad_out[x]>, then neighbour term added on top
    FLEX_HIP(launch_grad_pos_term(rows, nbr, nullptr, nullptr, thC, g_rows, grad_pos, -1.f, 0, B, N, K, Din, Dout, 0, s));
    FLEX_HIP(launch_grad_pos_term(g_rows, nullptr, in_off, in_src, thN, rows, grad_pos, 1.f, 1, B, N, K, Dout, Din, 1, s));
    return FLEX_OK;
}

int flexupsample_fwd(const float *feat_small, const int32_t *sel, const int32_t *nbr, float *out,
                     int32_t *argmax, int B, int Ns, int Nf, int K, int C, int layout, void *workspace,
                     size_t workspace_bytes, void *stream)
{
    if (!feat_small || !sel || !nbr || !out || !argmax) return FLEX_ERR_NULL;
    if (!sizes_ok(B, Nf, K, C, 1) || Ns <= 0 || Ns > Nf) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    if (!ws_ok(workspace, workspace_bytes, align256(sizeof(int32_t) * (size_t)B * Nf))) return FLEX_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    int32_t *inv = (int32_t *)workspace;
    FLEX_HIP(launch_upsample_inv(sel, inv, B, Ns, Nf, s));
    FLEX_HIP(launch_upsample_fwd(feat_small, inv, nbr, out, argmax, B, Ns, Nf, K, C, layout == FLEX_LAYOUT_BNC, s));
    return FLEX_OK;
}

int flexupsample_bwd(const float *grad_out, const int32_t *argmax, const int32_t *sel,
                     const int32_t *in_off, const int32_t *in_src, float *grad_small, int B, int Ns,
                     int Nf, int K, int C, int layout, void *stream)
{
    if (!grad_out || !argmax || !sel || !in_off || !in_src || !grad_small) return FLEX_ERR_NULL;
    if (!sizes_ok(B, Nf, K, C, 1) || Ns <= 0 || Ns > Nf) return FLEX_ERR_SHAPE;
    if (layout != FLEX_LAYOUT_BCN && layout != FLEX_LAYOUT_BNC) return FLEX_ERR_SHAPE;
    FLEX_HIP(launch_upsample_bwd(grad_out, argmax, sel, in_off, in_src, grad_small, B, Ns, Nf, C,
                                 layout == FLEX_LAYOUT_BNC, (hipStream_t)stream));
    return FLEX_OK;
}

int flex_validate_selection(const int32_t *sel, int B, int Ns, int Nf, int32_t *bad_count_dev,
                            void *workspace, size_t workspace_bytes, void *stream)
{
    if (!sel || !bad_count_dev) return FLEX_ERR_NULL;
    if (!sizes_ok(B, Nf, 1, 1, 1) || Ns <= 0 || Ns > Nf) return FLEX_ERR_SHAPE;
    if (!ws_ok(workspace, workspace_bytes, align256(sizeof(int32_t) * (size_t)B * Nf))) return FLEX_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    int32_t *inv = (int32_t *)workspace;
    FLEX_HIP(launch_upsample_inv(sel, inv, B, Ns, Nf, s));
    FLEX_HIP(launch_upsample_check_sel(sel, inv, B, Ns, Nf, bad_count_dev, s));
    return FLEX_OK;
}

int flex_validate_neighbors(const int32_t *nbr, int B, int N, int K, int32_t *bad_count_dev,
                            void *stream)
{
    if (!nbr || !bad_count_dev) return FLEX_ERR_NULL;
    if (!sizes_ok(B, N, K, 1, 1)) return FLEX_ERR_SHAPE;
    FLEX_HIP(launch_count_bad(nbr, (int64_t)B * K * N, N, bad_count_dev, (hipStream_t)stream));
    return FLEX_OK;
}

}  // extern "C"
