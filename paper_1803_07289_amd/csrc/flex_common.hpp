// Shared host/device helpers for libflexconv (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace flex {

constexpr int cdiv_c(int a, int b) { return (a + b - 1) / b; }
constexpr int rup_c(int a, int b) { return cdiv_c(a, b) * b; }
constexpr int npow2_c(int x) { int p = 1; while (p < x) p <<= 1; return p; }

static inline int64_t cdiv64(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Number of compute units of the current device (cached per process).
int device_cu_count();

// Persistent-grid size: a multiple of 8 (one share per XCD), at most
// `wg_per_cu` workgroups per CU, at most one workgroup per tile.
int persistent_grid(int64_t total_tiles, int wg_per_cu);

typedef float v4f __attribute__((ext_vector_type(4)));

// The channel-major kernels' workgroups take 64 points and 16 channels at a time: into how many parts their channels are dealt, so that
// a cloud of few tiles fills the device (full: the workgroups that do).  A part sorts its tile's neighbours out for itself.
// us, in one part and in as many, upsampling forward, 26k points x 128, K = 12, 35 and 27, 10k x 64, K = 8, 14.2 and 11.6; pooling to a quarter, 200k x 64,
// K = 4, 26.8 and 25.2.
static inline unsigned channel_parts(int64_t tiles, int C, int64_t full)
{
    const int64_t most = (C + 15) / 16, wanted = full / (tiles > 0 ? tiles : 1);
    return (unsigned)(wanted < 1 ? 1 : wanted < most ? wanted : most);
}

// Rows of C channels, four to a lane.  ODD: C (at least 4) is no multiple of four: rows begin at any element, and the last lane takes the
// row's last four channels, of which it stores those that the lane before has not.
template <class T, bool ODD>
struct RowChunk {
    typedef T V __attribute__((ext_vector_type(4), aligned(ODD ? 4 : 16)));
    typedef T V16 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ int first(int c4, int C) { return ODD ? min(4 * c4, C - 4) : 4 * c4; }
    // at: the chunk's first channel in the row
    static __device__ __forceinline__ V16 load(const T *at) { return *reinterpret_cast<const V *>(at); }
    // STREAM: outputs that are not read again by their kernel should not displace gathered rows in L2
    template <bool STREAM = true>
    static __device__ __forceinline__ void store(T *at, int c4, int C, const V16 &v)
    {
        if (!ODD || 4 * c4 + 4 <= C) {
            if (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<V *>(at));
            else *reinterpret_cast<V *>(at) = v;
            return;
        }
#pragma unroll
        for (int i = 1; i < 4; ++i)
            if (i >= 4 - C % 4) at[i] = v[i];
    }
};
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

// ---- launchers implemented in the .hip translation units -------------------

// thetaP[(j*RP + r)*CP + c], j in 0..3 (x,y,z,bias), zero padded.
//   transpose == 0: r = input channel, c = output channel  (forward / grad_theta)
//   transpose == 1: r = output channel, c = input channel  (grad_feat)
hipError_t launch_pack_theta(const float *theta, const float *bias, float *thetaP,
                             int Din, int Dout, int RP, int CP, int transpose, hipStream_t s);

// The steps in front of a call's main kernels as jobs of one launch (flex_prep.hip): collect, then launch once.
// None of a list's jobs may read what another one writes.
constexpr int PACK_MAX_KD = 512, PREP_MAX_JOBS = 6, PREP_JOB_BYTES = 80;
struct PrepList {
    int n = 0;
    bool bad = false;
    alignas(8) char storage[PREP_MAX_JOBS * PREP_JOB_BYTES];
    // Split-half (f16 hi/lo) fragment form of the parameters for the wave-specialised kernels (layout: flex_prep.hip).
    // RP = rows per component (4 * RP <= PACK_MAX_KD), CP = columns (a multiple of 16) of a block; block (i, j) of
    // n_i x n_j (rows RP * i.., columns CP * j..) lands theta_f16_bytes(RP, CP) * (j * n_i + i) bytes into thetaF.
    // transpose == 0: rows = input channels, columns = output channels; 1: the other way round.  Din, Dout: the real
    // tensor's widths; what a block reaches beyond them is zero.
    void pack_theta(const float *theta, const float *bias, void *thetaF, int Din, int Dout, int RP, int CP, int n_i,
                    int n_j, int transpose);
    // The location gradient's form of theta's block of input channels ci0.. and output channels co0.. (KDP deep, CP
    // columns; zero outside theta).
    void pack_theta_pos(const float *theta, void *thetaF, int Din, int Dout, int ci0, int co0, int KDP, int CP,
                        int transpose);
    // order[b*N + p] = point at position p: the cloud's points sorted by in-edge list length inside windows of nearby
    // points (the walking order of the gather kernels over in-edge lists); inedges_order_bytes(B * N)
    void order(const int32_t *in_off, int B, int N, int32_t *order);
    // dst[b, n, c] = src[b, n, c_off + c] where that channel exists, else 0 (c < Cd); *_bcn: that tensor is channel-major
    void copy(const float *src, float *dst, int B, int N, int Cs, int Cd, int src_bcn, int dst_bcn, int c_off = 0);
    // pos4[b*N + n] = (x, y, z, 0)
    void pack_pos(const float *pos, float *pos4, int B, int N);
    // the records of rows of W <= 16 channels (flex_narrow.hip): rec [B*N, 16], rec4 [B*N, 4] (only with four channels a quad);
    // feat as the caller has it, *_bcn: channel-major; nbr [B,K,N] or null: read on the way (flex_prep.hip)
    void records(const float *pos, const float *feat, float *rec, float *rec4, int B, int N, int W, int bcn, const int32_t *nbr, int K);
    void clear(void *dst, int words);
    hipError_t launch(hipStream_t s);
};
size_t theta_f16_exp_offset(int RP, int CP);
size_t theta_f16_rscale_offset(int RP, int CP);
size_t theta_f16_bytes(int RP, int CP);

// Control words of the one-pass backward kernel (bwd_fused_lean_kernel) in the workspace: the flag (0: its parameter
// gradients stand; FUSED_OVERFLOW: a feature row overflowed f16 while the kernel ran; FUSED_UNRESOLVED: the check after
// the reduction found the result too small for the f16 halves to resolve; either way the stand-alone kernel
// recomputes them), then one record per workgroup: its last running exponent, its number of terms, its DO channel
// exponents.
constexpr int FUSED_FLAG_INTS = 64, FUSED_RECORD_INTS = 128, FUSED_MAX_WG = 1024;
constexpr int FUSED_OVERFLOW = 1, FUSED_UNRESOLVED = 2;
constexpr size_t fused_control_bytes() { return sizeof(int) * (size_t)(FUSED_FLAG_INTS + FUSED_RECORD_INTS * FUSED_MAX_WG); }
// what reduce_partials_fused_kernel leaves in the records' spare words, as doubles
constexpr int FUSED_Q_INT = 96;      // record c: Q_c
constexpr int FUSED_ROW_INT = 98;    // record kd: the sum of squares of the result's row kd
hipError_t launch_reduce_partials_fused(const float *partials, int n_wg, int *control, int Din, int Dout,
                                        float *grad_theta, float *grad_bias, hipStream_t s);
hipError_t launch_reduce_partials_if(const int *flag, const float *partials, int n_wg, int DIP, int DOP, int Din,
                                     int Dout, float *grad_theta, float *grad_bias, hipStream_t s);

// Location gradient (flex_ws.hpp grad_pos_kernel): Theta_d fragments and one term of the gradient.
// launch_grad_pos_term returns hipErrorNotSupported when (DI, DO, N, K) has no lean kernel.
size_t theta_pos_exp_offset(int KDP, int CP);
size_t theta_pos_bytes(int KDP, int CP);
hipError_t launch_grad_pos_term(const float *rows, const int32_t *nbr, const int32_t *off, const int32_t *src,
                                const void *thetaF, const float *dot_rows, float *grad_pos, float sign,
                                int accumulate, int B, int N, int K, int DI, int DO, int csr, hipStream_t s);
bool grad_pos_supported(int DI, int DO, int N, int K);
// direct-form fallback for any shape (fp32 atomics)
hipError_t launch_generic_bwd_pos(const float *feat, const int32_t *nbr, const float *theta,
                                  const float *grad_out, float *grad_pos, int B, int N, int K, int Din,
                                  int Dout, int bnc, hipStream_t s);

// A PrepList of one copy.
hipError_t launch_copy_rows(const float *src, float *dst, int B, int N, int Cs, int Cd, int src_bcn, int dst_bcn,
                            hipStream_t s, int c_off = 0);

// Point locations as the lean kernels read them: the tensor [B,3,N] itself, or packed as (x, y, z, 0) records
// (PrepList::pack_pos; the tile kernels read the tensor).  A component's byte offset inside a cloud is (point << shift) + component * col.
struct PosRef {
    const float *p;
    unsigned col;            // bytes from component to component
    int shift;               // log2 of the bytes from point to point
    int64_t cloud;           // bytes from cloud to cloud
};
inline PosRef pos_planar(const float *pos, int N) { return PosRef{pos, 4u * (unsigned)N, 2, 12 * (int64_t)N}; }
inline PosRef pos_packed(const float *pos4, int N) { return PosRef{pos4, 4u, 4, 16 * (int64_t)N}; }

// channels of a row of w of at most 16 in each quad of its record
constexpr int narrow_record_channels(int w) { return (w + 3) / 4; }
// sixteens of points that a call from such records has at most (32-bit wave numbers)
static constexpr int64_t NARROW_RECORD_WAVES_MAX = 1 << 27;

// Tiled matrix-core path.  `rows` is point-major [B*N, DI].  Returns
// hipErrorNotSupported when (DI,DO) has no instantiation.
//   csr == 0: neighbours from nbr [B,K,N], dp = pos[nbr]-pos[centre]
//   csr == 1: in-edge lists (off,src), dp = pos[centre]-pos[src]
//   theta_fmt: what thetaP holds, as answered by gather_contract_theta_format for the same
//   (DI, DO, N, K, csr): 0 = fp32 ThetaP (launch_pack_theta), 1 = split-half fragments
//   (PrepList::pack_theta).
//   order (csr == 1 only): the walking order of these lists (PrepList::order)
hipError_t launch_gather_contract(const float *rows, const float *pos, const PosRef &pr, const int32_t *nbr,
                                  const int32_t *off, const int32_t *src, const int32_t *order,
                                  const void *thetaP, int theta_fmt, float *out, int B, int N, int K, int DI,
                                  int DO, int csr, int out_bcn, hipStream_t s);
bool gather_contract_supported(int DI, int DO);
int gather_contract_theta_format(int DI, int DO, int N, int K, int csr);
// true when the environment asks for the fp32 matrix op in the wave-specialised kernels
// (FLEX_CONTRACT=f32; read once).  For A/B measurements; both forms meet the same tolerance.
bool contract_in_fp32();
// Producer choice for the fixed-K forward (FLEX_PRODUCER, read once; for A/B measurements):
// 0 "staged" = LDS-staged producer, 1 "lean" = lean producers, one per consumer wave,
// 2 (default) = lean producers, three per consumer wave where the shape allows.
int lean_producer_mode();

// The 64-point tile kernels (flex_tile.hpp): layers of any width.
struct TileArgs {
    const float *rows, *pos;
    const int32_t *nbr, *off, *src, *order;
    const char *theta;           // packed blocks [output block][input block]
    const float *bias;           // null; or theta is the tensor [3, w_in, w_out], this one [w_in, w_out] (narrow_conv_kernel)
    float *out;
    int64_t out_c, out_l, out_b; // output strides: channel, point, cloud
    int rs, w_in, w_out;         // row stride (floats), real widths
    int blk_bytes, exp_off, rs_off;
    int N, K, tpc, total;        // tiles per cloud, tiles
    int n_in, chunks;            // input blocks; workgroups per output block
};

// Workspace of the per-workgroup partial sums of grad_theta / grad_bias ([n_wg, KD, DOP] floats).
size_t grad_theta_partial_bytes(int64_t B, int64_t N, int Din, int Dout);

// Generic (any Din/Dout) direct-form kernels; strides select the layout.
hipError_t launch_generic_fwd(const float *feat, const float *pos, const int32_t *nbr,
                              const float *theta, const float *bias, float *out,
                              int B, int N, int K, int Din, int Dout, int bnc, hipStream_t s);
hipError_t launch_generic_bwd(const float *feat, const float *pos, const int32_t *nbr,
                              const float *theta, const float *bias, const float *grad_out,
                              float *grad_feat, float *grad_theta, float *grad_bias,
                              int B, int N, int K, int Din, int Dout, int bnc, hipStream_t s);

// In-edge lists.
hipError_t launch_inedges_build(const int32_t *nbr, int B, int N, int K, int32_t *in_off,
                                int32_t *in_src, void *ws, hipStream_t s);
hipError_t launch_inedges_build_sub(const int32_t *nbr, const int32_t *sel, int B, int N, int Ns, int K,
                                    int32_t *in_off, int32_t *in_src, void *ws, hipStream_t s);
size_t inedges_ws_bytes(int64_t BN, int K);
size_t inedges_order_bytes(int64_t BN);
size_t knn_ws_bytes(int B, int N, int K);
bool knn_k_supported(int K);
hipError_t launch_knn(const float *pos, int32_t *nbr, int B, int N, int K, void *ws, hipStream_t s);

// Pooling.
hipError_t launch_pool_fwd(const float *feat, const int32_t *nbr, float *out, int32_t *argmax,
                           int B, int N, int K, int C, int bnc, hipStream_t s);
hipError_t launch_pool_bwd(const float *grad_out, const int32_t *argmax, float *grad_feat,
                           int B, int N, int C, int bnc, hipStream_t s);
hipError_t launch_pool_bwd_gather(const float *grad_out, const int32_t *argmax, const int32_t *in_off,
                                  const int32_t *in_src, float *grad_feat, int B, int N, int C, int bnc,
                                  hipStream_t s);

// Flex-upsampling: inverse selection map (inv[b*Nf + sel[b,j]] = j, -1 elsewhere), pooling through it,
// routing back over the larger layer's in-edge lists, and a check of the selection (out of range / repeated).
hipError_t launch_pool_sub_fwd(const float *feat, const int32_t *nbr, const int32_t *sel, float *out,
                               int32_t *argmax, int B, int N, int Ns, int K, int C, int bnc, hipStream_t s);
hipError_t launch_pool_sub_bwd(const float *grad_out, const int32_t *argmax, float *grad_feat, int B,
                               int N, int L, int C, int bnc, hipStream_t s);
// static gather plan of the pooling backward pass (point-major, C = 64, 128 or 256)
size_t pool_plan_bytes(int B, int N, int K);
hipError_t launch_pool_plan_build(const int32_t *in_off, const int32_t *in_src, void *plan, int B, int N, int K,
                                  hipStream_t s);
hipError_t launch_pool_bwd_planned(const float *grad_out, const int32_t *argmax, const int32_t *in_off,
                                   const int32_t *in_src, void *plan, float *grad_feat, int B, int N, int K, int C,
                                   hipStream_t s);
hipError_t launch_pool_fwd_plan_build(const int32_t *nbr, void *plan, int B, int N, int K, hipStream_t s);
hipError_t launch_pool_fwd_planned(const float *feat, const int32_t *nbr, void *plan, float *out, int32_t *argmax,
                                   int B, int N, int K, int C, hipStream_t s);
hipError_t launch_pool_sub_bwd_gather(const float *grad_out, const int32_t *argmax, const int32_t *in_off,
                                      const int32_t *in_src, float *grad_feat, int B, int N, int L, int C,
                                      int bnc, hipStream_t s);
hipError_t launch_upsample_inv(const int32_t *sel, int32_t *inv, int B, int Ns, int Nf, hipStream_t s);
hipError_t launch_upsample_fwd(const float *feat_small, const int32_t *inv, const int32_t *nbr, float *out,
                               int32_t *argmax, int B, int Ns, int Nf, int K, int C, int bnc, hipStream_t s);
hipError_t launch_upsample_bwd(const float *grad_out, const int32_t *argmax, const int32_t *sel,
                               const int32_t *in_off, const int32_t *in_src, float *grad_small, int B, int Ns,
                               int Nf, int C, int bnc, hipStream_t s);
hipError_t launch_upsample_bwd_bcn(const float *grad_out, const int32_t *argmax, const int32_t *sel, const int32_t *in_off,
                                   const int32_t *in_src, float *grad_small, int B, int Ns, int Nf, int C, hipStream_t s);
hipError_t launch_upsample_check_sel(const int32_t *sel, const int32_t *inv, int B, int Ns, int Nf, int32_t *bad,
                                     hipStream_t s);

hipError_t launch_count_bad(const int32_t *nbr, int64_t count, int N, int32_t *bad, hipStream_t s);
hipError_t launch_fill_zero(void *ptr, size_t bytes, hipStream_t s);
size_t idiss_ws_bytes(int B, int N);
size_t distinct_ws_bytes(int B, int Ns);
hipError_t launch_selection_make_distinct(int32_t *sel, int B, int N, int Ns, void *ws, hipStream_t s);
hipError_t launch_idiss_phi(const float *pos, const int32_t *nbr, float *phi, float *pos4, int B, int N, int K, hipStream_t s);
hipError_t launch_idiss_sample(const float *phi, const uint32_t *u, int32_t *sel, int B, int N, int Ns, void *ws,
                               hipStream_t s);
hipError_t launch_compose_1x1(const float *W, const float *theta, const float *bias, float *theta_c, float *bias_c,
                              int Din0, int Dmid, int Dout, hipStream_t s);
hipError_t launch_compose_1x1_bwd(const float *W, const float *theta, const float *bias, const float *gtheta_c,
                                  const float *gbias_c, float *gW, float *gtheta, float *gbias, int Din0, int Dmid,
                                  int Dout, hipStream_t s);

}  // namespace flex
