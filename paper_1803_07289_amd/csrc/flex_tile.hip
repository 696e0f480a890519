// Instantiations of the 64-point tile kernels (flex_tile.hpp), compiled once per list form with -DFLEX_TILE_CSR=.
#include "flex_tile.hpp"

#if !defined(FLEX_TILE_CSR)
#error "build with -DFLEX_TILE_CSR"
#endif

#define FLEX_TILE_CAT(a, b) a##b
#define FLEX_TILE_NAME(a, b) FLEX_TILE_CAT(a, b)

namespace flex {

template <int WM, int NSW>
static hipError_t launch(const TileArgs &a, int grid, hipStream_t s)
{
    constexpr bool CSR = FLEX_TILE_CSR != 0;
    if (a.n_in == 1)
        hipLaunchKernelGGL((tile_conv_kernel<WM, NSW, CSR, false>), dim3(grid), dim3(1024), 0, s, a);
    else
        hipLaunchKernelGGL((tile_conv_kernel<WM, NSW, CSR, true>), dim3(grid), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t FLEX_TILE_NAME(launch_tile_, FLEX_TILE_CSR)(const TileArgs &a, int outw, int grid, hipStream_t s)
{
    switch (outw) {
    case 64: return launch<2, 1>(a, grid, s);
    case 128: return launch<1, 1>(a, grid, s);
    case 256: return launch<1, 2>(a, grid, s);
    default: return hipErrorInvalidValue;
    }
}

#if FLEX_TILE_CSR == 0
hipError_t launch_tile_grad_theta(const TileArgs &a, const float *g_rows, int n_hi, int n_ho, int oc, bool f32, float *partials, hipStream_t s)
{
    const dim3 grid(n_hi * n_ho * a.chunks), block(1024);
    if (oc == 128) hipLaunchKernelGGL(tile_grad_theta128_kernel, grid, block, 0, s, a, g_rows, n_ho, partials);
    else if (f32) {
        // of a block's four by two parts of 16 and of twice 16 channels, those that have any.  us, all waves contracting and these alone: 7 of 8
        // parts: 100 -> 50, 300k points 217 and 222; 6 of 16: 96 -> 9, 20k 32.9 and 29.8; 3 of 16 and 4: 16 -> 80, 20k 32.8 and 22.1, 9 -> 100, 3k 16.7
        // and 12.6, 3 -> 100, 300k 240 and 171, 15 -> 79, 8 x 78k, K = 10, 506 and 361
        const int parts = (a.w_in + 15) / 16 * (2 * n_ho - (a.w_out - 64 * (n_ho - 1) <= 16));
        if (4 * parts <= 3 * 8 * n_hi * n_ho) hipLaunchKernelGGL((tile_grad_theta_kernel<true, true>), grid, block, 0, s, a, g_rows, n_ho, partials);
        else hipLaunchKernelGGL((tile_grad_theta_kernel<true, false>), grid, block, 0, s, a, g_rows, n_ho, partials);
    } else hipLaunchKernelGGL((tile_grad_theta_kernel<false, false>), grid, block, 0, s, a, g_rows, n_ho, partials);
    return hipGetLastError();
}
#endif

}  // namespace flex
