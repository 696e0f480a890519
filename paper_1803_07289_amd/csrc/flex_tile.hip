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
    else if (f32) hipLaunchKernelGGL(tile_grad_theta_kernel<true>, grid, block, 0, s, a, g_rows, n_ho, partials);
    else hipLaunchKernelGGL(tile_grad_theta_kernel<false>, grid, block, 0, s, a, g_rows, n_ho, partials);
    return hipGetLastError();
}
#endif

}  // namespace flex
