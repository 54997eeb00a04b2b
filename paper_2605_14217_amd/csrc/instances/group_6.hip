// written by gen_instances.py: do not edit by hand
#include "../expand_kernel.hpp"
#include "../f32_kernel.hpp"
#include "../mfma_kernel.hpp"
#include "../mfma_wide_kernel.hpp"
#include "../small_kernel.hpp"
#include "../valu_kernel.hpp"

template __global__ void preft::f32_tile_kernel<1, true, false, false, true>(preft::ApplyArgs);
template __global__ void preft::f32_tile_kernel<2, false, true, true, true>(preft::ApplyArgs);
template __global__ void preft::f32_tile_kernel<4, true, false, false, true>(preft::ApplyArgs);
template __global__ void preft::f32_tile_kernel<8, true, true, false, true>(preft::ApplyArgs);
template __global__ void preft::f32_tile_layers_kernel<1, false>(preft::ApplyArgs);
template __global__ void preft::f32_tile_layers_kernel<8, true>(preft::ApplyArgs);
template __global__ void preft::mfma_expand_kernel<1, 2, true, (preft::YHint)1>(preft::ApplyArgs, int);
template __global__ void preft::mfma_tile_kernel<1, 1, 4, 0, false, 3, false, 2, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_kernel<1, 1, 8, 0, false, 1, false, 0, true, true>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_kernel<1, 1, 8, 0, false, 2, false, 2, true, true>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_kernel<1, 1, 8, 0, true, 1, false, 4, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_kernel<2, 1, 4, 0, false, 1, false, 0, false, false>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_kernel<2, 2, 4, 0, false, 1, false, 0, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_kernel<4, 1, 4, 0, false, 1, false, 0, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_kernel<4, 2, 4, 0, true, 1, false, 0, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_layers_kernel<1, 1, 8, 4, false, 0>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_layers_kernel<2, 2, 4, 0, false, 0>(preft::ApplyArgs);
template __global__ void preft::mfma_tile_layers_kernel<8, 1, 4, 0, false, 1>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<1, 2, 4, 1, false, 1, false, false, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<2, 1, 4, 1, false, 2, false, false, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<2, 1, 4, 1, false, 3, true, false, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<2, 1, 4, 2, false, 3, false, false, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<4, 1, 4, 1, false, 1, false, true, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<4, 1, 4, 1, false, 3, false, false, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<4, 1, 4, 1, true, 1, true, true, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<4, 1, 8, 1, false, 2, true, true, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<8, 1, 4, 1, false, 1, true, false, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_kernel<8, 1, 8, 1, true, 1, false, false, false, true>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_layers_kernel<1, 1, 4, 2, false>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_layers_kernel<2, 2, 4, 1, false>(preft::ApplyArgs);
template __global__ void preft::mfma_wide_layers_kernel<8, 1, 8, 1, false>(preft::ApplyArgs);
template __global__ void preft::panel_expand_kernel<4, 4, 2, false, false, true>(preft::ApplyArgs, int);
template __global__ void preft::panel_expand_kernel<8, 4, 1, false, true, false>(preft::ApplyArgs, int);
template __global__ void preft::small_shrink_kernel<3, false, 0, 4>(preft::ApplyArgs, int);
template __global__ void preft::small_tile_kernel<1, false, false, false, 8, false, 3, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<1, false, false, false, 8, true, 4, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<1, false, false, true, 8, false, 8, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<1, false, true, false, 8, false, 0, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<1, false, true, true, 8, true, 8, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<1, true, false, true, 8, true, 0, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<1, true, true, true, 8, false, 8, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<2, false, false, true, 8, false, 24, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<2, false, false, true, 8, true, 28, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<2, true, false, true, 8, true, 0, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<4, false, false, true, 4, true, 0, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<4, true, false, true, 8, false, 0, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<8, false, false, true, 8, true, 0, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_kernel<8, true, true, true, 8, false, 0, true>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_layers_kernel<1, false, false, 8>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_layers_kernel<1, true, false, 0>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_layers_kernel<2, false, false, 28>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_layers_kernel<4, false, false, 0>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::small_tile_layers_kernel<8, true, true, 0>(preft::ApplyArgs, preft::SmallLaunch);
template __global__ void preft::thin_expand_kernel<2, 2>(preft::ApplyArgs, int);
template __global__ void preft::valu_tile_kernel<1, 4, 1, true, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<1, 4, 4, false, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<2, 2, 4, true, 1, 8, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<2, 4, 4, false, 2, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<3, 4, 1, true, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<3, 4, 4, false, 3, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<4, 4, 2, true, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<5, 2, 4, false, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<6, 2, 4, false, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<7, 2, 4, false, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_kernel<8, 2, 4, false, 1, 0, false>(preft::ApplyArgs);
template __global__ void preft::valu_tile_layers_kernel<2, 4, 1, 0>(preft::ApplyArgs);
template __global__ void preft::valu_tile_layers_kernel<4, 2, 4, 8>(preft::ApplyArgs);
template __global__ void preft::valu_tile_layers_kernel<5, 2, 4, 8>(preft::ApplyArgs);
template __global__ void preft::valu_tile_layers_kernel<7, 2, 4, 0>(preft::ApplyArgs);
