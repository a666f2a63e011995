// bf16 storage family: the many-rows GEMM whose wave groups take the k-steps of a slot in turn (kernel in gemm_tile.h, plans and
// the other tiles in bf16_gemm_tile.hip).
//
// 128 x 128 of several row groups: four waves of 64 x 64 twice, one k-step of a slot each.  Of a k-step eight waves of 32 x 64 read
// 24 KB of LDS for 16 multiplications, these 16 KB, and from three row groups on the reads are the bound: down of 1024 rows (4096 x
// 11008) 124.8 -> 116.4 us, O 60.6 -> 58.6; 480 rows of 6656 x 6656 84.8 -> 76.4.  With one or two row groups the weights' way from HBM is
// the bound, and a row group of 96 rows multiplies a whole row block for nothing (LM head 53 -> 66 us); takes_halves() in
// bf16_gemm_tile.hip has the measurements and the rule.  256 x 128 and 128 x 192 split the same way gain nothing; four waves of 64 x 64
// alone are slower than eight of 32 x 64 (102 us), one wave to a SIMD hides nothing.
#include <hip/hip_ext.h>

#include "gemm_epilogues.h"
#include "gemm_tile.h"
#include "internal.h"

namespace hydra {

typedef TileShape<2, 2, 2, 2, 8, 2> Tile128x128Halves;

template <class Epi>
void launch_tile_halves(dim3 grid, hipStream_t s, const GemmGeom &g, const Epi &epi, hipEvent_t e0, hipEvent_t e1) {
    typedef Tile128x128Halves S;
    if (e0) hipExtLaunchKernelGGL((gemm_tile_kernel<S, Epi>), grid, dim3(S::WAVES * 64), S::LDS, s, e0, e1, 0, GEMM_GEOM_ARGS(g), epi);
    else    hipLaunchKernelGGL((gemm_tile_kernel<S, Epi>), grid, dim3(S::WAVES * 64), S::LDS, s, GEMM_GEOM_ARGS(g), epi);
}
template void launch_tile_halves<EpiPlain>(dim3, hipStream_t, const GemmGeom &, const EpiPlain &, hipEvent_t, hipEvent_t);
template void launch_tile_halves<EpiResidStaged>(dim3, hipStream_t, const GemmGeom &, const EpiResidStaged &, hipEvent_t, hipEvent_t);
template void launch_tile_halves<EpiSilu>(dim3, hipStream_t, const GemmGeom &, const EpiSilu &, hipEvent_t, hipEvent_t);

hipError_t tile_halves_attr() {
    hipError_t e = hipFuncSetAttribute((const void *)gemm_tile_kernel<Tile128x128Halves, EpiPlain>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)gemm_tile_kernel<Tile128x128Halves, EpiResidStaged>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)gemm_tile_kernel<Tile128x128Halves, EpiSilu>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    return e;
}

}  // namespace hydra
