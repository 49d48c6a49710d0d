// Instantiations of the tiled projection: O and down projections.
#include "tile_launch_impl.h"

using namespace sprk;

template void sprk::launch_tile_gemm<BF16, 2, EpiResidRows<BF16>>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiResidRows<BF16>&, const SplitRoom&);
template void sprk::launch_tile_gemm<BF16, 2, EpiResidRows<BF16x3>>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiResidRows<BF16x3>&, const SplitRoom&);
template void sprk::launch_tile_gemm<F32, 1, EpiResidRows<F32>>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiResidRows<F32>&, const SplitRoom&);
