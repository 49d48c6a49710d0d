// Instantiations of the tiled projection: gate/up.
#include "tile_launch_impl.h"

using namespace sprk;

template void sprk::launch_tile_gemm<BF16, 2, EpiSwiGLURows<BF16>>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiSwiGLURows<BF16>&, const SplitRoom&);
template void sprk::launch_tile_gemm<F32, 1, EpiSwiGLURows<F32>>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiSwiGLURows<F32>&, const SplitRoom&);
