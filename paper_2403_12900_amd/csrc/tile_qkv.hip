// Instantiations of the tiled projection: QKV.
#include "tile_launch_impl.h"

using namespace sprk;
using EpiBB = EpiQKVRows<BF16, BF16>;
using EpiBF = EpiQKVRows<BF16, F32>;
using EpiFF = EpiQKVRows<F32, F32>;

template void sprk::launch_tile_gemm<BF16, 3, EpiBB>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiBB&, const SplitRoom&);
template void sprk::launch_tile_gemm<BF16x3, 3, EpiBB>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiBB&, const SplitRoom&);
template void sprk::launch_tile_gemm<BF16, 3, EpiBF>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiBF&, const SplitRoom&);
template void sprk::launch_tile_gemm<BF16x3, 3, EpiBF>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiBF&, const SplitRoom&);
template void sprk::launch_tile_gemm<F32, 1, EpiFF>(hipStream_t, int, const uint4*, const uint4*, int, int,
                                              const EpiFF&, const SplitRoom&);
