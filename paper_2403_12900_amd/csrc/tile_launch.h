// Launch of the tiled projection (k_tile_gemm) of a prefill chunk.  The
// kernel's instantiations are compiled in translation units of their own
// (tile_*.hip).
#pragma once

#include "panel_launch.h"
#include "prefill_kernels.h"

namespace sprk {

// Enqueues out = W X^T for the NT weight tiles of W over Rp padded rows.  LP:
// parts per K-block of the activation record X (P::parts are used).
template <class P, int LP, class Epi>
void launch_tile_gemm(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, int Rp, const Epi& epi,
                      const SplitRoom& room);

}  // namespace sprk
