// Instantiations of the panel launch: gate/up and LM head.
#include "panel_launch_impl.h"

using namespace sprk;
using EpiSwiGLURs = EpiSwiGLU<BF16, true>;

template void sprk::launch_panel_gemm<BF16, EpiSwiGLU<BF16>>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiSwiGLU<BF16>&, const SplitRoom&, const PanelPick&);
template void sprk::launch_panel_gemm<BF16, EpiSwiGLURs>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiSwiGLURs&, const SplitRoom&, const PanelPick&);
template void sprk::launch_panel_gemm<F32, EpiSwiGLU<F32>>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiSwiGLU<F32>&, const SplitRoom&, const PanelPick&);
template void sprk::launch_panel_gemm<BF16, EpiLogits<BF16>>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiLogits<BF16>&, const SplitRoom&, const PanelPick&);
template void sprk::launch_panel_gemm<F32, EpiLogits<F32>>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiLogits<F32>&, const SplitRoom&, const PanelPick&);
