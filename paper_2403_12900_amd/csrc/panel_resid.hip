// Instantiations of the panel launch: O and down projections.
#include "panel_launch_impl.h"

using namespace sprk;

template void sprk::launch_panel_gemm<BF16, EpiResid<BF16>>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiResid<BF16>&, const SplitRoom&, const PanelPick&);
template void sprk::launch_panel_gemm<BF16, EpiResid<BF16x3>>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiResid<BF16x3>&, const SplitRoom&, const PanelPick&);
template void sprk::launch_panel_gemm<F32, EpiResid<F32>>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiResid<F32>&, const SplitRoom&, const PanelPick&);
