// Instantiations of the panel launch: QKV of prefill chunks (given row scales).
#include "panel_launch_impl.h"

using namespace sprk;
using EpiQKVbb = EpiQKV<BF16, BF16, true>;
using EpiQKVbf = EpiQKV<BF16, F32, true>;

template void sprk::launch_panel_gemm<BF16x3, EpiQKVbb>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiQKVbb&, const SplitRoom&, const PanelPick&);
template void sprk::launch_panel_gemm<BF16x3, EpiQKVbf>(hipStream_t, int, const uint4*, const uint4*, int,
                                            const EpiQKVbf&, const SplitRoom&, const PanelPick&);
