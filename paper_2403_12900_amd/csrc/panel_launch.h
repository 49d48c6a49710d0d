// Launch of the panel kernel (panel_kernels.h).  The kernel's instantiations
// are compiled in translation units of their own (panel_*.hip).
#pragma once

#include <type_traits>

#include "launch_rule.h"
#include "panel_kernels.h"

namespace sprk {

// Activation format of the QKV projection's input: all 24 bits of the fp32
// residual for bf16 models (three parts), the plain format otherwise.
template <class P>
using QKVIn = std::conditional_t<std::is_same_v<P, BF16>, BF16x3, P>;

// Room for split-K partials and arrival counters (see SplitK): the regions of
// the attention split partials and counters, which every launch that uses them
// leaves zero.  The rules split no further than it holds.
struct SplitRoom {
  float* part = nullptr;  // null: no split-K
  int32_t* cnt = nullptr;
  size_t part_floats = 0;
  int n_cnt = 0;
  SplitCap cap() const { return part == nullptr ? SplitCap{} : SplitCap{part_floats, n_cnt}; }
};

// Enqueues the projection of epi.n_rows rows (at most kRows; the activation
// record has row_tiles(n_rows) row tiles) in the shape that gemm_pick chose.
// P: activation format of the input.
template <class P, class Epi>
void launch_panel_gemm(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, const Epi& epi,
                       const SplitRoom& room, const PanelPick& pick);

}  // namespace sprk
