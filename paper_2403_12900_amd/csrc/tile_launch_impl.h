// Launch of a picked shape of the tiled projection (see tile_launch.h).
#pragma once

#include <iterator>
#include <type_traits>
#include <utility>

#include "tile_launch.h"

namespace sprk {

template <class P, int LP, size_t I, class Epi>
void launch_tile_shape(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, int Rp, const Epi& epi,
                       const SplitRoom& room, int S) {
  constexpr TileShape s = kTileShapes[I];
  const dim3 grid(rule_div(NT, s.tn), rule_div(Rp / 16, s.tm), S);
  const TileSplit ts{room.part, room.cnt};
  if (S == 1) {
    k_tile_gemm<P, s.tn, s.tm, s.nst, false, Epi, LP><<<grid, kTileWaves * 64, 0, st>>>(w, x, NT, KB, Rp, ts, epi);
  } else {
    k_tile_gemm<P, s.tn, s.tm, s.nst, true, Epi, LP><<<grid, kTileWaves * 64, 0, st>>>(w, x, NT, KB, Rp, ts, epi);
  }
}

template <class P, int LP, class Epi, size_t... I>
void launch_tile_pick(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, int Rp, const Epi& epi,
                      const SplitRoom& room, std::index_sequence<I...>) {
  if constexpr (std::is_same_v<P, F32>) {
    // fp32 (the cost fit above covers bf16 only): 128 x 128 where that gives two
    // work-groups per CU, else 64 x 64, which has four times as many; never
    // split.  A two-layer pass of 256 features over 2931 rows took 411 us with
    // 128 x 128 and takes 369 us so (k_row_rscale's narrow form included).
    const TileSplit ts{};
    const dim3 big(rule_div(NT, 8), rule_div(Rp / 16, 8)), small(rule_div(NT, 4), rule_div(Rp / 16, 4));
    if (static_cast<int64_t>(big.x) * big.y >= 512) {
      k_tile_gemm<P, 8, 8, 2, false, Epi, LP><<<big, kTileWaves * 64, 0, st>>>(w, x, NT, KB, Rp, ts, epi);
    } else {
      k_tile_gemm<P, 4, 4, 3, false, Epi, LP><<<small, kTileWaves * 64, 0, st>>>(w, x, NT, KB, Rp, ts, epi);
    }
  } else {
    const TilePick pick = tile_pick(NT, KB, Rp, P::parts, room.cap());
    (void)((static_cast<int>(I) == pick.shape &&
            (launch_tile_shape<P, LP, I>(st, NT, w, x, KB, Rp, epi, room, pick.slices), true)) ||
           ...);
  }
}

template <class P, int LP, class Epi>
void launch_tile_gemm(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, int Rp, const Epi& epi,
                      const SplitRoom& room) {
  launch_tile_pick<P, LP>(st, NT, w, x, KB, Rp, epi, room, std::make_index_sequence<std::size(kTileShapes)>{});
}

}  // namespace sprk
