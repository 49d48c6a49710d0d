// Shapes of the tiled projection and the rule that picks one (see
// tile_launch.h).
#pragma once

#include <cmath>
#include <iterator>
#include <type_traits>
#include <utility>

#include "tile_launch.h"

namespace sprk {

inline int tile_div(int a, int b) { return (a + b - 1) / b; }

// A shape of k_tile_gemm and its measured times in microseconds (MI355X, two
// and three activation parts): a K-block of a tile when its work-group is
// alone on its CU, and when others share the CU (per tile); the start and end
// of a tile; the publication of a split tile, and of each further slice.  The
// last shape's four stages cover HBM latency where tiles are few.
struct TileShape {
  int tn, tm, nst;
  struct Cost {
    double alone, shared, tile, split, slice;
  } two, three;
};
constexpr TileShape kTileShapes[] = {
    {16, 8, 2, {0.827, 0.743, 1.8, 14.1, 1.26}, {1.067, 1.057, 0.0, 15.4, 1.07}},
    {8, 8, 2, {0.692, 0.420, 0.0, 11.5, 0.66}, {0.756, 0.595, 0.0, 12.4, 0.54}},
    {8, 4, 2, {0.618, 0.257, 0.8, 7.9, 0.28}, {0.627, 0.275, 3.0, 7.0, 0.06}},
    {8, 4, 4, {0.289, 0.250, 1.0, 8.3, 0.21}, {0.386, 0.307, 1.7, 8.1, 0.13}},
};

// The pick: the least estimated time.  The busiest CU's tiles (halfway between
// the whole number and the mean, since a CU left with fewer runs them faster)
// are multiplied one after another at the shared rate, but a tile alone is
// bound by its own latency; the HBM time of the weights adds in quadrature.
// Fitted to 900 timings of the 7B, 13B and 70B projections at 128 to 4096 rows
// with weights from HBM; its choices are 2% slower than the fastest on average.
struct TilePick {
  int shape = 0, slices = 1;
};
inline TilePick tile_pick(int NT, int KB, int Rp, int parts, const SplitRoom& room) {
  constexpr int kCUs = 256, kMaxSlices = 8;
  TilePick best;
  double best_us = -1;
  for (int i = 0; i < static_cast<int>(std::size(kTileShapes)); ++i) {
    const TileShape& s = kTileShapes[i];
    const TileShape::Cost& c = parts == 3 ? s.three : s.two;
    const int64_t tiles = int64_t{tile_div(NT, s.tn)} * tile_div(Rp / 16, s.tm);
    const size_t slice_floats = static_cast<size_t>(s.tn) * s.tm * 256;
    for (int S = 1; S <= kMaxSlices && S <= KB; ++S) {
      if (S > 1 && (room.part == nullptr || tiles * kTileWaves > room.n_cnt ||
                    static_cast<size_t>(tiles) * S * slice_floats > room.part_floats))
        break;
      const double mean = static_cast<double>(tiles) * S / kCUs;
      const double k = 0.5 * static_cast<double>((tiles * S + kCUs - 1) / kCUs) + 0.5 * (mean > 1 ? mean : 1);
      const double kb_us = c.alone > k * c.shared ? c.alone : k * c.shared;
      const double chain = tile_div(KB, S) * kb_us + k * c.tile, hbm = 1.62e-4 * NT * KB;
      double us = std::sqrt(chain * chain + hbm * hbm);
      if (S > 1) us += c.split + c.slice * S * static_cast<double>((tiles * S + kCUs - 1) / kCUs);
      if (best_us < 0 || us < best_us) {
        best = TilePick{i, S};
        best_us = us;
      }
    }
  }
  return best;
}

template <class P, int LP, size_t I, class Epi>
void launch_tile_shape(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, int Rp, const Epi& epi,
                       const SplitRoom& room, int S) {
  constexpr TileShape s = kTileShapes[I];
  const dim3 grid(tile_div(NT, s.tn), tile_div(Rp / 16, s.tm), S);
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
    const dim3 big(tile_div(NT, 8), tile_div(Rp / 16, 8)), small(tile_div(NT, 4), tile_div(Rp / 16, 4));
    if (static_cast<int64_t>(big.x) * big.y >= 512) {
      k_tile_gemm<P, 8, 8, 2, false, Epi, LP><<<big, kTileWaves * 64, 0, st>>>(w, x, NT, KB, Rp, ts, epi);
    } else {
      k_tile_gemm<P, 4, 4, 3, false, Epi, LP><<<small, kTileWaves * 64, 0, st>>>(w, x, NT, KB, Rp, ts, epi);
    }
  } else {
    const TilePick pick = tile_pick(NT, KB, Rp, P::parts, room);
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
