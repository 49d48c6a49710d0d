// Shapes of the panel kernel and the rule that picks one (see panel_launch.h).
#pragma once

#include <cmath>
#include <iterator>
#include <utility>

#include "host_state.h"
#include "panel_launch.h"

namespace sprk {

inline int panel_div(int a, int b) { return (a + b - 1) / b; }

// Whether an epilogue is QKV's.
template <class E>
struct IsQKV : std::false_type {};
template <class F, class KP>
struct IsQKV<EpiQKV<F, KP>> : std::true_type {};

// Shapes of k_panel_gemm by row tiles: waves, tiles per wave, K-blocks per
// chunk.  A work-group's NW x RT tiles are what one activation byte moved into
// LDS serves; the set covers group sizes that divide the usual tile counts
// into close to 256 work-groups (one per CU) with few slices.
struct PanelShape {
  int nw, rt, uc;
};
template <bool kF32, int JT>
struct PanelShapes {
  static constexpr PanelShape s[] = {{4, 1, 1}, {8, 1, 1}, {8, 2, 1}, {4, 3, 1}};  // 65 to 128 rows
};
template <>
struct PanelShapes<false, 1> {
  static constexpr PanelShape s[] = {{4, 1, 4}, {6, 1, 2}, {4, 2, 2}, {7, 2, 2}};
};
template <>
struct PanelShapes<false, 2> {
  static constexpr PanelShape s[] = {{4, 1, 2}, {6, 1, 2}, {8, 1, 2}, {7, 2, 2}};
};
template <>
struct PanelShapes<false, 3> {
  static constexpr PanelShape s[] = {{4, 1, 2}, {8, 1, 2}, {4, 2, 2}, {6, 2, 2}, {7, 2, 2}};
};
template <>
struct PanelShapes<false, 4> {
  static constexpr PanelShape s[] = {{4, 1, 2}, {8, 1, 2}, {4, 2, 2}, {6, 2, 2}, {7, 2, 2}};
};
// fp32 models (no full-size fp32 model is served): one shape.
template <int JT>
struct PanelShapes<true, JT> {
  static constexpr PanelShape s[] = {{4, 1, 1}};
};

// Shape (index) and slices of a panel launch: the least of an estimated time
// in microseconds, fitted to 2600 timings of the kernel on MI355X (the
// projections of the 7B, 13B and 70B shapes and uneven ones, 14 to 128 rows,
// 1 to 10 slices): the busiest CU's chain of K-blocks -- its weight tiles, and
// the activation tiles they share, which every wave reads from LDS -- combined
// with the HBM time of the matrix, plus the publication of the slices.  Its
// choices are on average 2% slower than the fastest.  More than one work-group
// per CU is priced up by 5% each (512 tiles x 256 K-blocks, 14 rows: 768
// work-groups 30 us, 192 take 23.5).  Slices of
// 64 K-blocks of 256-K-block tiles are priced up: every work-group then
// starts at a multiple of 64 KiB (512 tiles x 256 K-blocks, 14 rows: four
// slices 31 us, three 23.5 us).
struct PanelPick {
  int shape = -1, slices = 1;
};
inline PanelPick panel_pick(const PanelShape* sh, int n_shapes, int NT, int KB, int JT, int parts, bool norm) {
  constexpr int kCUs = 256, kMaxSlices = 16;
  const size_t room = JT <= 4 ? spr::kSplitPartBytes : spr::kSplitPartBytesWide;
  PanelPick best;
  double best_us = 0;
  for (int i = 0; i < n_shapes; ++i) {
    const int T = sh[i].nw * sh[i].rt, groups = panel_div(NT, T), chunks = panel_div(KB, sh[i].uc);
    const size_t quads = sh[i].rt * JT + (norm ? (JT + 3) / 4 : 0);
    for (int S = 1; S <= kMaxSlices && S <= chunks; ++S) {
      if (S > 1 && static_cast<size_t>(groups) * sh[i].nw * S * quads * 256 * sizeof(float) > room) break;
      const int rounds = panel_div(groups * S, kCUs);
      const double chain = 1.0 * rounds * panel_div(KB, S) *
                           (0.012 * T + (0.0097 + 0.003 * sh[i].nw) * JT * parts);
      const double hbm = 1.62e-4 * NT * KB;
      double us = std::sqrt(chain * chain + hbm * hbm);
      if (S > 1) us += 2.2 + 0.23 * S * sh[i].rt * JT;
      if (S > 1 && KB % 256 == 0 && KB % (64 * S) == 0) us *= 1.25;
      us *= 1.0 + 0.05 * (rounds - 1);
      if (best.shape < 0 || us < best_us) {
        best = PanelPick{i, S};
        best_us = us;
      }
    }
  }
  return best;
}

template <class P, int JT, size_t I, class Epi>
void launch_panel_shape(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, const Epi& epi, int S,
                        const SplitRoom& room) {
  constexpr PanelShape sh = PanelShapes<std::is_same_v<P, F32>, JT>::s[I];
  const int groups = panel_div(NT, sh.nw * sh.rt);
  const SplitK sk{room.part, room.cnt};
  if constexpr (IsQKV<Epi>::value && P::parts == 3) {
    const int q_tiles = epi.H * epi.hd / 16;
    k_panel_gemm_qkv<JT, sh.nw, sh.rt, sh.uc, Epi>
        <<<groups * S, sh.nw * 64, 0, st>>>(w, x, KB, NT, 16 * JT, S, sk, epi, q_tiles);
  } else {
    k_panel_gemm<P, JT, sh.nw, sh.rt, sh.uc, Epi>
        <<<groups * S, sh.nw * 64, 0, st>>>(w, x, KB, NT, 16 * JT, S, sk, epi);
  }
}

template <class P, int JT, class Epi, size_t... I>
void launch_panel(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, const Epi& epi,
                  const SplitRoom& room, std::index_sequence<I...>) {
  const PanelPick pick = panel_pick(PanelShapes<std::is_same_v<P, F32>, JT>::s, sizeof...(I), NT, KB, JT, P::parts, Epi::kNorm);
  (void)((static_cast<int>(I) == pick.shape &&
          (launch_panel_shape<P, JT, I>(st, NT, w, x, KB, epi, pick.slices, room), true)) ||
         ...);
}

template <class P, class Epi>
void launch_panel_gemm(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, const Epi& epi,
                       const SplitRoom& room) {
  auto panel = [&](auto jt) {
    constexpr int JT = decltype(jt)::value;
    launch_panel<P, JT>(st, NT, w, x, KB, epi, room,
                        std::make_index_sequence<std::size(PanelShapes<std::is_same_v<P, F32>, JT>::s)>{});
  };
  switch (row_tiles(epi.n_rows)) {
    case 1: panel(std::integral_constant<int, 1>{}); break;
    case 2: panel(std::integral_constant<int, 2>{}); break;
    case 3: panel(std::integral_constant<int, 3>{}); break;
    case 4: panel(std::integral_constant<int, 4>{}); break;
    case 6: panel(std::integral_constant<int, 6>{}); break;
    default: panel(std::integral_constant<int, 8>{}); break;
  }
}

}  // namespace sprk
