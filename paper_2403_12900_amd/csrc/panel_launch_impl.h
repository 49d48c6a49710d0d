// Launch of a picked shape of the panel kernel (see panel_launch.h).
#pragma once

#include <iterator>
#include <utility>

#include "panel_launch.h"

namespace sprk {

// Whether an epilogue is QKV's.
template <class E>
struct IsQKV : std::false_type {};
template <class F, class KP, bool RS>
struct IsQKV<EpiQKV<F, KP, RS>> : std::true_type {};

template <class P, int JT, size_t I, class Epi>
void launch_panel_shape(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, const Epi& epi, int S,
                        const SplitRoom& room) {
  constexpr PanelShape sh = PanelShapes<std::is_same_v<P, F32>, JT>::s[I];
  const int groups = rule_div(NT, sh.nw * sh.rt);
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
                  const SplitRoom& room, const PanelPick& pick, std::index_sequence<I...>) {
  (void)((static_cast<int>(I) == pick.shape &&
          (launch_panel_shape<P, JT, I>(st, NT, w, x, KB, epi, pick.slices, room), true)) ||
         ...);
}

template <class P, class Epi>
void launch_panel_gemm(hipStream_t st, int NT, const uint4* w, const uint4* x, int KB, const Epi& epi,
                       const SplitRoom& room, const PanelPick& pick) {
  constexpr bool kF32 = std::is_same_v<P, F32>;
  auto panel = [&](auto jt) {
    constexpr int JT = decltype(jt)::value;
    launch_panel<P, JT>(st, NT, w, x, KB, epi, room, pick,
                        std::make_index_sequence<std::size(PanelShapes<kF32, JT>::s)>{});
  };
  switch (row_tiles(epi.n_rows)) {
    case 1:
      if constexpr (!kF32) panel(std::integral_constant<int, 1>{});  // fp32: always streamed
      break;
    case 2: panel(std::integral_constant<int, 2>{}); break;
    case 3: panel(std::integral_constant<int, 3>{}); break;
    case 4: panel(std::integral_constant<int, 4>{}); break;
    case 6:
      if constexpr (!(kF32 && IsQKV<Epi>::value)) panel(std::integral_constant<int, 6>{});  // fp32 passes end at 64 rows
      break;
    default:
      if constexpr (!(kF32 && IsQKV<Epi>::value)) panel(std::integral_constant<int, 8>{});
      break;
  }
}

}  // namespace sprk
