// The rules that pick a projection's kernel, tile shape and K slices from its
// sizes.  Pure C++ (no HIP): the launches and the host test library share them.
//
// Sizes: NT 16-row weight tiles, KB K-blocks per tile, JT 16-row activation
// tiles, parts = activation parts (fp32 1, bf16 2, bf16 QKV input 3).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <iterator>

#include "host_state.h"

namespace sprk {

inline int rule_div(int a, int b) { return (a + b - 1) / b; }

// 16-row activation tiles of a pass over n rows (kernels exist for these
// counts).
inline int row_tiles(int n) {
  const int t = (n + 15) / 16;
  return t <= 4 ? t : t <= 6 ? 6 : 8;
}

// What a split-K launch may use: floats of partial sums and arrival counters.
struct SplitCap {
  size_t floats = 0;
  int counters = 0;
};

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
// fp32: one shape, for two row tiles or more (one row tile is streamed).
template <int JT>
struct PanelShapes<true, JT> {
  static constexpr PanelShape s[] = {{4, 1, 1}};
};

struct PanelShapeSet {
  const PanelShape* s;
  int n;
};
inline PanelShapeSet panel_shapes(bool f32, int JT) {
  auto set = [](const auto& a) { return PanelShapeSet{a, static_cast<int>(std::size(a))}; };
  if (f32) return set(PanelShapes<true, 1>::s);
  switch (JT) {
    case 1: return set(PanelShapes<false, 1>::s);
    case 2: return set(PanelShapes<false, 2>::s);
    case 3: return set(PanelShapes<false, 3>::s);
    case 4: return set(PanelShapes<false, 4>::s);
    default: return set(PanelShapes<false, 8>::s);
  }
}

// Shape (index) and slices of a panel launch: the least of an estimated time
// in microseconds, fitted to 2600 timings of the kernel on MI355X (the
// projections of the 7B, 13B and 70B shapes and uneven ones, 14 to 128 rows,
// 1 to 10 slices): the busiest CU's chain of K-blocks -- its weight tiles, and
// the activation tiles they share, which every wave reads from LDS -- combined
// with the HBM time of the matrix, plus the publication of the slices.  Its
// choices are on average 2% slower than the fastest.  More than one work-group
// per CU is priced up by 5% each (512 tiles x 256 K-blocks, 14 rows: 768
// work-groups 30 us, 192 take 24).  Slices of a multiple of 64 K-blocks in
// tiles of a multiple of 256 are priced up by a quarter, since all work-groups
// then start at multiples of 64 KiB and the slices of a tile at fractions of a
// power of two (in groups of 8 tiles, four slices against three: 512 tiles x
// 256 K-blocks, 14 rows 28.4 us / 24.1, 32 rows 32.0 / 27.2; of 4 tiles, 256 x
// 512, 14 rows 26.8 / 25.4).  Two slices of 128 lose less than that, but are
// never the best there; tiles of 128 K-blocks in two slices of 64 lose nothing.
struct PanelPick {
  int shape = -1, slices = 1;
  double us = 0;  // the estimate
};
inline PanelPick panel_pick(bool f32, int NT, int KB, int JT, int parts, bool norm, const SplitCap& cap) {
  constexpr int kCUs = 256, kMaxSlices = 16;
  const PanelShapeSet sh = panel_shapes(f32, JT);
  const size_t room = std::min(cap.floats, (JT <= 4 ? spr::kSplitPartBytes : spr::kSplitPartBytesWide) / sizeof(float));
  PanelPick best;
  for (int i = 0; i < sh.n; ++i) {
    const PanelShape& s = sh.s[i];
    const int T = s.nw * s.rt, groups = rule_div(NT, T), chunks = rule_div(KB, s.uc);
    const size_t quads = s.rt * JT + (norm ? (JT + 3) / 4 : 0);
    for (int S = 1; S <= kMaxSlices && S <= chunks; ++S) {
      if (S > 1 && (groups * s.nw > cap.counters || static_cast<size_t>(groups) * s.nw * S * quads * 256 > room)) break;
      const int rounds = rule_div(groups * S, kCUs);
      const double chain = 1.0 * rounds * rule_div(KB, S) * (0.012 * T + (0.0097 + 0.003 * s.nw) * JT * parts);
      const double hbm = 1.62e-4 * NT * KB;
      double us = std::sqrt(chain * chain + hbm * hbm);
      if (S > 1) us += 2.2 + 0.23 * S * s.rt * JT;
      if (S > 1 && KB % 256 == 0 && KB % (64 * S) == 0) us *= 1.25;
      us *= 1.0 + 0.05 * (rounds - 1);
      if (best.shape < 0 || us < best.us) best = PanelPick{i, S, us};
    }
  }
  return best;
}

// Rows up to which a bf16 pass takes the register-streaming kernel, packed.
constexpr int kPackedRows = 8;

// Whether the streaming kernel takes its wide form: one-wave work-groups of
// two tiles.
inline bool stream_wide(int NT, int JT, int parts) {
  return JT == 1 && parts < 3 && NT >= 1024 && NT % 2 == 0;
}

// Estimated time (us) of the streaming kernel's four-wave form at one to four
// row tiles, and of the panel kernel on the same scale, fitted to 600 timings
// on MI355X: all five projections of models of 256 to 5120 features, fp32 and
// bf16, 9 to 64 rows.  Streaming, a work-group per tile reads the whole
// activation, so its time grows with NT x KB x JT; the panel kernel starts
// with about three microseconds of staging and barriers, and an fp32 fragment
// costs it four MFMAs, which the pick's estimate prices as one.
inline double stream_us(bool f32, int NT, int KB, int JT, int parts) {
  const double rounds = rule_div(NT, 256), act = JT * parts, fill = NT / 256.0;
  if (f32)
    return 2.1 + 0.44 * JT +
           KB * (0.0028 + 0.011 * rounds + act * (0.021 * rounds + 0.0057 * fill + (fill > 1 ? 0.0313 * (fill - 1) : 0)));
  return 2.0 + 0.38 * JT + KB * (0.026 * rounds + act * (0.002 + 0.0061 * rounds + 0.0052 * fill));
}
inline double panel_us(bool f32, const PanelPick& p) { return f32 ? 2.6 + 1.55 * p.us : 3.2 + 0.7 * p.us; }

// The kernel of a projection of n rows: streaming (panel.shape < 0) or panel.
//   * up to 8 rows: streaming, but for bf16 matrices whose 14-tile work-groups
//     (7 waves x 2) fill three quarters or more of the CUs in one round, over
//     192 K-blocks or more.  Panel against streamed, 1 row: 2688 x 256 108 us /
//     114, 3584 x 256 (70B gate/up) 133 / 140, 3200 x 192 91 / 95.  Outside:
//     2304 x 256 102 / 97 and 2560 x 256 106 / 104 (CUs left idle), 4608 x 256
//     209 / 185, 5120 x 192 165 / 146 and 8016 x 256 (an LM head) 340 / 306 (a
//     second round), 1376 x 128 30.2 / 29.7; 3840 x 160 equal;
//   * one row tile (9 to 16 rows) of fp32: streaming (the panel kernel took 1.2 to 2.9 times
//     as long, but for 300 tiles x 260 K-blocks, 26.3 us against 27.6);
//   * one row tile of bf16 in the wide form: streaming below 96 K-blocks (9
//     rows, 2000 tiles x 64: 21.1 us, panel 26.0; 1024 x 96: 18.4, panel 17.8);
//   * up to 64 rows otherwise: the lesser estimate.  It is wrong by 0.5%
//     (bf16) and 0.2% (fp32) of the time on average; always taking the panel
//     kernel would cost 12% and 35% (fp32 down, 64 tiles x 64, 24 rows: 6.2 us
//     streamed, panel 8.7; bf16 down, 256 x 344, 24 rows: 27.0, panel 21.6);
//   * more rows: panel.
inline PanelPick gemm_pick(bool f32, int n, int NT, int KB, int parts, bool norm, const SplitCap& cap) {
  const int JT = row_tiles(n);
  const PanelPick stream;
  if (n <= kPackedRows) {
    const int groups = rule_div(NT, 14);
    return !f32 && KB >= 192 && groups >= 192 && groups <= 256 ? panel_pick(f32, NT, KB, JT, parts, norm, cap) : stream;
  }
  if (JT == 1 && (f32 || (stream_wide(NT, JT, parts) && KB < 96))) return stream;
  const PanelPick p = panel_pick(f32, NT, KB, JT, parts, norm, cap);
  if (JT > 4 || stream_wide(NT, JT, parts)) return p;
  return panel_us(f32, p) < stream_us(f32, NT, KB, JT, parts) ? p : stream;
}

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
constexpr int kTileWaves = 4;
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
inline TilePick tile_pick(int NT, int KB, int Rp, int parts, const SplitCap& cap) {
  constexpr int kCUs = 256, kMaxSlices = 8;
  TilePick best;
  double best_us = -1;
  for (int i = 0; i < static_cast<int>(std::size(kTileShapes)); ++i) {
    const TileShape& s = kTileShapes[i];
    const TileShape::Cost& c = parts == 3 ? s.three : s.two;
    const int64_t tiles = int64_t{rule_div(NT, s.tn)} * rule_div(Rp / 16, s.tm);
    const size_t slice_floats = static_cast<size_t>(s.tn) * s.tm * 256;
    for (int S = 1; S <= kMaxSlices && S <= KB; ++S) {
      if (S > 1 && (tiles * kTileWaves > cap.counters || static_cast<size_t>(tiles) * S * slice_floats > cap.floats))
        break;
      const double mean = static_cast<double>(tiles) * S / kCUs;
      const double k = 0.5 * static_cast<double>((tiles * S + kCUs - 1) / kCUs) + 0.5 * (mean > 1 ? mean : 1);
      const double kb_us = c.alone > k * c.shared ? c.alone : k * c.shared;
      const double chain = rule_div(KB, S) * kb_us + k * c.tile, hbm = 1.62e-4 * NT * KB;
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

}  // namespace sprk
