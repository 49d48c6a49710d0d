// Projection for up to 128 token rows (decode passes past 8 rows and prompt
// chunks of at most 128, where gemm_pick finds it faster than streaming, and a
// few large matrices at any row count): y[b][n] = sum_k W[n][k] x[b][k], with
// the op that follows fused into the epilogue.
//
// At these row counts a projection is still bound by its weight stream, but
// every work-group needs the activations of its K range too: with the
// register-streaming kernel of gemm_kernels.h each wave reads them for its own
// one to four weight tiles, and from 32 rows on that L2 traffic exceeds the
// weights'.  Here the NW waves of a work-group share them:
//   * a work-group owns NW x RT weight tiles (RT per wave) and a slice of the
//     K-blocks; weight fragments go straight from HBM into the registers of
//     the one wave that uses them (nontemporal, each byte read once);
//   * the activation fragments of a chunk of UC K-blocks go from L2 into LDS
//     once per work-group and all waves read them there: one activation byte
//     moved per NW x RT tiles instead of per RT;
//   * a wave's weight registers hold three chunks in turn and its share of the
//     activations two, so two chunks are in flight while one is multiplied;
//     the activations are written to LDS (two buffers) once they have arrived,
//     one barrier per chunk.  They are staged in registers, not sent straight
//     to LDS: with direct-to-LDS loads in flight the compiler waits for every
//     outstanding load before it uses a loaded weight register.
// K is split over S work-groups per group of tiles (SplitK below).
#pragma once

#include <type_traits>

#include "gemm_kernels.h"
#include "lds_pipe.h"

namespace sprk {

// Split-K across work-groups: the S work-groups of a group of NW x RT tiles
// each take a contiguous 1/S of the K-blocks, so that projections with few
// tiles still fill the CUs with large groups.  Each wave publishes its partial
// sums (and the rows' partial sums of squares) with agent-coherent stores and
// counts itself in; the last slice's wave to arrive adds the S partials in
// slice order -- the same order whichever arrives last, so the result stays
// bitwise reproducible -- and runs the epilogue.  No work-group waits on
// another.  Slice = block mod S, so a slice's work-groups share XCDs (work-
// groups go to the XCDs round robin) and each L2 holds only its slices'
// activations.
struct SplitK {
  float* part;    // [group][wave][slice][fragment][64 lanes][4] floats
  int32_t* cnt;   // [group][wave] arrived slices; zero between launches
};

// Fragments of four floats a lane publishes per slice: accumulators, then sums
// of squares.
template <int JT, int RT, bool kNorm>
struct SplitKQuads {
  static constexpr int value = RT * JT + (kNorm ? (JT + 3) / 4 : 0);
};

template <int RT, int UC>
struct PanelWeights {
  u32x4_t a[UC][RT];  // weight fragments of a chunk
};
template <int PARTS, int JT, int UC, int NW>
struct PanelActs {
  static constexpr int frags = UC * JT * PARTS;  // of a chunk
  static constexpr int per_wave = (frags + NW - 1) / NW;
  static constexpr int u4 = frags * 64;          // LDS uint4 of a buffer
  u32x4_t x[per_wave];                           // this wave's share of a chunk
};

// The barrier of a chunk: this wave's LDS writes are done, then all waves'.
// (No fence: it would wait for the loads in flight as well.)
__device__ __forceinline__ void panel_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// One work-group's tiles nt0 .. nt0 + NW RT - 1 over slice `slice` of S.
// lds: two buffers of PanelActs<PARTS, JT, UC, NW>::u4.  LP: parts per K-block of
// the record.
template <class P, int LP, int JT, int NW, int RT, int UC, class Epi>
__device__ __forceinline__ void panel_tiles(const uint4* W, const uint4* X, int KB, int NT, int Rp, const Epi& epi,
                                            int nt0, int slice, int S, const SplitK& sk, u32x4_t* lds) {
  constexpr int PARTS = P::parts;
  using Weights = PanelWeights<RT, UC>;
  using Acts = PanelActs<PARTS, JT, UC, NW>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt = nt0 + wave * RT;
  const int NC = (KB + UC - 1) / UC;
  const int c0 = (NC * slice) / S, c1 = (NC * (slice + 1)) / S;

  // Fragment of the i-th activation load of this wave (waves past the last
  // fragment repeat it).
  auto frag = [&](int i) __attribute__((always_inline)) { return min(wave + NW * i, Acts::frags - 1); };
  // Addresses: a wave-uniform base per chunk plus 32-bit lane offsets.  A last
  // chunk of fewer than UC K-blocks reads past the tile (the next tile, or
  // what follows the matrix in the workspace) and past the record; those
  // K-blocks are not multiplied.
  const uint32_t xpart = static_cast<uint32_t>(Rp) * 4;  // uint4 per (K-block, part)
  constexpr ActRec xr = act_rec(16 * JT);
  uint32_t xoff[Acts::per_wave];
#pragma unroll
  for (int i = 0; i < Acts::per_wave; ++i) {
    const int f = frag(i), u = f / (JT * PARTS), r = f % (JT * PARTS), q = r / JT, j = r % JT;
    xoff[i] = (u * LP + q) * xpart + j * 64 + (lane & 15) * xr.rs + (lane >> 4) * xr.gs;
  }
  const uint4* wt[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) wt[t] = W + static_cast<size_t>(min(nt + t, NT - 1)) * KB * 64;
  auto issue = [&](int c, Weights& w, Acts& x) __attribute__((always_inline)) {
    const u32x4_t* xc = reinterpret_cast<const u32x4_t*>(X + static_cast<size_t>(c) * (UC * LP) * xpart);
#pragma unroll
    for (int i = 0; i < Acts::per_wave; ++i) x.x[i] = xc[xoff[i]];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const u32x4_t* wc = reinterpret_cast<const u32x4_t*>(wt[t] + static_cast<size_t>(c) * (UC * 64));
#pragma unroll
      for (int u = 0; u < UC; ++u) w.a[u][t] = __builtin_nontemporal_load(wc + static_cast<uint32_t>(lane + u * 64));
    }
    __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products that follow
  };
  auto stage = [&](const Acts& x, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < Acts::per_wave; ++i) lds[buf * Acts::u4 + frag(i) * 64 + lane] = x.x[i];
  };

  // Sums of squares (RMSNorm) come from Gram products of the activations with
  // themselves, see stream_gemm_tiles, shared by the first GW waves: with
  // three row tiles or more, wave w takes tiles w, w + GW, ..; with one or
  // two, tile w mod JT of every (4 / JT)-th K-block.
  static_assert(NW >= 4, "the Gram products are shared by up to four waves");
  constexpr int GW = JT <= 2 || JT % 4 == 0 ? 4 : 3;
  constexpr int GT = JT <= 2 ? 1 : JT / GW;
  static_assert(JT <= 2 || GT * GW == JT, "row tiles split evenly over the Gram waves");
  f32x4_t acc[RT][JT], gram[GT];
#pragma unroll
  for (int k = 0; k < GT; ++k) gram[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < JT; ++j) {
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // Products of chunk c (its activations in LDS buffer buf).  kTail: the chunk
  // may hold fewer than UC K-blocks.
  auto compute = [&](auto tail, int c, const Weights& w, int buf) __attribute__((always_inline)) {
    constexpr bool kTail = decltype(tail)::value;
    const u32x4_t* base = lds + buf * Acts::u4 + lane;
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      if (kTail && c * UC + u >= KB) break;
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        uint4 x[PARTS];
#pragma unroll
        for (int q = 0; q < PARTS; ++q) x[q] = __builtin_bit_cast(uint4, base[((u * PARTS + q) * JT + j) * 64]);
#pragma unroll
        for (int q = 0; q < PARTS; ++q)
#pragma unroll
          for (int t = 0; t < RT; ++t) acc[t][j] = P::mma(acc[t][j], __builtin_bit_cast(uint4, w.a[u][t]), x[q]);
      }
    }
    if constexpr (!kTail && std::is_same_v<typename P::elem, uint16_t>) {
      // LDS reads run two row tiles ahead of the products.
      constexpr int kDs = 0x100, kMfma = 0x8, kSteps = UC * JT;
      __builtin_amdgcn_sched_group_barrier(kDs, (kSteps < 2 ? kSteps : 2) * PARTS, 0);
#pragma unroll
      for (int i = 0; i < kSteps; ++i) {
        __builtin_amdgcn_sched_group_barrier(kMfma, RT * PARTS, 0);
        if (i + 2 < kSteps) __builtin_amdgcn_sched_group_barrier(kDs, PARTS, 0);
      }
    }
    if constexpr (Epi::kNorm) {
      if (wave < GW) {
#pragma unroll
        for (int u = 0; u < UC; ++u) {
          if (kTail && c * UC + u >= KB) break;
          if constexpr (JT <= 2) {
            if ((c * UC + u) % (4 / JT) != wave / JT) continue;
          }
#pragma unroll
          for (int k = 0; k < GT; ++k) {
            const int j = JT <= 2 ? wave % JT : wave + GW * k;
            uint4 x[PARTS];
#pragma unroll
            for (int q = 0; q < PARTS; ++q) x[q] = __builtin_bit_cast(uint4, base[((u * PARTS + q) * JT + j) * 64]);
            gram[k] = P::mma(gram[k], x[0], x[0]);
            if constexpr (PARTS >= 2) {
              gram[k] = P::mma(gram[k], x[0], x[1]);
              gram[k] = P::mma(gram[k], x[1], x[0]);
            }
            if constexpr (PARTS == 3) {
              gram[k] = P::mma(gram[k], x[1], x[1]);
              gram[k] = P::mma(gram[k], x[0], x[2]);
              gram[k] = P::mma(gram[k], x[2], x[0]);
            }
          }
        }
      }
    }
  };
  // Chunk c, whose activations are in LDS buffer b: load chunk c + 2, multiply,
  // hand chunk c + 1's activations to the other buffer (which every wave has
  // finished reading before this step's barrier).
  auto step = [&](int c, const Weights& w, Weights& w2, Acts& x2, const Acts& x1, int b)
      __attribute__((always_inline)) {
    panel_barrier();
    issue(c + 2, w2, x2);
    compute(std::false_type{}, c, w, b);
    stage(x1, b ^ 1);
  };
  // The last one or two chunks.
  auto finish = [&](int c, const Weights& w, const Weights& w1, const Acts& x1, int b) __attribute__((always_inline)) {
    panel_barrier();
    compute(std::true_type{}, c, w, b);
    if (c + 1 < c1) {
      stage(x1, b ^ 1);
      panel_barrier();
      compute(std::true_type{}, c + 1, w1, b ^ 1);
    }
  };

  Weights w0, w1, w2;
  Acts x0, x1;
  issue(c0, w0, x0);
  issue(min(c0 + 1, c1 - 1), w1, x1);
  stage(x0, 0);
  int c = c0;
  for (; c + 7 < c1; c += 6) {  // six steps: three weight stages, two activation stages and buffers
    step(c, w0, w2, x0, x1, 0);
    step(c + 1, w1, w0, x1, x0, 1);
    step(c + 2, w2, w1, x0, x1, 0);
    step(c + 3, w0, w2, x1, x0, 1);
    step(c + 4, w1, w0, x0, x1, 0);
    step(c + 5, w2, w1, x1, x0, 1);
  }
  // One to seven chunks left.
  if (c + 2 < c1) {
    step(c, w0, w2, x0, x1, 0);
    if (c + 3 < c1) {
      step(c + 1, w1, w0, x1, x0, 1);
      if (c + 4 < c1) {
        step(c + 2, w2, w1, x0, x1, 0);
        if (c + 5 < c1) {
          step(c + 3, w0, w2, x1, x0, 1);
          if (c + 6 < c1) {
            step(c + 4, w1, w0, x0, x1, 0);
            finish(c + 5, w2, w0, x0, 1);
          } else {
            finish(c + 4, w1, w2, x1, 0);
          }
        } else {
          finish(c + 3, w0, w1, x0, 1);
        }
      } else {
        finish(c + 2, w2, w0, x1, 0);
      }
    } else {
      finish(c + 1, w1, w2, x0, 1);
    }
  } else {
    finish(c, w0, w1, x1, 0);
  }

  typename Epi::Pre pre[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) pre[t] = epi.template prefetch<JT>(min(nt + t, NT - 1), lane);

  float ssq[JT];
  if constexpr (Epi::kNorm) {
    float* red = reinterpret_cast<float*>(lds);  // [Gram wave][its tile][16]
    const int c = lane & 15;
    __syncthreads();
    if (wave < GW) {
#pragma unroll
      for (int k = 0; k < GT; ++k) {
        const float s = gram_entry(gram_pick(gram[k], lane), c, c);
        if (lane < 16) red[(wave * GT + k) * 16 + lane] = s;
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      if constexpr (JT <= 2) {
        ssq[j] = red[j * 16 + c];
#pragma unroll
        for (int w = j + JT; w < 4; w += JT) ssq[j] += red[w * 16 + c];
      } else {
        ssq[j] = red[(j % GW * GT + j / GW) * 16 + c];
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < JT; ++j) ssq[j] = 0.f;
  }

  if (S > 1) {
    // Fragments of four floats a lane: accumulators, then sums of squares.
    constexpr int NA = RT * JT, NQ = SplitKQuads<JT, RT, Epi::kNorm>::value;
    const int g = __builtin_amdgcn_readfirstlane((nt0 / (NW * RT)) * NW + wave);
    const CoherentBuffer buf(sk.part + static_cast<size_t>(g) * S * NQ * 256, static_cast<uint32_t>(S) * NQ * 1024);
    auto at = [&](int q, int i) __attribute__((always_inline)) {
      return static_cast<uint32_t>((q * NQ + i) * 1024 + lane * 16);
    };
#pragma unroll
    for (int i = 0; i < NA; ++i) buf.store4(at(slice, i), acc[i / JT][i % JT]);
    if constexpr (Epi::kNorm) {
#pragma unroll
      for (int i = 0; i < NQ - NA; ++i) {
        f32x4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = 4 * i + e < JT ? ssq[4 * i + e] : 0.f;
        buf.store4(at(slice, NA + i), v);
      }
    }
    wait_vmem<0>();  // this slice's partial stores are complete
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    int last = 0;
    if (lane == 0) last = __hip_atomic_fetch_add(sk.cnt + g, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == S - 1;
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    if (lane == 0) __hip_atomic_store(sk.cnt + g, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    // Sum in slice order; all of a slice's loads are in flight at once.
    f32x4_t sum[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) sum[i] = buf.load4(at(0, i));
    for (int q = 1; q < S; ++q) {
      f32x4_t nx[NQ];
#pragma unroll
      for (int i = 0; i < NQ; ++i) nx[i] = buf.load4(at(q, i));
#pragma unroll
      for (int i = 0; i < NQ; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[i][e] += nx[i][e];
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i / JT][i % JT] = sum[i];
    if constexpr (Epi::kNorm) {
#pragma unroll
      for (int j = 0; j < JT; ++j) ssq[j] = sum[NA + j / 4][j % 4];
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t)
    if (nt + t < NT) epi.template apply<JT>(nt + t, acc[t], ssq, lane, pre[t]);
}

template <class P, int JT, int NW, int RT, int UC, class Epi>
__global__ __launch_bounds__(NW * 64) void k_panel_gemm(const uint4* W, const uint4* X, int KB, int NT, int Rp, int S,
                                                        SplitK sk, Epi epi) {
  __shared__ u32x4_t lds[2 * PanelActs<P::parts, JT, UC, NW>::u4];
  panel_tiles<P, P::parts, JT, NW, RT, UC, Epi>(W, X, KB, NT, Rp, epi, (blockIdx.x / S) * NW * RT, blockIdx.x % S, S, sk,
                                                lds);
}

// QKV projection over a three-part record: work-groups of query tiles take its
// first two parts, those that hold a key or value tile all three (see
// k_stream_gemm_qkv).  The branch is uniform per work-group.
template <int JT, int NW, int RT, int UC, class Epi>
__global__ __launch_bounds__(NW * 64) void k_panel_gemm_qkv(const uint4* W, const uint4* X, int KB, int NT, int Rp, int S,
                                                            SplitK sk, Epi epi, int q_tiles) {
  __shared__ u32x4_t lds[2 * PanelActs<BF16x3::parts, JT, UC, NW>::u4];
  const int nt0 = (blockIdx.x / S) * NW * RT, slice = blockIdx.x % S;
  if (nt0 + NW * RT <= q_tiles) {
    panel_tiles<BF16, 3, JT, NW, RT, UC, Epi>(W, X, KB, NT, Rp, epi, nt0, slice, S, sk, lds);
  } else {
    panel_tiles<BF16x3, 3, JT, NW, RT, UC, Epi>(W, X, KB, NT, Rp, epi, nt0, slice, S, sk, lds);
  }
}

}  // namespace sprk
