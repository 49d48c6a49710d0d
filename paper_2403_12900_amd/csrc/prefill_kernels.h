// Prefill: the prompt of every new request runs through the model in chunks
// of up to kPrefillRows token rows, filling the KV cache (Section II-A: the
// prompt's keys and values are computed once and cached; generation follows).
// Unlike decode, each weight byte now meets hundreds of rows, so the
// projections are compute-bound: a tiled MFMA GEMM stages output tiles of up
// to 256 features x 128 rows through LDS.  Attention is causal over each request's own
// positions; a wave's 16 MFMA columns are 16 consecutive query positions of
// one request and head, and the four waves of a work-group share each K/V
// tile they read from LDS, so every tile read feeds up to 64 queries.
#pragma once

#include "attn_kernels.h"
#include "launch_rule.h"
#include "lds_pipe.h"

namespace sprk {

constexpr int kPrefillRows = 4096;  // token rows per prefill chunk

// One token row of a chunk.
struct PrefillRow {
  int slot, pos, tok, pad;
};

// Up to 64 consecutive rows of one request (positions pos0 .. pos0 + n - 1
// at chunk rows row0 .. row0 + n - 1): one attention query tile.
struct PrefillTile {
  int slot, row0, n, pos0;
};

// x = E[tok], and its activation record (K-block-major, Rp rows).
template <class P>
__global__ __launch_bounds__(64) void k_embed_rows(const typename P::elem* __restrict__ emb,
                                                   const PrefillRow* __restrict__ rows, float* x,
                                                   typename P::elem* act, int d, int V, ActRec rec) {
  const int b = blockIdx.y;
  const int n0 = 4 * (blockIdx.x * 64 + threadIdx.x);
  if (n0 >= d) return;
  const int t = min(max(rows[b].tok, 0), V - 1);
  const typename P::elem* e = emb + static_cast<size_t>(t) * d + n0;
  const float v0 = P::to_f32(e[0]), v1 = P::to_f32(e[1]), v2 = P::to_f32(e[2]), v3 = P::to_f32(e[3]);
  *reinterpret_cast<float4*>(x + static_cast<size_t>(b) * d + n0) = make_float4(v0, v1, v2, v3);
  store_resid4<P>(act, rec, b, n0, d, make_float4(v0, v1, v2, v3));
}

// Tiled projection: out[b][n] = sum_k W[n][k] x[b][k] for rows b < M, fused
// with the op that follows (Epi).  An output tile is TN weight tiles (16
// output features each) x TM row tiles (16 rows each); the four waves (2 x 2)
// of a work-group each own a TN/2 x TM/2 block of 16 x 16 MFMA tiles.  Per
// K-block the tile's operands -- TN weight fragments and TM x parts activation
// fragments, 1 KiB each -- go from global memory straight into LDS
// (global_load_lds, no register staging) in MFMA lane order, the order both
// are stored in.  NST LDS stages keep NST - 1 K-blocks in flight; each K-block
// costs one barrier: wait for its own loads, barrier (which also frees the
// stage read one K-block earlier), issue the loads NST - 1 K-blocks ahead,
// multiply.  Weight tiles past NT re-read tile NT - 1 and row tiles past Rp
// re-read the last one; neither is stored.
//
// What bounds it (MI355X, 4096 rows of the 7B gate/up projection, in a six-
// layer prefill): 1140 us, of which its LDS reads and MFMAs alone take 925 and
// its loads alone 687.  The two overlap only across work-groups, since within
// one every wave waits at the same barrier.  So a shape is chosen for two or
// more work-groups per CU -- two stages of 256 features x 128 rows are 64 KiB
// of LDS (80 KiB with three parts) -- instead of one larger work-group with
// deeper stages: 4096 rows of O (7B) take 188 us launched alone (1460 TFLOP/s
// issued), 217 us in a prefill, against 262 and 265 us for one eight-wave 256 x
// 256 work-group of three stages.
//
// K is split over gridDim.z slices (kSplit) where the tiles alone leave the
// chip idle: each wave publishes its partial sums with agent-coherent stores
// and counts itself in, and the last slice's wave to arrive adds the partials
// in slice order -- bitwise reproducible -- and runs the epilogue (no work-
// group waits on another).  Cutting all tiles' K-blocks into one equal range
// per resident work-group instead, so that none idles, was 1.4 times slower:
// the work-groups of an XCD then read different K-blocks and share nothing in
// its L2.
struct TileSplit {
  float* part;    // [tile][slice][wave][tile fragment][64 lanes][4] floats
  int32_t* cnt;   // [tile][wave] arrived slices; zero between launches
};
template <int TN, int TM>
constexpr size_t tile_slice_floats() {  // floats a wave publishes per slice
  return static_cast<size_t>(TN / 2) * (TM / 2) * 256;
}

// LP: parts per K-block of the activation record (the first P::parts are used).
// Grid: (weight tiles / TN, row tiles / TM, K slices).
template <class P, int TN, int TM, int NST, bool kSplit, class Epi, int LP = P::parts>
__global__ __launch_bounds__(256, 2) void k_tile_gemm(const uint4* W, const uint4* X, int NT, int KB, int Rp,
                                                      TileSplit ts, Epi epi) {
  constexpr int PARTS = P::parts, NW = kTileWaves;
  static_assert(LP >= PARTS, "the record holds the parts used");
  constexpr int NFRAG = TN + TM * PARTS;
  constexpr int LW = TN / NW, L = (NFRAG + NW - 1) / NW;  // loads per wave per stage: weights, all
  static_assert(TN % NW == 0, "weight fragments split over the waves");
  constexpr int WN = TN / 2, WM = TM / 2;
  __shared__ uint4 lds[NST * NFRAG * 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave % 2, wm = wave / 2;
  // Work-groups go to the eight XCDs in turn (linear id mod 8), and each XCD
  // has its own L2.  XCD x takes the contiguous range of tiles from x * total
  // / 8 in an order that runs over groups of four row tiles, the row tile
  // fastest: the work-groups an XCD holds at a time then work on the same
  // K-blocks of neighbouring tiles and share both operands in its L2.  Without
  // groups every row tile reads the weights again: 15 row tiles of the 70B
  // shape (1833 rows, four layers) 24.0 ms, 21.3 in groups.
  int nt0, m0, tile;
  {
    const int total = gridDim.x * gridDim.y, b = blockIdx.y * gridDim.x + blockIdx.x;
    const int q = total / 8, r = total % 8, x = b % 8, j = b / 8;
    tile = x * q + min(x, r) + j;
    const int per_group = 4 * gridDim.x;
    const int mg = tile / per_group, rem = tile % per_group;
    const int gm = min(4, static_cast<int>(gridDim.y) - 4 * mg);  // the last group may be smaller
    nt0 = (rem / gm) * TN;
    m0 = (4 * mg + rem % gm) * TM * 16;
  }
  const int S = kSplit ? gridDim.z : 1, slice = kSplit ? blockIdx.z : 0;
  const int kb0 = KB * slice / S, kb1 = KB * (slice + 1) / S;
  // Loads: a running base each for weights and activations, and a 32-bit lane
  // offset per fragment (bytes).  A wave past the last fragment repeats it.
  const uint32_t xpart = static_cast<uint32_t>(Rp) * 64;  // bytes per (K-block, part)
  const char* wbase = reinterpret_cast<const char*>(W) + static_cast<size_t>(nt0) * KB * 1024;
  const char* xbase = reinterpret_cast<const char*>(X);
  auto act_frag = [&](int i) __attribute__((always_inline)) { return min(wave + NW * (i - LW), TM * PARTS - 1); };
  uint32_t off[L];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    if (i < LW) {
      off[i] = static_cast<uint32_t>(min(nt0 + wave + NW * i, NT - 1) - nt0) * KB * 1024 + lane * 16;
    } else {
      const int f = act_frag(i), q = f / TM, tt = f % TM;
      off[i] = q * xpart + min(m0 + 16 * tt, Rp - 16) * 64 + lane * 16;
    }
  }
  auto issue = [&](int kb, int stage) __attribute__((always_inline)) {
    const char* wk = wbase + static_cast<size_t>(kb) * 1024;
    const char* xk = xbase + static_cast<size_t>(kb) * LP * xpart;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int f = i < LW ? wave + NW * i : TN + act_frag(i);
      __builtin_amdgcn_global_load_lds((global_void*)((i < LW ? wk : xk) + off[i]),
                                       (lds_void*)(lds + (stage * NFRAG + f) * 64), 16, 0, 0);
    }
  };

  f32x4_t acc[WN][WM];
#pragma unroll
  for (int i = 0; i < WN; ++i)
#pragma unroll
    for (int j = 0; j < WM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const uint32_t abase = lds_address(lds + wn * WN * 64 + lane), bbase = lds_address(lds + (TN + wm * WM) * 64 + lane);
  auto multiply = [&](int stage) __attribute__((always_inline)) {
    // The weight fragments, then row tile by row tile the activation
    // fragments, one row tile ahead of the products.
    const uint32_t ab = abase + stage * (NFRAG * 1024), bb = bbase + stage * (NFRAG * 1024);
    u32x4_t a[WN], b[2][PARTS];
    auto read_a = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      a[i] = lds_read16_at<i * 1024>(ab);
    };
    auto read_b = [&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value;
      auto part = [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        b[j & 1][q] = lds_read16_at<(q * TM + j) * 1024>(bb);
      };
      static_for<PARTS>(part);
    };
    read_b(std::integral_constant<int, 0>{});
    static_for<WN>(read_a);
    auto row_tile = [&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value;
      if constexpr (j + 1 < WM) {
        read_b(std::integral_constant<int, j + 1>{});
        lds_reads_left<PARTS>();
      } else {
        lds_reads_left<0>();
      }
      if constexpr (j == 0) {
#pragma unroll
        for (int i = 0; i < WN; ++i) lds_value_ready(a[i]);
      }
#pragma unroll
      for (int q = 0; q < PARTS; ++q) lds_value_ready(b[j & 1][q]);
#pragma unroll
      for (int q = 0; q < PARTS; ++q)
#pragma unroll
        for (int i = 0; i < WN; ++i)
          acc[i][j] = P::mma(acc[i][j], __builtin_bit_cast(uint4, a[i]), __builtin_bit_cast(uint4, b[j & 1][q]));
      // Keep these products ahead of the next tile's wait (the scheduler
      // would otherwise sink them below it).
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<WM>(row_tile);
  };

  // K-block kb (LDS stage st): its loads are the oldest in flight; the next
  // NST - 2 K-blocks' (if any) may stay in flight.  Then the stage read at
  // kb - 1 is free for kb + NST - 1.
  auto step = [&](int kb, int st, int free_st) __attribute__((always_inline)) {
    if (kb + NST - 2 < kb1) {
      wait_vmem<(NST - 2) * L>();
    } else {  // the last K-blocks: fewer loads in flight
      wait_vmem<0>();
    }
    lds_stage_barrier();
    if (kb + NST - 1 < kb1) issue(kb + NST - 1, free_st);
    multiply(st);
  };
#pragma unroll
  for (int k = 0; k < NST - 1; ++k)
    if (kb0 + k < kb1) issue(kb0 + k, k);
  for (int kb = kb0; kb < kb1; kb += NST) {
    auto one = [&](auto sc) __attribute__((always_inline)) {
      constexpr int st = decltype(sc)::value;
      if (kb + st < kb1) step(kb + st, st, (st + NST - 1) % NST);
    };
    static_for<NST>(one);
  }
  if constexpr (kSplit) {
    constexpr uint32_t kWave = tile_slice_floats<TN, TM>() * sizeof(float);  // bytes of a wave's slice
    const CoherentBuffer buf(ts.part + static_cast<size_t>(tile) * S * NW * (kWave / 4), S * NW * kWave);
    auto at = [&](int q, int i) __attribute__((always_inline)) {
      return static_cast<uint32_t>((q * NW + wave) * kWave + i * 1024 + lane * 16);
    };
#pragma unroll
    for (int i = 0; i < WN * WM; ++i) buf.store4(at(slice, i), acc[i / WM][i % WM]);
    wait_vmem<0>();  // this wave's partial sums are complete
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    int32_t* cnt = ts.cnt + tile * NW + wave;
    int last = 0;
    if (lane == 0) last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == S - 1;
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    if (lane == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    for (int q = 0; q < S; ++q) {
#pragma unroll
      for (int i = 0; i < WN * WM; ++i) {
        const f32x4_t v = buf.load4(at(q, i));
        if (q == 0) {
          acc[i / WM][i % WM] = v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i / WM][i % WM][e] += v[e];
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < WN; ++i) {
    const int nt = nt0 + wn * WN + i;
    if (nt >= NT) continue;
#pragma unroll
    for (int j = 0; j < WM; ++j) epi.apply_tile(nt, m0 + 16 * (wm * WM + j), acc[i][j], lane);
  }
}

// QKV epilogue: RMSNorm scale, RoPE on q and k, q to the attention input,
// k and v appended to the paged KV cache (same tile orders as decode).
template <class P, class KP = P>
struct EpiQKVRows {
  int M, H, Hkv, hd, mb;
  int nt_base;                    // weight tile of the launch's tile 0 (the launch may cover part of QKV)
  float* q;                       // [rows][H * hd]
  typename KP::elem* kc;
  typename KP::elem* vc;
  const int32_t* bt;
  const float2* rope;
  const PrefillRow* rows;
  const float* rs;

  __device__ __forceinline__ void apply_tile(int nt, int m0, const f32x4_t& acc, int lane) const {
    const int b = m0 + (lane & 15);
    if (b >= M) return;
    const int n0 = 16 * (nt_base + nt) + 4 * (lane >> 4);
    const int qr = H * hd, kr = Hkv * hd;
    const float s = rs[b];
    float v0 = acc[0] * s, v1 = acc[1] * s, v2 = acc[2] * s, v3 = acc[3] * s;
    const PrefillRow row = rows[b];
    const int p = row.pos;
    if (n0 < qr + kr) {
      const int dd = (n0 < qr ? n0 : n0 - qr) % hd;
      const float4 cs = *reinterpret_cast<const float4*>(rope + static_cast<size_t>(p) * (hd / 2) + dd / 2);
      const float a0 = v0 * cs.x - v1 * cs.y, a1 = v0 * cs.y + v1 * cs.x;
      const float a2 = v2 * cs.z - v3 * cs.w, a3 = v2 * cs.w + v3 * cs.z;
      v0 = a0;
      v1 = a1;
      v2 = a2;
      v3 = a3;
    }
    if (n0 < qr) {
      *reinterpret_cast<float4*>(q + static_cast<size_t>(b) * qr + n0) = make_float4(v0, v1, v2, v3);
      return;
    }
    const int blk = bt[static_cast<size_t>(row.slot) * mb + (p >> 4)];
    const int off = p & 15;
    if (n0 < qr + kr) {
      const int m = n0 - qr, kvh = m / hd, dd = m % hd;
      typename KP::elem* dst = kc + (static_cast<size_t>(blk) * Hkv + kvh) * 16 * hd + ktile_offset<KP>(off, dd);
      dst[0] = KP::from_f32(v0);
      dst[1] = KP::from_f32(v1);
      dst[2] = KP::from_f32(v2);
      dst[3] = KP::from_f32(v3);
    } else {
      const int m = n0 - qr - kr, kvh = m / hd, dd = m % hd;
      typename KP::elem* dst = vc + (static_cast<size_t>(blk) * Hkv + kvh) * 16 * hd;
      dst[vtile_offset<KP>(off, dd)] = KP::from_f32(v0);
      dst[vtile_offset<KP>(off, dd + 1)] = KP::from_f32(v1);
      dst[vtile_offset<KP>(off, dd + 2)] = KP::from_f32(v2);
      dst[vtile_offset<KP>(off, dd + 3)] = KP::from_f32(v3);
    }
  }
};

// O and down projections: residual add, new residual as the next activation.
template <class P>
struct EpiResidRows {
  int M, d;
  ActRec rec;
  float* x;
  typename P::elem* act;

  __device__ __forceinline__ void apply_tile(int nt, int m0, const f32x4_t& acc, int lane) const {
    const int b = m0 + (lane & 15);
    if (b >= M) return;
    const int n0 = 16 * nt + 4 * (lane >> 4);
    float4* xp = reinterpret_cast<float4*>(x + static_cast<size_t>(b) * d + n0);
    float4 xv = *xp;
    xv.x += acc[0];
    xv.y += acc[1];
    xv.z += acc[2];
    xv.w += acc[3];
    *xp = xv;
    store_act4<P>(act, rec, b, n0, xv.x, xv.y, xv.z, xv.w);
  }
};

// Gate/up (interleaved rows): RMSNorm scale, h = SiLU(gate) * up.
template <class P>
struct EpiSwiGLURows {
  int M;
  ActRec rec;
  const float* rs;
  typename P::elem* act;

  __device__ __forceinline__ void apply_tile(int nt, int m0, const f32x4_t& acc, int lane) const {
    const int b = m0 + (lane & 15);
    if (b >= M) return;
    const int j0 = 8 * nt + 2 * (lane >> 4);
    const float s = rs[b];
    const float g0 = acc[0] * s, g1 = acc[1] * s, u0 = acc[2] * s, u1 = acc[3] * s;
    const float h[2] = {g0 / (1.f + __expf(-g0)) * u0, g1 / (1.f + __expf(-g1)) * u1};
    act_store<P, 2>(act, rec, b, j0, h);
  }
};

// Causal attention over each query tile's own request.  Work-group (tile of
// up to 64 consecutive rows of one request, query head): wave w owns rows
// 16 w .. 16 w + 15 as its 16 MFMA columns.  The work-group walks the KV blocks
// up to the tile's last position once.  Each block's K and V tiles come from
// global memory once, straight into LDS, and all four waves multiply their
// columns against them; the next block's loads are in flight while the
// current one is used (two LDS buffers, two barriers per block).  Sharing a
// block among 64 queries instead of 16 cuts the cache reads that bound this
// kernel fourfold.  A wave skips blocks that start after its last position;
// block 0 holds position 0, so every column's running maximum is finite after
// it.  Columns past the tile's rows repeat its last row and are not stored.
template <class P, class AP, int HD>
__global__ __launch_bounds__(256) void k_attn_prefill(const float* __restrict__ q, const void* kcv, const void* vcv,
                                                      const int32_t* __restrict__ bt,
                                                      const PrefillTile* __restrict__ tiles, void* actv, int H,
                                                      int Hkv, int mb, ActRec rec, float qscale) {
  using E = typename P::elem;
  using Blk = KVBlock<P, HD>;
  constexpr bool kBf16 = sizeof(E) == 2;
  constexpr int NF = Blk::NF, NV = Blk::NV;
  constexpr int NE = HD / 16;
  constexpr int KU = NF * 64, KVU = (NF + NV) * 64;  // uint4 of a block's K tile, of its K and V tiles
  constexpr int PER = KVU / 256;                     // uint4 each thread stages per block
  static_assert(KVU % 256 == 0, "a block's K and V tiles split evenly over the work-group");
  __shared__ uint4 skv[2][KVU];
  // Heads fastest, so that every XCD takes all of the tiles (their lengths
  // differ), and the tiles in reverse: of each prompt the last, whose walk is
  // longest, first.  Where H is a multiple of 8, an XCD takes H / 8 consecutive heads:
  // the heads of a KV group share its L2.  (1500 positions of the 70B shape, 4
  // layers: 17.5 ms against 18.3 ms tiles fastest, where the XCD of the last
  // tiles walked 1.3 times the mean.)
  const PrefillTile tile = tiles[gridDim.y - 1 - blockIdx.y];
  const int hx = blockIdx.x, hq = H % 8 == 0 ? (hx % 8) * (H / 8) + hx / 8 : hx, kvh = hq / (H / Hkv);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int r0 = 16 * wave;                            // the wave's first row of the tile
  const int rw = min(16, tile.n - r0);                 // its rows (none if <= 0)
  const int cq = rw > 0 ? r0 + (c < rw ? c : rw - 1) : tile.n - 1;
  const int pc = tile.pos0 + cq;                       // this column's position
  const int wave_last = tile.pos0 + (rw > 0 ? r0 + rw - 1 : 0);
  const int max_pos = tile.pos0 + tile.n - 1;
  const int nblk = (max_pos >> 4) + 1;
  const int32_t* btrow = bt + static_cast<size_t>(tile.slot) * mb;
  const E* kc = static_cast<const E*>(kcv);
  const E* vc = static_cast<const E*>(vcv);
  int ids = lane < nblk ? btrow[lane] : 0;             // block ids of blocks [i0, i0 + 64)

  // Block i's K and V tiles, straight from global memory into LDS buffer buf
  // (global_load_lds; no registers), thread t moving uint4 t, t + 256, ...
  // The block's id is lane (i mod 64) of ids.
  auto issue = [&](int i, int buf) __attribute__((always_inline)) {
    const int blk = __builtin_amdgcn_readlane(ids, i & 63);
    const size_t off = (static_cast<size_t>(blk) * Hkv + kvh) * 16 * HD;
    const uint4* kt = reinterpret_cast<const uint4*>(kc + off);
    const uint4* vt = reinterpret_cast<const uint4*>(vc + off);
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int idx = tid + 256 * p;
      const uint4* src = idx < KU ? kt + idx : vt + (idx - KU);
      __builtin_amdgcn_global_load_lds((global_void*)src, (lds_void*)&skv[buf][256 * p + 64 * wave], 16, 0, 0);
    }
  };

  uint4 qh[NF], ql[NF];
  {
    const float* qp = q + (static_cast<size_t>(tile.row0 + cq) * H + hq) * HD + g * P::per16;
    float4 qv[NF][P::per16 / 4];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int j4 = 0; j4 < P::per16 / 4; ++j4) qv[f][j4] = *reinterpret_cast<const float4*>(qp + f * P::kblk + 4 * j4);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      union {
        uint4 u;
        E e[P::per16];
      } vh, vl;
#pragma unroll
      for (int j = 0; j < P::per16; ++j) {
        const float4 t = qv[f][j / 4];
        const float v = (j % 4 == 0 ? t.x : j % 4 == 1 ? t.y : j % 4 == 2 ? t.z : t.w) * qscale;
        vh.e[j] = P::from_f32(v);
        vl.e[j] = P::from_f32(v - P::to_f32(vh.e[j]));
      }
      qh[f] = vh.u;
      ql[f] = vl.u;
    }
  }

  f32x4_t O[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) O[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  issue(0, 0);
  for (int i = 0; i < nblk; ++i) {
    const int cur = i & 1;
    // The next block goes into the other buffer, which every wave finished
    // reading before the previous block's closing barrier.
    if (i + 1 < nblk) {
      if (((i + 1) & 63) == 0) ids = i + 1 + lane < nblk ? btrow[i + 1 + lane] : 0;
      issue(i + 1, cur ^ 1);
      wait_vmem<PER>();  // this thread's loads of block i have landed
    } else {
      wait_vmem<0>();
    }
    lds_stage_barrier();  // every thread's loads of block i have landed
    if (rw > 0 && i * 16 <= wave_last) {  // wave-uniform: the block has keys some column sees
      Blk B;
      u32x4_t kr[NF], vr[NV];
#pragma unroll
      for (int f = 0; f < NF; ++f) kr[f] = lds_read16(&skv[cur][f * 64 + lane]);
#pragma unroll
      for (int v = 0; v < NV; ++v) vr[v] = lds_read16(&skv[cur][KU + v * 64 + lane]);
      lds_reads_done();
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        lds_value_ready(kr[f]);
        B.kf[f] = __builtin_bit_cast(uint4, kr[f]);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        lds_value_ready(vr[v]);
        B.vf[v] = __builtin_bit_cast(uint4, vr[v]);
      }
      f32x4_t S = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        S = P::mma(S, B.kf[f], qh[f]);
        if constexpr (kBf16) S = P::mma(S, B.kf[f], ql[f]);
      }
      if (i * 16 + 15 > tile.pos0 + r0) {  // block reaches past the wave's first position: causal mask
        const int valid = pc - (i * 16 + 4 * g) + 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) S[r] = r < valid ? S[r] : -INFINITY;
      }
      if (i == nblk - 1) B.mask_v(max_pos - (i * 16 + 4 * g) + 1);
      float mb2 = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3]));
      mb2 = fmaxf(mb2, __shfl_xor(mb2, 16));
      mb2 = fmaxf(mb2, __shfl_xor(mb2, 32));
      const float m_new = fmaxf(m_run, mb2);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
      float p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(S[r] - m_use);
      l_run = l_run * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
      if (i != 0 && __ballot(m_new != m_run) != 0) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          O[e][0] *= alpha;
          O[e][1] *= alpha;
          O[e][2] *= alpha;
          O[e][3] *= alpha;
        }
      }
      m_run = m_new;
      B.pv(O, p);
    }
    lds_stage_barrier();  // buffer cur is free for block i + 2
  }
  if (rw <= 0) return;
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (c >= rw) return;
  const float inv = 1.f / l_run;
  typename AP::elem* act = static_cast<typename AP::elem*>(actv);
#pragma unroll
  for (int e = 0; e < NE; ++e)
    store_act4<AP>(act, rec, tile.row0 + r0 + c, hq * HD + 16 * e + 4 * g, O[e][0] * inv, O[e][1] * inv,
                   O[e][2] * inv, O[e][3] * inv);
}

// Rows src[k] of the residual as rows k of an activation record (Rp rows),
// for the LM head of the rows that emit a token.
struct GatherArgs {
  const float* x;
  void* act;
  int d, n;
  ActRec rec;
  int src[kRows];
};
template <class P>
__global__ __launch_bounds__(64) void k_gather_rows(GatherArgs a) {
  const int k = blockIdx.y;
  const int n0 = 4 * (blockIdx.x * 64 + threadIdx.x);
  if (n0 >= a.d || k >= a.n) return;
  const float4 v = *reinterpret_cast<const float4*>(a.x + static_cast<size_t>(a.src[k]) * a.d + n0);
  store_resid4<P>(static_cast<typename P::elem*>(a.act), a.rec, k, n0, a.d, v);
}

}  // namespace sprk
