// Direct global-to-LDS loads and their waits: the pieces that the pipelined
// kernels share.
#pragma once

#include <utility>

#include "device_common.h"

namespace sprk {

typedef __attribute__((address_space(1))) void global_void;
typedef __attribute__((address_space(3))) void lds_void;

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// Waits until at most N vector-memory operations of this wave are in flight
// (expcnt and lgkmcnt not waited on).
template <int N>
__device__ __forceinline__ void wait_vmem() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// 16-byte LDS read issued as plain ds_read_b128.  The compiler treats LDS
// that global_load_lds fills as possibly still in flight and, at loop
// back-edges, would wait for every load in flight (vmcnt(0)) before any LDS
// read; the kernel's own vmcnt wait plus barrier already orders the read, so
// the read bypasses that tracking.  The caller waits with lds_reads_done()
// before using the results.
__device__ __forceinline__ u32x4_t lds_read16(const uint4* p) {
  u32x4_t v;
  const uint32_t a = static_cast<uint32_t>(reinterpret_cast<size_t>((lds_void*)p));
  asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(a));
  return v;
}
// The same read at LDS byte address `addr` + OFF: one address register serves
// all reads of a stage (with an address each, the compiler keeps them all in
// registers across the loop).
__device__ __forceinline__ uint32_t lds_address(const uint4* p) {
  return static_cast<uint32_t>(reinterpret_cast<size_t>((lds_void*)p));
}
template <int OFF>
__device__ __forceinline__ u32x4_t lds_read16_at(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds_read offset range");
  u32x4_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Calls f(std::integral_constant<int, j>) for j = 0 .. N - 1 in order.
template <class F, int... J>
__device__ __forceinline__ void static_for_seq(F& f, std::integer_sequence<int, J...>) {
  (f(std::integral_constant<int, J>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// Waits until at most N of this wave's LDS reads are in flight (they return
// in issue order, so every read but the last N has landed).
template <int N>
__device__ __forceinline__ void lds_reads_left() {
  static_assert(N >= 0 && N < 16, "lgkmcnt range");
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
// Ties a value read by lds_read16 to a point after lds_reads_done(): volatile
// asm statements keep their order, so no use of v can move above the wait.
__device__ __forceinline__ void lds_value_ready(u32x4_t& v) { asm volatile("" : "+v"(v)); }

// Work-group barrier for LDS filled by global_load_lds: each wave first waits
// for its own loads (vmcnt), so after the barrier every wave's fragments of
// that stage are in LDS.  No memory fence: a workgroup fence here would wait
// for every load in flight (vmcnt(0)), including the stages being prefetched.
// The empty asm statements keep the compiler from moving LDS accesses across.
__device__ __forceinline__ void lds_stage_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace sprk
