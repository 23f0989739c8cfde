// Shared declarations of the gfx950 clustered sparse-attention library (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/adacluster.h"

namespace adac {

typedef uint16_t bf16raw;   // storage of one bfloat16

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_t;

__device__ __forceinline__ float bf16_to_f32(bf16raw v) { return __uint_as_float(((uint32_t)v) << 16); }

// round-to-nearest-even fp32 -> bf16 (inputs here are finite)
__device__ __forceinline__ bf16raw f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16raw)(u >> 16);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2_t x = {lo, hi};
  bf16x2_t y = __builtin_convertvector(x, bf16x2_t);
  return *reinterpret_cast<uint32_t*>(&y);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float load(const float* p) { return *p; }
};
template <> struct Elem<bf16raw> {
  static __device__ __forceinline__ float load(const bf16raw* p) { return bf16_to_f32(*p); }
};

// Direct global -> LDS loads, written as inline assembly on purpose.  The compiler orders every LDS read
// behind an outstanding direct-to-LDS load that it cannot prove to touch another object (it then drains ALL
// loads in flight: vmcnt(0)), and its proof is fragile (it fails across the branches of a four-stage ring).
// The tile pipelines keep several tiles in flight and wait for exactly the one they need, by count,
// before a workgroup barrier; hiding the loads from the compiler leaves that protocol in charge.  Each lane
// loads `bytes` at sbase + voff; the wave's data land at lds_addr + lane * bytes (M0 carries the LDS address).
__device__ __forceinline__ void dma_b128(uint32_t lds_addr, uint32_t voff, const void* sbase) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(sbase) : "memory", "m0");
}
__device__ __forceinline__ void dma_b128(uint32_t lds_addr, const void* src) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ void dma_b32(uint32_t lds_addr, uint32_t voff, const void* sbase) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(sbase) : "memory", "m0");
}

// s_waitcnt with only the vector-memory counter set (gfx9 encoding: vmcnt[3:0] and [15:14])
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() carries a release fence over global memory
// as well, which makes every wave drain all of its loads in flight (vmcnt(0)) at every barrier; kernels
// that wait for exactly the loads they need by count, or for none of their stores, use this one.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // this wave's LDS reads and writes are done
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");                         // nothing that touches memory moves across
}

// per-head state of the multi-stage key clustering (Algorithm 1), device resident
struct KState {
  int32_t ucount;      // |U|
  int32_t ccount;      // |C| so far
  int32_t m_t;         // centres of the running stage
  int32_t stage;       // t
  int32_t done;        // the stage loop has ended for this head
  int32_t full;        // F
  int32_t active;      // this stage runs (set by stage_open)
  int32_t pad;
  int32_t stage_offs[ADACLUSTER_MAX_STAGES + 1];
  int32_t u_hist[ADACLUSTER_MAX_STAGES + 1];   // |U| at the head of stage t; entry `stage` = what staging left over
};

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

}  // namespace adac
