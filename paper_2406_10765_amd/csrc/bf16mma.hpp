// Device helpers shared by the split-bf16 GEMMs (gemm16.hip, gemm_pairs.hip): MFMA 16x16x32 bf16,
// the LDS chunk layout of K-contiguous tiles, and the direct global-to-LDS loads of gfx950.
#pragma once

#include <hip/hip_runtime.h>

#include "bf16split.hpp"
#include "pipe_addr.hpp"

namespace pw {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f16 __attribute__((ext_vector_type(4)));

constexpr int hBK = 16;       // complex K per tile = 32 real k' = one MFMA slab
constexpr int hFlush = 256;   // K tiles (4096 complex K) per fp32 MFMA accumulation before fp64
constexpr int hXcd = 8;
__device__ __forceinline__ int chunk_of(int row, int slot) {
  return (((row >> 4) << 2) + slot) * 16 + ((row & 15) ^ slot);
}

__device__ __forceinline__ int xcd_tile16(int w, int total) {
  const int per = total / hXcd, rem = total % hXcd;
  const int x = w % hXcd, i = w / hXcd;
  return x < rem ? x * (per + 1) + i : rem * (per + 1) + (x - rem) * per + i;
}

__device__ __forceinline__ v4f16 mma16(v8bf a, v8bf b, v4f16 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Fragment of rows row0..row0+15 (row0 a multiple of 16): lane l reads chunk (row0 + l % 16, l / 16).
__device__ __forceinline__ v8bf frag(const uint4* plane, int row0, int lane) {
  const int slot = lane >> 4, i = lane & 15;
  return __builtin_bit_cast(v8bf, plane[((row0 >> 4) << 6) + slot * 16 + (i ^ slot)]);
}

__device__ __forceinline__ void dma16(const unsigned int* g, void* l) {
  __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
}
// s_waitcnt vmcnt(N) alone (expcnt and lgkmcnt left at their maxima)
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xc07f); }  // lgkmcnt(0)

// Address of the 16 bytes a lane loads: a wave-uniform base plus a per-lane 32-bit byte offset.
__device__ __forceinline__ const unsigned int* at_off(const unsigned int* base, unsigned int byte_off) {
  return reinterpret_cast<const unsigned int*>(reinterpret_cast<const unsigned char*>(base) + byte_off);
}

}  // namespace pw
