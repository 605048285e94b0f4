// Device helpers shared by the attention kernels.
#pragma once

#include "common.h"

namespace tu {

namespace {

constexpr float kTau = 8.f;  // lazy-rescale threshold (log2 units): P < 2^8 fits f16

typedef __attribute__((address_space(3))) void lds_void;

// s_waitcnt immediate that waits on the vector-memory counter only
constexpr int vm_wait(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// Fourth word of a raw buffer resource (32-bit data, no swizzle) on CDNA
constexpr int kBufWord3 = 0x00020000;

// Copies 16 bytes per lane from base + voff + soff to LDS (lane i writes lds + 16 i).
// The resource covers `bytes` from base; lanes past it write zeros. base and bytes are
// wave-uniform; reading them through readfirstlane lets the compiler see that, so the
// resource stays in scalar registers (no per-lane loop around the load).
__device__ __forceinline__ void dma16(const void* base, int bytes, uint32_t voff, uint32_t soff, void* lds) {
  const uint64_t b = (uint64_t)base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  void* ub = (void*)(((uint64_t)hi << 32) | lo);
  const __amdgpu_buffer_rsrc_t res =
      __builtin_amdgcn_make_buffer_rsrc(ub, 0, __builtin_amdgcn_readfirstlane(bytes), kBufWord3);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(res, (lds_void*)lds, 16, voff, soff, 0, 0);
}

// Scales an MFMA accumulator (the rare move of the softmax reference max).
__device__ __forceinline__ void scale_acc(f32x16& acc, float s) {
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] *= s;
}

}  // namespace

}  // namespace tu
