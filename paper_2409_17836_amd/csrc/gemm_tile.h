// Pieces the bf16 matrix kernels share: operand types, the workgroup -> tile
// order and buffer resources.
#pragma once

#include "epilogue.h"

namespace lmgc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int kXcds = 8;

// s_waitcnt immediate: vmcnt(n) with expcnt and lgkmcnt at their maxima (vmcnt
// bits 3:0 and 15:14)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0xF70; }

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Tile of workgroup bid: each XCD (bid % 8) walks a contiguous range of the
// tiles in an order grouped by GM row tiles.
template <int GM>
__device__ inline bool map_tile(int bid, int nblocks, int ntm, int ntn, int& tm, int& tn) {
  const int total = ntm * ntn;
  const int per = nblocks / kXcds;  // nblocks is a multiple of kXcds
  const int t = (bid % kXcds) * per + bid / kXcds;
  if (t >= total) return false;
  const int in_group = GM * ntn;
  const int g = t / in_group;
  const int first = g * GM;
  const int gs = min(ntm - first, GM);
  const int r = t - g * in_group;
  tm = first + r % gs;
  tn = r / gs;
  return true;
}

// Raw buffer resource (gfx9 layout: stride 0, dword 3 = 0x00020000) over
// `bytes` bytes at p; loads at offsets >= bytes return zero.
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, 0x00020000);
}

}  // namespace lmgc
