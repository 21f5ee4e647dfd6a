// device.h -- device helpers shared by the matrix-core kernels of
// libmoesplit: MFMA operands, direct global -> LDS loads with hand-placed
// waits, and LDS fragment reads (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace msk {

// v_mfma_f32_16x16x32_bf16: lane l holds A[row l%16][8 k from 8*(l/16)],
// B[8 k from 8*(l/16)][column l%16] and the result C[rows 4*(l/16)+r][column
// l%16].  The k order inside a step is the same for A and B, which is all
// the contraction needs.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

__device__ __forceinline__ f32x4_t mfma16(bf16x8_t a, bf16x8_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Work-groups are dispatched to the 8 XCDs round-robin by index, and each
// XCD has its own L2.  The matrix-core kernels renumber them so that every
// XCD runs a contiguous range of logical indices.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_local(int wg, int n) {
  const int q = n / kXcds, r = n % kXcds;
  const int x = wg % kXcds, i = wg / kXcds;
  return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// 16 bytes per lane from global memory to LDS byte address lds + 16 lane
// (lds uniform over the wave); M0 is restored for the compiler.  A load into
// LDS needs one wait state after a scalar write of M0, which the hardware does
// not insert and the compiler does not look for inside inline asm.
__device__ __forceinline__ void lds_load16(const void* g, uint32_t lds) {
  uint32_t keep;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(keep)
      : "v"(g), "s"(lds)
      : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)(p)));
}

// wait until at most N of this wave's vector memory loads are in flight
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// barrier without a memory fence (a fence would wait for every load in
// flight into LDS): this wave's LDS reads are complete first, and the
// clobber keeps the compiler from moving LDS accesses across it
__device__ __forceinline__ void bare_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ bf16x8_t lds_frag(const unsigned char* p) {
  return as_bf16x8(*reinterpret_cast<const uint4*>(p));
}

typedef short v4i16_t __attribute__((ext_vector_type(4)));

// Transposing read at LDS byte address p (ds_read_b64_tr_b16): in each
// 16-lane group, lanes 4 r .. 4 r + 3 give row r of a 4 x 16 tile of 16-bit
// values and lane i receives its column i.
__device__ __forceinline__ v4i16_t lds_read_tr16(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16_t*)((const __attribute__((address_space(3))) unsigned char*)(p)));
}

}  // namespace msk
