// Device helpers of the BF16 MFMA GEMMs whose operand tiles go straight from
// global memory into LDS (k_pose.hip, k_cnn.hip).
//
// An operand tile is R rows x 64 k of bfloat16, row after row (128 bytes per
// row, no padding: a wave's load writes 64 x 16 consecutive bytes of LDS).  So
// that the fragment reads of 16 lanes (16 rows, one 16-byte chunk of each) do
// not meet in the same banks, chunk c of row r lies at slot c ^ (r & 7); the
// permutation is applied to the global addresses of the loads.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cs {

typedef __attribute__((__vector_size__(8 * sizeof(short)))) short mma_bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float mma_f32x4;

constexpr int kMmaK = 64;  // K staged per step: two v_mfma_f32_16x16x32_bf16

// 16 bytes per lane from `src` (any address, 16-byte aligned) to `dst` + 16 x
// lane in LDS; `dst` is the same for the whole wave.
__device__ __forceinline__ void dma16(const void *src, void *dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                   (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// Every load of this wave has arrived (the tiles it staged are in LDS).
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Nothing is scheduled across this point.
__device__ __forceinline__ void mma_order() { __builtin_amdgcn_sched_barrier(0); }

// 16-byte piece e = row * 8 + slot of a tile: which chunk of the row it holds.
__device__ __forceinline__ int mma_chunk(int e) { return (e & 7) ^ ((e >> 3) & 7); }

// Fragment of MFMA k-slice ks (0, 1) for tile row `row`: the 8 values at
// k = 32 ks + 8 (lane >> 4).
__device__ __forceinline__ mma_bf16x8 mma_frag(const unsigned short *tile, int row, int ks, int lane) {
  const int c = (ks * 4 + (lane >> 4)) ^ (row & 7);
  return *(const mma_bf16x8 *)(tile + row * kMmaK + c * 8);
}

}  // namespace cs
