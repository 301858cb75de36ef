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

// Operand source of direct loads: 32-bit byte offsets from `base` (on a 16-byte
// boundary) below `bytes`; a load at or past the end puts zeros into LDS.
typedef __amdgpu_buffer_rsrc_t DmaSrc;
constexpr unsigned kDmaMax = 0x7fffff00u;   // longest source
constexpr unsigned kDmaZero = 0x80000000u;  // an offset past the end of any source
__device__ __forceinline__ DmaSrc dma_src(const void *base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)(bytes < kDmaMax ? bytes : kDmaMax), 0x00020000);
}

// 16 bytes per lane from byte `off` (a multiple of 16) of `src` to `dst` + 16 x
// lane in LDS; `dst` is the same for the whole wave.  (A buffer load: the
// compiler counts it exactly, while a global load to LDS makes it wait for
// every load and LDS read in flight.)
__device__ __forceinline__ void dma16(DmaSrc src, unsigned off, void *dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void *)dst, 16, (int)off, 0, 0, 0);
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

// The same for tiles of 32 k (64 bytes per row): chunk c of row r lies at slot
// c ^ ((r >> 2) & 3).
__device__ __forceinline__ int mma_chunk32(int e) { return (e & 3) ^ ((e >> 4) & 3); }
__device__ __forceinline__ mma_bf16x8 mma_frag32(const unsigned short *tile, int row, int lane) {
  const int c = (lane >> 4) ^ ((row >> 2) & 3);
  return *(const mma_bf16x8 *)(tile + row * 32 + c * 8);
}

// Block-wide: every wave's loads but its N youngest have arrived, and every
// wave's LDS reads are done.  Unlike __syncthreads() the younger loads stay
// in flight.
template <int N>
__device__ __forceinline__ void dma_wait_but() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace cs
