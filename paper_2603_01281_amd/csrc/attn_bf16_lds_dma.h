// Tile transport of the direct-to-LDS kernels (gfx950):
//   * K/V tiles (64 keys) go from global memory straight into LDS with global_load_lds
//     (16 bytes per lane, no register staging), two tiles ahead of the math, into rings of three
//     stages.  Completion is tracked with an explicit vmcnt wait followed by the per-tile barrier.
//   * A direct-to-LDS load writes 64 lanes x 16 bytes contiguously, so rows cannot be padded; bank
//     conflicts are avoided by choosing WHICH 16-byte chunk of a row each lane fetches (an XOR
//     swizzle of the chunk index with the row index; see pipe_k_swizzle / pipe_v_swizzle).
#pragma once
#include "common.h"

namespace seka {

constexpr int DMA_BK = 64;                       // keys per tile
constexpr int DMA_STAGES = 3;

typedef __attribute__((address_space(3))) s16x4* dma_lds_s16x4_ptr;
typedef __attribute__((address_space(3))) void* dma_lds_void_ptr;

template <int N>
__device__ __forceinline__ void dma_wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Workgroup barrier that waits for this wave's LDS traffic only.  (__syncthreads() would also drain
// every outstanding vector-memory operation, i.e. the tile loads that are meant to stay in flight.)
__device__ __forceinline__ void dma_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

}  // namespace seka
