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

// Direct-to-LDS load with a scalar 64-bit base and a 32-bit per-lane byte offset: the wave's 64 x 16 bytes land contiguously at
// the (wave-uniform) LDS byte address.  Inline assembly keeps it outside the compiler's own vmcnt bookkeeping (the waits
// are placed by hand) and outside its wait states: such a load needs one between it and the write of m0, and five between it
// and a vector instruction that wrote its base (a spilled base comes back by v_readlane).  The copy of the base is the
// first, and lifts the second: the hardware itself waits where a scalar instruction reads or writes.
__device__ __forceinline__ void dma_load_16B(const void* base, uint32_t lane_off, uint32_t lds) {
  const void* copy;
  asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0"
               : "=&s"(copy) : "s"(lds), "v"(lane_off), "s"(base) : "memory", "m0");
}

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
