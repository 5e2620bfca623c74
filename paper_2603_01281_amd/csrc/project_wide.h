// Query projection in 256 x 256 tiles: Q[t, n] = sum_e X[t, e] W[n, e], bf16 in, fp32 accumulate, bf16 out, with the
// routing sums of its outputs (project_tile.h has the smaller tiles, for sizes whose 256 x 256 ones would leave the chip
// idle).
//
// What bounds it: the matrix pipe under the chip's power limit, and the LDS reads beside it.  A 64-wide slice of E is 2048
// cycles of MFMA per SIMD, 1536 cycles of LDS operand reads and 512 of tile writes.  The products are
// v_mfma_f32_16x16x32_bf16: an MFMA of that shape reads and writes half as much accumulator per multiply-add as
// v_mfma_f32_32x32x16_bf16, and alone, on random operands, the chip sustains 1.95 PFLOP/s of it against 1.76 (mfma_rate_probe.hip; the clock is
// what gives; nothing else changes, operand bytes and register counts are the same).  Eight waves as 2 x 4; a wave owns 64 x 32 outputs in each
// of the four quadrants of the tile (128 tokens x 128 features), so that operands of one half are kept in registers
// for two quadrants.  The schedule is the eight-wave ping-pong that is published for CDNA matrix products (HipKittens,
// 2025): two groups of waves half a step apart, half tiles requested ahead.  A slice is four phases, one quadrant each;
// a phase is a memory part (the operands that the phase adds, one half tile requested) and a matrix part (8 MFMAs)
// between barriers, and waves 4-7 run one part behind waves 0-3: on every SIMD one wave multiplies while the other
// reads.
//
//   phase   reads (16 bytes per lane)      requests             quadrant (A half, B half)
//     0     A half 0 of slice k:     8     B half 1 of k + 1      (0, 0)
//     1     B half 1 of slice k:     4     A half 1 of k + 1      (0, 1)
//     2     A half 1 of slice k:     8     A half 0 of k + 2      (1, 1)
//     3     B half 0 of slice k + 1: 4     B half 0 of k + 2      (1, 0)
//
// Half tiles (128 rows x 64 elements, 16 KB) travel straight into LDS, two 1 KB loads per wave, whole 128-byte lines;
// the 16-byte chunks of a row are swizzled (chunk ^ (row / 2) % 8) for conflict-free operand reads.  Slices k and
// k + 1 have a buffer each (128 KB).  A half is overwritten two phases or more after its last read, so both groups
// of waves are done with it, and it is requested four to six phases before it is read.  The loads return in order:
// before the barrier that a read relies on, every wave waits until only the requests after that half are left.
//
// Measured at 32768 tokens, E = 4096, N = 4096 with the routing sums: 759 us (1449 TFLOP/s), 806 with 32 x 32 x 16 products in
// the same schedule on the same box, 1336 with the register-staged 128 x 128 kernel; the outputs come out with the same bits.
#pragma once
#include <type_traits>

#include "attn_bf16_lds_dma.h"

namespace seka {

constexpr int kWideTile = 256, kWideK = 64, kWideHalf = 128 * kWideK * 2;     // bytes of a half tile

// Where a wave's routing sums go: those of 64 tokens from `tok` on (they lie in one prompt, S is a multiple of 128) and of up to
// 64 features from `col` on (of one head, D = 128).  Wave-uniform, one scalar division by S and one by G.  (Where the sums are
// formed, for every 16 features, they were vector code, the one by S of 64 bits: 8 of the 18 KB of the wide kernel, and 0.5
// to 1 us per launch: 32 / 8 heads, E = 512, 128 tokens 9.8 -> 9.1 us.)
__device__ __forceinline__ float* project_sums(float* workspace, size_t tok, int col, int S, int G, int Hkv) {
  const unsigned block = (unsigned)(tok >> 6), blocks = (unsigned)S >> 6, b = block / blocks, tchunk = block % blocks;
  const unsigned hq = (unsigned)col >> 7, h = hq / (unsigned)G, g = hq % (unsigned)G;
  return workspace + ((((size_t)b * Hkv + h) * blocks + tchunk) * G + g) * 128 + (col & 127);
}

template <bool ROUTE>
__global__ __launch_bounds__(512) void project_route_wide_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
                                                                 uint16_t* __restrict__ Qout, int E, long long tokens, int N,
                                                                 int S, int G, int Hkv, float* __restrict__ workspace) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char wide_smem[];     // A: [2 slices][2 halves], then B
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  // Workgroups go round-robin over the 8 XCDs: each XCD takes a contiguous run of tiles, in groups of 8 token tiles x
  // all feature tiles walked by columns, so that the 32 tiles of an XCD at a time share 8 + 4 operand panels in its L2.
  const int nM = (int)((tokens + kWideTile - 1) / kWideTile), nN = (N + kWideTile - 1) / kWideTile;
  const int tiles = nM * nN, per = (tiles + 7) / 8;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || t >= tiles) return;         // workgroup-uniform, before any barrier
  const int group = t / (8 * nN), in = t % (8 * nN), gm = min(8, nM - 8 * group);
  const int mt = 8 * group + in % gm, nt = in / gm;
  const size_t row0 = (size_t)mt * kWideTile;
  const int col0 = nt * kWideTile;
  const bool rows_hi = (long long)row0 + 128 < tokens, cols_hi = col0 + 128 < N;    // else the tile has one half only

  // Row r of an A half is token 128 half + r; row r of a B half is feature 64 (r / 32) + 32 half + r % 32, so a wave's
  // features of both halves are 64 in a row.  A missing half repeats rows of the other (its results are not stored).
  const size_t rowbytes = (size_t)E * 2;
  uint32_t aoff[2], boff[2], slot_lds[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int slot = wave + 8 * s, r = 8 * slot + (lane >> 3);
    const uint32_t chunk = 16u * ((lane & 7) ^ ((r >> 1) & 7));
    const int block = r >> 5;
    aoff[s] = (uint32_t)r * (uint32_t)rowbytes + chunk;
    boff[s] = (uint32_t)(64 * (cols_hi ? block : block & 1) + (r & 31)) * (uint32_t)rowbytes + chunk;
    slot_lds[s] = 1024u * slot;
  }
  const unsigned char* Xb = reinterpret_cast<const unsigned char*>(X) + row0 * rowbytes;
  const unsigned char* Wb = reinterpret_cast<const unsigned char*>(W) + (size_t)col0 * rowbytes;
  const size_t a_half = rows_hi ? 128 * rowbytes : 0, b_half = 32 * rowbytes;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(dma_lds_void_ptr)wide_smem, ldsB = lds0 + 4 * kWideHalf;
  const int nk = E / kWideK;
  auto issue_a = [&](int half, int k, int buf) __attribute__((always_inline)) {     // past the end: a slice nobody uses
    const unsigned char* src = Xb + (half ? a_half : 0) + (size_t)min(k, nk - 1) * (kWideK * 2);
#pragma unroll
    for (int s = 0; s < 2; ++s) dma_load_16B(src, aoff[s], lds0 + (2 * buf + half) * kWideHalf + slot_lds[s]);
  };
  auto issue_b = [&](int half, int k, int buf) __attribute__((always_inline)) {
    const unsigned char* src = Wb + (half ? b_half : 0) + (size_t)min(k, nk - 1) * (kWideK * 2);
#pragma unroll
    for (int s = 0; s < 2; ++s) dma_load_16B(src, boff[s], ldsB + (2 * buf + half) * kWideHalf + slot_lds[s]);
  };

  typedef __attribute__((address_space(3))) const bf16x8* lds_frag;
  constexpr int KK = kWideK / 32;          // products of a slice
  uint32_t a_addr[KK], b_addr[KK];         // operand (row l16, elements 32 kk + 8 grp .. + 7) of the wave's rows in buffer 0, half 0
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const uint32_t in_row = 16u * ((4 * kk + grp) ^ ((l16 >> 1) & 7));
    a_addr[kk] = lds0 + (64 * wm + l16) * 128 + in_row;
    b_addr[kk] = ldsB + (32 * wn + l16) * 128 + in_row;
  }
  f32x4 acc[2][2][4][2];                   // [A half][B half][block of 16 tokens][block of 16 features]
#pragma unroll
  for (int i = 0; i < 32; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i >> 4][(i >> 3) & 1][(i >> 1) & 3][i & 1][r] = 0.f;
  struct OperandB { bf16x8 f[2][KK]; };
  bf16x8 a[4][KK];
  OperandB b0, b1;
  auto read_a = [&](int off) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) a[rb][kk] = *(lds_frag)(uintptr_t)(a_addr[kk] + off + 2048 * rb);
  };
  auto read_b = [&](OperandB& b, int off) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) b.f[cb][kk] = *(lds_frag)(uintptr_t)(b_addr[kk] + off + 2048 * cb);
  };
  auto multiply = [&](f32x4 (&c)[4][2], const OperandB& b) __attribute__((always_inline)) {
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          c[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb][kk], b.f[cb][kk], c[rb][cb], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
  };
  // One slice; B half 0 is in bc on entry, B half 0 of the next slice in bn on return.
  auto slice = [&](auto buf_c, int k, OperandB& bc, OperandB& bn) __attribute__((always_inline)) {
    constexpr int C = decltype(buf_c)::value;
    read_a(2 * C * kWideHalf);
    issue_b(1, k + 1, C ^ 1);
    dma_wait_vmcnt<8>();
    multiply(acc[0][0], bc);
    read_b(bn, (2 * C + 1) * kWideHalf);
    issue_a(1, k + 1, C ^ 1);
    dma_wait_vmcnt<8>();
    multiply(acc[0][1], bn);
    read_a((2 * C + 1) * kWideHalf);
    issue_a(0, k + 2, C);
    dma_wait_vmcnt<6>();
    multiply(acc[1][1], bn);
    read_b(bn, 2 * (C ^ 1) * kWideHalf);
    issue_b(0, k + 2, C);
    dma_wait_vmcnt<10>();
    multiply(acc[1][0], bc);
  };
  issue_a(0, 0, 0);
  issue_b(0, 0, 0);
  issue_b(1, 0, 0);
  issue_a(1, 0, 0);
  issue_a(0, 1, 1);
  issue_b(0, 1, 1);
  dma_wait_vmcnt<8>();
  asm volatile("s_barrier" ::: "memory");
  if (wave >= 4) asm volatile("s_barrier" ::: "memory");           // one part behind
  read_b(b0, 0);
  int k = 0;
#pragma nounroll
  for (; k + 1 < nk; k += 2) {
    slice(std::integral_constant<int, 0>{}, k, b0, b1);
    slice(std::integral_constant<int, 1>{}, k + 1, b1, b0);
  }
  if (k < nk) slice(std::integral_constant<int, 0>{}, k, b0, b1);
  if (wave < 4) asm volatile("s_barrier" ::: "memory");
  dma_wait_vmcnt<0>();                     // the last requests still write to the buffers
  dma_barrier();

  // ---- epilogue: round, sum for the routing, stage 64 tokens x 64 features per wave, store whole lines ----
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  unsigned char* const stage = wide_smem + 16384 * wave;           // [2][64 tokens][128 bytes], chunks swizzled with the token
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  const uint32_t sel = (l16 & 1) ? 0x03020706u : 0x05040100u;      // bytes of {neighbour, own}: see below
  const bool cols = cols_hi || wn < 2;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if ((i == 1 && !rows_hi) || !cols) continue;                   // wave-uniform
    float* const sums = ROUTE ? project_sums(workspace, row0 + 128 * i + 64 * wm, col0 + 64 * wn, S, G, Hkv) : nullptr;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        float colsum = 0.f;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            // tokens m, m + 1 of feature column l16; an even lane keeps token m of columns l16, l16 + 1, an odd one
            // token m + 1 of columns l16 - 1, l16
            const bf16x2 own = {(__bf16)acc[i][j][rb][cb][r], (__bf16)acc[i][j][rb][cb][r + 1]};
            colsum = __builtin_amdgcn_fdot2_f32_bf16(own, ones, colsum, false);
            const uint32_t mine = __builtin_bit_cast(uint32_t, own);
            const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xB1, 0xf, 0xf, true);   // lane ^ 1
            const uint32_t pair = __builtin_amdgcn_perm(other, mine, sel);
            const int m = 16 * rb + 4 * grp + r + (l16 & 1), byte = 64 * j + 32 * cb + 4 * (l16 >> 1);
            *reinterpret_cast<uint32_t*>(stage + 8192 * i + 128 * m + (byte ^ (16 * (m & 7)))) = pair;
          }
        if (ROUTE) {
          colsum += __shfl_xor(colsum, 16);
          const float tot = colsum + __shfl_xor(colsum, 32);
          if (grp == 0) sums[32 * j + 16 * cb + l16] = tot;
        }
      }
    }
    asm volatile("" ::: "memory");         // a wave's LDS accesses complete in program order
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int m = 8 * it + (lane >> 3);
      const u32x4 line = *reinterpret_cast<const u32x4*>(stage + 8192 * i + 128 * m + ((16 * (lane & 7)) ^ (16 * (m & 7))));
      *reinterpret_cast<u32x4*>(Qout + (row0 + 128 * i + 64 * wm + m) * (size_t)N + col0 + 64 * wn + 8 * (lane & 7)) = line;
    }
  }
}

}  // namespace seka
