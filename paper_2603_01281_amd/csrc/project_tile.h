// Query projection in BM x BN tiles: Q[t, n] = sum_e X[t, e] W[n, e], bf16 in, fp32 accumulate, bf16 out, with the routing
// sums of its outputs (project_wide.h has the sizes that fill the chip with 256 x 256 tiles).
//
// WM x WN waves, each TM x TN outputs, on v_mfma_f32_16x16x32_bf16 (see project_wide.h).  64-wide slices of E travel straight
// into a ring of NS stages in LDS, NS of them ahead (three where a slice is 32 or 48 KB; four of the 24 KB slices of 128 x 64
// tiles, whose one wave per SIMD finishes a slice before the third one ahead has come.  Against three with 32 x 32 x 16 products,
// 28 shapes of up to 240 such tiles, geometric means at E = 512, 1024, 2048, 4096: four 0.99 / 0.98 / 0.95 / 0.93, six 1.02 / 1.00 /
// 0.98 / 0.95);
// the operands of a slice are read one slice before its products.  One barrier per slice: behind barrier k slice k + 1 is in
// LDS (every wave has waited for its own loads of it) and slice k in registers (and for its reads of it), so its stage
// takes slice k + NS, and the reads of slice k + 1 run beside the products of slice k.
#pragma once
#include <type_traits>

#include "project_wide.h"

namespace seka {

template <int BM, int BN, int WM, int WN, int NS, bool ROUTE>
__global__ __launch_bounds__(64 * WM * WN) void project_route_tile_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
                                                                          uint16_t* __restrict__ Qout, int E, long long tokens, int N,
                                                                          int S, int G, int Hkv, float* __restrict__ workspace) {
  constexpr int NW = WM * WN, TM = BM / WM, TN = BN / WN, RBS = TM / 16, CBS = TN / 16;
  constexpr int ROWS = BM + BN, STAGE = ROWS * kWideK * 2;         // a slice: BM rows of X, then BN rows of W, 128 bytes each
  constexpr int LPW = ROWS / 8 / NW;                               // 1 KB loads per wave and slice
  static_assert(ROWS / 8 % NW == 0 && TM == 64, "whole loads; a wave's routing sums are those of 64 tokens");
  extern __shared__ __attribute__((aligned(1024))) unsigned char tile_smem[];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // Each XCD takes a contiguous run of tiles, in groups of 8 token tiles x all feature tiles walked by columns.
  const int nM = (int)((tokens + BM - 1) / BM), nN = (N + BN - 1) / BN;
  const int tiles = nM * nN, per = (tiles + 7) / 8;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || t >= tiles) return;         // workgroup-uniform, before any barrier
  const int group = t / (8 * nN), in = t % (8 * nN), gm = min(8, nM - 8 * group);
  const int mt = 8 * group + in % gm, nt = in / gm;
  const size_t row0 = (size_t)mt * BM;
  const int col0 = nt * BN;

  // Load n of a wave: rows 8 (wave + NW n) .. + 7 of the stage, lane l chunk l % 8 of row l / 8; the 16-byte chunks of a row are
  // swizzled (chunk ^ (row / 2) % 8) for conflict-free operand reads.  Rows past the tensors' ends repeat the last one.
  const size_t rowbytes = (size_t)E * 2;
  uint32_t off[LPW];
  const int last_row = (int)min((long long)BM, tokens - (long long)row0) - 1, last_col = min(BN, N - col0) - 1;
#pragma unroll
  for (int n = 0; n < LPW; ++n) {
    const int r = 8 * (wave + NW * n) + (lane >> 3);
    const uint32_t chunk = 16u * ((lane & 7) ^ ((r >> 1) & 7));
    off[n] = (uint32_t)(r < BM ? min(r, last_row) : min(r - BM, last_col)) * (uint32_t)rowbytes + chunk;
  }
  const unsigned char* Xb = reinterpret_cast<const unsigned char*>(X) + row0 * rowbytes;
  const unsigned char* Wb = reinterpret_cast<const unsigned char*>(W) + (size_t)col0 * rowbytes;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(dma_lds_void_ptr)tile_smem;
  const int nk = E / kWideK;
  auto issue_one = [&](int n, size_t at, int stage) __attribute__((always_inline)) {
    // BM / 8 is a multiple of NW or the other way round: wave-uniform either way
    dma_load_16B((8 * (wave + NW * n) < BM ? Xb : Wb) + at, off[n], lds0 + stage * STAGE + 1024 * (wave + NW * n));
  };
  auto at_of = [&](int k) __attribute__((always_inline)) { return (size_t)min(k, nk - 1) * (kWideK * 2); };     // past the end: a slice nobody uses

  typedef __attribute__((address_space(3))) const bf16x8* lds_frag;
  constexpr int KK = kWideK / 32;          // products of a slice
  uint32_t a_addr[KK], b_addr[KK];         // operand (row l16, elements 32 kk + 8 grp .. + 7) of the wave's rows in stage 0
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const uint32_t in_row = 16u * ((4 * kk + grp) ^ ((l16 >> 1) & 7));
    a_addr[kk] = lds0 + (TM * wm + l16) * 128 + in_row;
    b_addr[kk] = lds0 + (BM + TN * wn + l16) * 128 + in_row;
  }
  f32x4 acc[RBS][CBS];
#pragma unroll
  for (int i = 0; i < RBS; ++i)
#pragma unroll
    for (int j = 0; j < CBS; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
  struct Operands { bf16x8 a[RBS][KK], b[CBS][KK]; };
  Operands even, odd;
  constexpr int PER_KK = RBS + CBS, READS = KK * PER_KK, PRODUCTS = KK * RBS * CBS;
  auto read_one = [&](Operands& f, int i, int stage) __attribute__((always_inline)) {
    const int kk = i / PER_KK, r = i % PER_KK;
    if (r < RBS) f.a[r][kk] = *(lds_frag)(uintptr_t)(a_addr[kk] + stage * STAGE + 2048 * r);
    else f.b[r - RBS][kk] = *(lds_frag)(uintptr_t)(b_addr[kk] + stage * STAGE + 2048 * (r - RBS));
  };
  // One slice, in program order: a product, then an operand read of the next slice, then a request, until all are issued.
  // Left to itself the compiler moves the reads to the end of the slice, in front of the products that wait for them (E = N =
  // 4096: 1024 tokens 40.3 -> 35.9 us, 2048 67.2 -> 60.2, 128 26.0 -> 24.4).
  auto slice = [&](auto turn_c, int k) __attribute__((always_inline)) {      // turn_c: k modulo the unrolled turns
    constexpr int TURN = decltype(turn_c)::value;
    Operands &now = TURN % 2 ? odd : even, &next = TURN % 2 ? even : odd;
    dma_wait_vmcnt<(NS - 2) * LPW>();
    dma_barrier();
    const size_t at = at_of(k + NS);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < PRODUCTS; ++p) {
      const int kk = p / (RBS * CBS), i = p / CBS % RBS, j = p % CBS;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(now.a[i][kk], now.b[j][kk], acc[i][j], 0, 0, 0);
      if (p < READS) read_one(next, p, (TURN + 1) % NS);
      if (p < LPW) issue_one(p, at, TURN % NS);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int k = 0; k < NS; ++k)
#pragma unroll
    for (int n = 0; n < LPW; ++n) issue_one(n, at_of(k), k);
  dma_wait_vmcnt<(NS - 1) * LPW>();
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int i = 0; i < READS; ++i) read_one(even, i, 0);
  constexpr int TURNS = NS % 2 ? 2 * NS : NS;
  int k = 0;
  auto turns = [&](auto n_c) __attribute__((always_inline)) {
    constexpr int LEFT = decltype(n_c)::value;                     // the first LEFT slices of a round of turns, as far as there are any
    auto one = [&](auto i_c) __attribute__((always_inline)) {
      constexpr int I = decltype(i_c)::value;
      if constexpr (I < LEFT)
        if (LEFT == TURNS || k + I < nk) slice(i_c, k + I);
    };
    one(std::integral_constant<int, 0>{});
    one(std::integral_constant<int, 1>{});
    one(std::integral_constant<int, 2>{});
    one(std::integral_constant<int, 3>{});
    one(std::integral_constant<int, 4>{});
    one(std::integral_constant<int, 5>{});
  };
#pragma nounroll
  for (; k + TURNS <= nk; k += TURNS) turns(std::integral_constant<int, TURNS>{});
  turns(std::integral_constant<int, TURNS - 1>{});
  dma_wait_vmcnt<0>();                     // the last requests still write to the ring
  dma_barrier();

  // ---- epilogue: round, sum for the routing, stage TM tokens x TN features per wave, store whole lines ----
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  constexpr int LINE = TN * 2, LC = LINE / 16;                     // bytes and 16-byte chunks of a staged row
  unsigned char* const stage = tile_smem + TM * LINE * wave;       // chunks swizzled with the token
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  const uint32_t sel = (l16 & 1) ? 0x03020706u : 0x05040100u;      // bytes of {neighbour, own}: see below
  if (TM * wm > last_row || TN * wn > last_col) return;            // wave-uniform; no barrier follows
  float* const sums = ROUTE ? project_sums(workspace, row0 + TM * wm, col0 + TN * wn, S, G, Hkv) : nullptr;
#pragma unroll
  for (int j = 0; j < CBS; ++j) {
    float colsum = 0.f;
#pragma unroll
    for (int rb = 0; rb < RBS; ++rb)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        // tokens m, m + 1 of feature column l16; an even lane keeps token m of columns l16, l16 + 1, an odd one token
        // m + 1 of columns l16 - 1, l16
        const bf16x2 own = {(__bf16)acc[rb][j][r], (__bf16)acc[rb][j][r + 1]};
        colsum = __builtin_amdgcn_fdot2_f32_bf16(own, ones, colsum, false);
        const uint32_t mine = __builtin_bit_cast(uint32_t, own);
        const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xB1, 0xf, 0xf, true);   // lane ^ 1
        const uint32_t pair = __builtin_amdgcn_perm(other, mine, sel);
        const int m = 16 * rb + 4 * grp + r + (l16 & 1), byte = 32 * j + 4 * (l16 >> 1);
        *reinterpret_cast<uint32_t*>(stage + LINE * m + (byte ^ (16 * (m & (LC - 1))))) = pair;
      }
    if (ROUTE) {
      colsum += __shfl_xor(colsum, 16);
      const float tot = colsum + __shfl_xor(colsum, 32);
      if (grp == 0) sums[16 * j + l16] = tot;
    }
  }
  asm volatile("" ::: "memory");           // a wave's LDS accesses complete in program order
#pragma unroll
  for (int it = 0; it < TM * LC / 64; ++it) {
    const int m = (64 / LC) * it + lane / LC, c = lane % LC;
    const u32x4 line = *reinterpret_cast<const u32x4*>(stage + LINE * m + ((16 * c) ^ (16 * (m & (LC - 1)))));
    *reinterpret_cast<u32x4*>(Qout + (row0 + TM * wm + m) * (size_t)N + col0 + TN * wn + 8 * c) = line;
  }
}

}  // namespace seka
