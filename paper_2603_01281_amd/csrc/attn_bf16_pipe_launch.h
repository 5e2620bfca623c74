// Launch-side dispatch of the software-pipelined bf16 attention kernel.  The plain kernels and the steered kernels of
// each compile-time rank are instantiated in translation units of their own, per head dimension.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstring>

#include "attn_bf16_pipe_kernel.h"
#include "compute_units.h"

namespace seka {

// Compute units of the current device (256 on MI355X).
inline int pipe_compute_units() {
  static PerDeviceCount cus;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  return cus.of(dev, [](int d) {
    int n = 0;
    return hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, d) == hipSuccess && n > 0 ? n : 256;
  });
}

struct PipeWidth {
  int width;
  double cost;
};

// Workgroups that share the nQB blocks of query rows of a prompt (back and forth, see the kernel): the W of the least
// estimated time, in units of one 64-key tile of one workgroup.  Candidates are pairs of blocks and as many
// workgroups as fill the chip 1, 2, 3 or 4 times.  A workgroup's load is the same for every slot up to the last deal;
// with a quarter of the compute units idle the others run a fifth faster (the chip is limited by its power).
// Pairs alone left the last round of workgroups mostly empty at most lengths (Hq=32, Hkv=8, us, pairs / chosen):
// S=1024 37 / 31, S=5000 250 / 199, S=9000 672 / 575, B=2 S=4423 356 / 298; at the lengths whose pairs fill the
// chip a whole number of times they stay (S=4096, B=4 S=8192).
inline PipeWidth pipe_width(int D, int nQB, int BQ, int nHC, int B, int cus) {
  const double tiles = BQ / 64.0;
  PipeWidth best = {1, 0};
  for (int m = 0; m <= 4; ++m) {
    const long long fill = (long long)m * cus / ((long long)nHC * B);
    const int W = m == 0 ? (nQB + 1) / 2 : (int)std::max(1LL, std::min((long long)nQB, fill));
    const long long groups = (long long)W * nHC * B, rounds = (groups + cus - 1) / cus;
    const int passes = (nQB + W - 1) / W;
    const double pairs = nQB / (2 * W), rest = nQB - 2.0 * W * pairs;
    const double load = pairs * (2.0 * nQB + 1) - 2.0 * W * pairs * pairs + rest;     // blocks of the first slot, the most
    const double full = load * tiles + passes * pipe_block_tiles(D) + pipe_start_tiles(D);
    const double last = (double)(groups - (rounds - 1) * cus) / cus;                  // share of the chip in the last round
    double cost = (rounds - 1 + 0.8 + 0.2 * std::max(0.0, 4 * last - 3)) * full;
    if (rounds > 1 && W == nQB)   // single blocks, dealt out as workgroups finish
      cost = std::max(nQB * tiles + pipe_block_tiles(D) + pipe_start_tiles(D),
                      ((double)nQB * (nQB + 1) / 2 * tiles + nQB * (pipe_block_tiles(D) + pipe_start_tiles(D))) * nHC * B / cus +
                          0.5 * (tiles + pipe_block_tiles(D) + pipe_start_tiles(D)));
    const double prompts = std::min((double)B, (double)cus / ((double)W * nHC));      // whose K and V an L2 serves at a time
    const double l2 = prompts * nQB * BQ * 4.0 * D / 4.2e6;
    // Rank 32, D = 128, us, without this term / with it: B=4 S=8192 32 / 8 heads 1934 / 1902, B=8 S=8192 16 / 8 1960 / 1919, B=16
    // S=4096 32 / 4 2080 / 2012, B=6 S=5000 32 / 8 1190 / 1163, B=16 S=6000 8 / 2 1112 / 1084, B=8 S=3000 32 / 32 728 / 665; no
    // difference at B=2 S=8192 and B=4 S=4096 32 / 8 and B=4 S=12288 24 / 8; the other way at B=2 S=24576 28 / 4, 7298 / 7424.
    if (prompts > 1.01 && l2 > 1) cost *= 1 + 0.03 * std::log2(l2);
    if (m == 0 || cost < best.cost) best = {W, cost};
  }
  return best;
}

template <int D, int HPW, int RBW, bool STEER, int NKR>
hipError_t launch_attention_bf16_pipe_cfg(AttnArgs a, const SteerArgs* steer, hipStream_t s) {
  constexpr int BQ = 32 * RBW;
  const size_t smem = attention_bf16_pipe_smem_bytes(D, a.S, STEER, NKR, HPW * RBW);
  if (smem > 160 * 1024) return hipErrorNotSupported;
  auto kernel = attention_bf16_pipe_kernel<D, HPW, RBW, STEER, NKR>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  const int nQB = (a.S + BQ - 1) / BQ;
  const int nHC = a.Hq / HPW, cus = pipe_compute_units();
  long long items;                           // workgroups per head chunk
  a.slots = 0;
  if (a.lens || a.cu) {
    // The kernel shares the work out by the lengths it finds (12 prompts of 260 to 4096 tokens, rank 48, with the
    // routing: 515 us, pairs in prompt order 556).  More prompts than a wave has lanes, or than workgroups run at a
    // time: pairs of blocks in prompt order.
    const int slots = cus / nHC;
    a.width = (nQB + 1) / 2;
    items = (long long)a.width * a.B;
    if (a.B <= 64 && a.B < slots) {
      a.slots = slots;
      items = std::min((long long)nQB * a.B, (long long)PIPE_RAGGED_ROUNDS * slots);
      a.width = (int)items;
    }
  } else {
    a.width = pipe_width(D, nQB, BQ, nHC, a.B, cus).width;
    items = (long long)a.width * a.B;
  }
  const long long blocks = items * nHC;
  if (blocks > 0x7fffffffLL) return hipErrorNotSupported;
  SteerArgs sa;
  if (STEER) sa = *steer; else memset(&sa, 0, sizeof(sa));
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64 * HPW * RBW), smem, s, a, sa);
  return hipGetLastError();
}

// Workgroup shape by GQA group size: HPW query heads of one KV head x RBW blocks of 32 query rows.
template <int D, bool STEER, int NKR>
hipError_t launch_attention_bf16_pipe_group(const AttnArgs& a, const SteerArgs* steer, hipStream_t s) {
  const int G = a.Hq / a.Hkv;
  if (G % 4 == 0) return launch_attention_bf16_pipe_cfg<D, 4, 2, STEER, NKR>(a, steer, s);
  if (G % 7 == 0) {
    // Seven heads x 32 rows keeps seven waves of eight busy and repeats the edit in more workgroups; 256 rows of one or
    // two heads leaves a coarser grid.  Hq=28, Hkv=4, rank 32, us: B=16 S=500 67 against 86, B=8 S=1000 93 / 99,
    // B=2 S=2000 72 / 72, B=1 S=2000 63 / 54, B=2 S=4423 306 / 275, B=1 S=16384 1812 / 1608.
    const int hpw = G % 2 == 0 ? 2 : 1, bq = 256 / hpw, cus = pipe_compute_units();    // the shape the group falls to below
    const double seven = pipe_width(D, (a.S + 31) / 32, 32, a.Hq / 7, a.B, cus).cost;
    const double wide = pipe_width(D, (a.S + bq - 1) / bq, bq, a.Hq / hpw, a.B, cus).cost;
    if (wide > 1.02 * seven) return launch_attention_bf16_pipe_cfg<D, 7, 1, STEER, NKR>(a, steer, s);
  }
  if (G % 2 == 0) return launch_attention_bf16_pipe_cfg<D, 2, 4, STEER, NKR>(a, steer, s);
  return launch_attention_bf16_pipe_cfg<D, 1, 8, STEER, NKR>(a, steer, s);
}

}  // namespace seka
