// bf16 causal GQA prefill attention for gfx950, head dimensions 64 and 128, with the spectral key edit fused in
// (paper Sec. 2: logits q_i . k'_j / sqrt(d_k), k'_j = k_j + g P k_j for highlighted j; Sec. 3.3 for the
// blended P of AdaSEKA).  Flash-style: scores and edited keys never leave the CU.  Software-pipelined,
// 32 query rows per wave; attn_bf16_lds_dma.h describes how the tiles travel.
//
// Math mapping: S^T = K Q^T on v_mfma_f32_16x16x32_bf16 with A = K rows from LDS and B = Q fragments resident
// in registers, in tiles of 16 keys x 16 query rows: each lane owns one query row of each of its wave's two row tiles and
// 8 of a block's 32 keys; O^T = V^T P^T with B = P^T taken straight from the S^T accumulators (the
// contraction order over keys is permuted identically on the V side) and A = V^T fetched from the row-major V
// tile with the transposing LDS read ds_read_b64_tr_b16.  A workgroup is HPW query heads of one KV group x
// RBW blocks of 32 query rows, all sharing the K/V tiles (and the edit) of that KV head.
//
// What bounds this kernel on gfx950 is the chip's power limit and the SIMD's issue port, not the matrix pipe alone: with
// everything but the MFMAs removed a 64-key tile of a workgroup takes 0.99 us, the LDS operand reads add 0.15, the softmax
// 0.3, tile loads and barrier 0.1 (a stand-alone loop of this step, all compute units busy; each at its own clock).
// Consequences:
//   * the products are 16 x 16 x 32 and not 32 x 32 x 16: half the accumulator traffic per multiply-add, and on random operands
//     the chip sustains 1.95 PFLOP/s of them against 1.76 (mfma_rate_probe.hip).  With four plain vector instructions beside each 32 cycles of
//     MFMA that is 17.7 ns against 20.2;
//   * the row sums are products too (one more output tile, of ones): as v_dot2c_f32_bf16 of the packed probabilities, eight per
//     32-key block, they took 2.3 of 20.6 ns, as two MFMAs they take 1.0;
//   * every vector instruction in the loop that is not softmax arithmetic is removed: LDS read addresses
//     are a register plus an immediate (the loop is unrolled over the three ring stages so that stage
//     offsets are compile-time constants), tile loads take a scalar base plus a per-lane offset computed
//     once, and the common case of a step computes no row maximum at all (see `step`): 44 vector instructions
//     per 34 MFMAs;
//   * MFMAs and vector instructions alternate in program order, and every MFMA has vector work beside it:
//     a step handles three consecutive 32-key blocks at once: the S^T products of the next block, the softmax
//     of the current one and the PV products of the previous one (whose probabilities were formed one step
//     earlier), with one exponential for every second MFMA.
// Measured, us, 32 x 32 x 16 products with sums by dot products / now, launches of one box in turns: B=4 S=8192 32 / 8 heads D = 128
// plain 1800 / 1703, rank 32 1892 / 1801; B=1 S=4096 124 / 118; B=1 S=32768 28 / 4 heads rank 64 6364 / 6060; B=4 S=700 rank 32
// 32.9 / 32.7; D = 64 B=4 S=4096 plain 305 / 293, rank 32 317 / 305.
// Tried: 64 query rows per wave, one wave per SIMD, outputs and queries in accumulation registers (half the LDS reads):
// 1.6 % slower in the stand-alone loop and 15 % in the kernel, whose barrier and branches nothing overlaps then.
// The softmax runs per 32-key block (half a tile), which halves the score registers the pipeline needs.
// K tiles live in a ring of three LDS stages; V in a ring of six half tiles that runs half a tile behind K
// (see the tile loads).  K(t+2) and the V blocks 2t+3, 2t+4 are requested during iteration t (in the hot loop
// between its two steps, so that the first step's LDS reads follow the per-tile barrier directly).  The steering
// event of tile t+2 (highlighted keys only) sits between the two steps of iteration t + 1: at rank <= 32 the
// coordinates c .* U^T k of its keys are computed and the scores of that tile get a rank-32 correction against
// U^T q afterwards (score-side form, the tile itself stays as loaded); at larger ranks the keys are edited in LDS.
#pragma once
#include <type_traits>
#include <utility>

#include "attn_bf16_lds_dma.h"

namespace seka {

// LDS beyond the two tile rings (steered kernels): the edit's matrix operand, the per-column coefficients, one
// 64-bit highlight word per tile and, for rank <= 32, the buffers of the score-side form.
// Rank <= 32 (nkr == 1): the edit is applied to the scores, s_ij = q_i . k_j + (U^T q_i) . (c .* U^T k_j) for
// highlighted j (paper Sec. 2, the equivalence of key-side and score-side control, Eq. 5): U_cat is stored once, as
// the operand of U_cat^T K^T; the coordinates c .* U^T k of a tile's keys go to one of two 64 x 32 bf16 buffers,
// and every wave keeps U^T q of its 32 rows as two MFMA operands (2 KB).  Larger ranks: the keys themselves are edited with the dense D x D matrix
// g P = U_cat diag(c) U_cat^T, built once per workgroup; at rank >= 64 one product with it moves no more operand
// bytes than two low-rank products and has no intermediate.  Either way the operands are stored in the order the
// MFMAs read them (one 16-byte LDS read per lane and operand).
constexpr int PIPE_RA = 8;                          // MFMAs between an operand read from LDS and its use (5, 7 and 10 within 1 %)
constexpr int PIPE_Z_BYTES = DMA_BK * 64;           // one coordinate buffer: [4 blocks of 16 keys][64 lanes][8] bf16
constexpr int PIPE_QT_BYTES = 2048;                 // U^T q of one wave: [2 row tiles][64 lanes][8] bf16
// bf16 parts of an element of g P (dense form).  One part rounds it to 2^-9, at D = 128 less than the edited key's own
// rounding adds; a full-rank projector at D = 64 (whose diagonal is g) was further from the exact result than the form with
// two low-rank products (4.2e-3 against 3.3e-3, 2-norms), so there a second part carries the remainder.
constexpr int pipe_edit_parts(int D) { return D == 64 ? 2 : 1; }
inline size_t attention_bf16_pipe_smem_bytes(int D, int S, bool steer, int nkr, int nwaves) {
  size_t n = (size_t)2 * DMA_STAGES * DMA_BK * D * 2;
  if (D == 64) n += (size_t)4096 * nwaves;             // staging areas (at D = 128 the rings have room for them)
  if (steer) {
    const int Rpad = 32 * nkr;
    n += nkr == 1 ? (size_t)D * Rpad * 2 : (size_t)pipe_edit_parts(D) * D * D * 2;
    n += (size_t)Rpad * 4;
    if (nkr == 1) n += (size_t)2 * PIPE_Z_BYTES + (size_t)nwaves * PIPE_QT_BYTES;
    n += (size_t)((S + DMA_BK - 1) / DMA_BK) * 8;
  }
  return n;
}

typedef __attribute__((address_space(3))) const bf16x8* pipe_lds_bf16x8_ptr;

// The products of the tile loop are inline assembly: with the builtin the compiler takes other registers for a product's result than
// for its accumulator, and then waits before it lets anything else into the registers that became free.  It does not know what
// they are, so the waits that the instruction needs are placed by hand: a product's result may be read or overwritten by a vector
// instruction 8 wait states after it was issued at the earliest (4 passes and 4, which is what the compiler keeps behind its own;
// mfma_result_guard is 12; in the pipelined loop the products of the outputs and sums lie between, 18 at D = 128, 10 at D = 64),
// and a register that a vector instruction wrote may be read by a product after 2 (mfma_operand_guard).
__device__ __forceinline__ void pipe_mfma_first(f32x4& d, const bf16x8& a, const bf16x8& b) {      // d = a b
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void pipe_mfma(f32x4& d, const bf16x8& a, const bf16x8& b) {            // d += a b
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void pipe_mfma_result_guard(f32x4 (&s)[2][2]) {
  asm volatile("s_nop 11" : "+v"(s[0][0]), "+v"(s[0][1]), "+v"(s[1][0]), "+v"(s[1][1]));
}
__device__ __forceinline__ void pipe_mfma_operand_guard(bf16x8 (&p)[2]) { asm volatile("s_nop 3" : "+v"(p[0]), "+v"(p[1])); }
// What vector instructions made of the accumulators is complete here; the compiler may not move them past it.
template <int N>
__device__ __forceinline__ void pipe_pin_acc(f32x4 (&o)[N][2], f32x4 (&l)[2]) {
#pragma unroll
  for (int i = 0; i < N; i += 2) asm volatile("" : "+v"(o[i][0]), "+v"(o[i][1]), "+v"(o[i + 1][0]), "+v"(o[i + 1][1]));
  asm volatile("" : "+v"(l[0]), "+v"(l[1]));
}

__device__ __forceinline__ float pipe_max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// (the LDS address is wave-uniform, which the compiler does not always see)
__device__ __forceinline__ void pipe_load_16B(const void* base, uint32_t lane_off, uint32_t lds_base) {
  dma_load_16B(base, lane_off, __builtin_amdgcn_readfirstlane(lds_base));
}

// Sum / maximum over the 64 lanes (all active), the same value in all of them.
__device__ __forceinline__ float pipe_wave_sum(float v) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}
__device__ __forceinline__ int pipe_wave_max(int v) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v = max(v, __shfl_xor(v, m));
  return __builtin_amdgcn_readfirstlane(v);
}

// What a block of query rows and a workgroup cost beside their key tiles, in units of one 64-key tile (2800 cycles at
// D = 128, 1900 at D = 64):
// a block waits for its first tiles, runs its last ones outside the unrolled loop and writes its output (stamps: 4.7 tiles at D = 128,
// 5.4 at D = 64); a workgroup starts and prepares the edit (plain 2.4 and 2.1, rank <= 32 3.3 and 3.4, above 4.1).  Little hangs on
// them: over 330 drawn shapes at D = 128 and 140 at D = 64, each timed at all five widths that are considered, the widths chosen with
// half or twice these values are within 0.8 % of those chosen with these.
constexpr float pipe_block_tiles(int D) { return 4.f * 128 / D; }
constexpr float pipe_start_tiles(int D) { return 3.f * 128 / D; }

// Workgroup `item` of the a.width that a batch of prompts of different lengths (at most 64) gets per head chunk.
// Lane i looks after prompt i: its n_i blocks of query rows are T_i = sum over them of (tiles + pipe_block_tiles) of
// work, which W_i = floor(T_i / L) + 1 workgroups share.  L is the load of a workgroup if the batch is to take R
// rounds of the a.slots workgroups that run at a time, T / (R slots - B), and no less than the longest block;
// R = 1 .. PIPE_RAGGED_ROUNDS is the one with the smallest R (L + pipe_start_tiles).  The longest prompts come first,
// so the last workgroups to start are the shortest.  Returns false past the last workgroup.
constexpr int PIPE_RAGGED_ROUNDS = 6;
template <int BQ, int D>
__device__ __forceinline__ bool pipe_ragged_item(const AttnArgs& a, int item, int& b, int& slot, int& W) {
  const int lane = threadIdx.x & 63;
  size_t tok0;
  int len = 0;
  if (lane < a.B) prompt_extent(a, lane, tok0, len);
  const int nb = (len + BQ - 1) / BQ;
  constexpr float T = BQ / 64.f;                 // key tiles per block of query rows
  const float work = (float)nb * (0.5f * T * (float)(nb + 1) + pipe_block_tiles(D));
  const float total = pipe_wave_sum(work);
  const float longest = T * (float)pipe_wave_max(nb) + pipe_block_tiles(D);
  float best = 0.f, load = longest;
#pragma unroll
  for (int R = 1; R <= PIPE_RAGGED_ROUNDS; ++R) {
    const int share = R * a.slots - a.B;
    const float L = fmaxf(longest, total / (float)max(share, 1));
    const float cost = (float)R * (L + pipe_start_tiles(D));
    if (share > 0 && (best == 0.f || cost < best)) {
      best = cost;
      load = L;
    }
  }
  int w = min(nb, (int)(work / load) + 1);
  // sum of w <= total / load + B <= R slots <= a.width; should rounding ever break this, one workgroup per prompt
  if (pipe_wave_sum((float)w) > (float)a.width) w = min(nb, 1);
  int first = 0;                                 // this prompt's first workgroup
  for (int j = 0; j < a.B; ++j) {
    const int nj = __builtin_amdgcn_readlane(nb, j), wj = __builtin_amdgcn_readlane(w, j);
    first += (nj > nb || (nj == nb && j < lane)) ? wj : 0;
  }
  const unsigned long long hit = __ballot(item >= first && item < first + w);
  if (hit == 0ull) return false;
  b = __builtin_ctzll(hit);
  slot = item - __builtin_amdgcn_readlane(first, b);
  W = __builtin_amdgcn_readlane(w, b);
  return true;
}

// The 16-byte chunk of tile row `row` that lies at position p is p ^ swizzle: conflict-free 16-byte reads of one chunk
// of 16 consecutive rows (K), and conflict-free transposing reads of eight consecutive rows x 32 bytes (V).
template <int D>
__host__ __device__ constexpr int pipe_k_swizzle(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
template <int D>
__host__ __device__ constexpr int pipe_v_swizzle(int row) { return D == 128 ? 4 * (row & 3) + 2 * ((row >> 2) & 1) : 2 * ((row >> 1) & 3); }

template <class F, int... I>
__device__ __forceinline__ void pipe_static_for_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void pipe_static_for(F&& f) { pipe_static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// Which K fragment a step reads behind its MFMA m, and which of a lane's 16 scores it takes up there (-1: none); see `step`.
constexpr int pipe_kfrag_at(int m, int ks, int ahead) {
  for (int f = 2; f < 2 * ks; ++f)
    if (m == (2 * f - ahead < f - 2 ? f - 2 : 2 * f - ahead)) return f;
  return -1;
}
constexpr int pipe_element_at(int m, int mfmas) {
  for (int e = 0; e < 16; ++e)
    if (m == e * (mfmas >= 34 ? mfmas - 3 : 16) / 16) return e;
  return -1;
}

// HPW heads x RBW row groups = waves per workgroup; every wave owns 32 consecutive query rows, two row tiles of 16.
// NKR: rank of the concatenated basis in blocks of 32 columns (compile-time so that the edit is straight-line code).
template <int D, int HPW, int RBW, bool STEER, int NKR>
__global__ __launch_bounds__(64 * HPW * RBW) __attribute__((amdgpu_waves_per_eu(2, D == 64 ? 2 : 8))) void
attention_bf16_pipe_kernel(AttnArgs a, SteerArgs st) {
  static_assert(D == 64 || D == 128, "head dimensions of the tile layouts");
  constexpr int NW = HPW * RBW;
  constexpr int NT = 64 * NW;
  constexpr int WR = 32;
  constexpr int BQ = WR * RBW;
  constexpr int BK = DMA_BK;
  constexpr int KS = D / 32;                             // slices of the head dimension that a product contracts
  constexpr int DT = D / 16;                             // output tiles of 16 columns
  constexpr int RB = 2 * D, CH = D / 8;                  // bytes and 16-byte chunks of a tile row
  constexpr int TB = BK * RB;                            // bytes of a tile
  constexpr int SLOTS = TB / 1024;
  constexpr int SPW = (SLOTS + NW - 1) / NW;             // load instructions per wave per tensor per tile

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* Kst = smem;                                     // [3][TB] swizzled K tiles (16 KB each at D = 128, 8 KB at D = 64)
  unsigned char* Vst = smem + DMA_STAGES * TB;                   // [3][TB] swizzled V tiles
  constexpr int Rpad = 32 * NKR, NP = pipe_edit_parts(D);
  constexpr bool DENSE = NKR >= 2;         // edit with the dense matrix g P (see attention_bf16_pipe_smem_bytes)
  constexpr bool kEventsInHot = STEER && (!DENSE || NW == 8);   // steering events handled inside the hot loop (see the tile loop)
  uint16_t* UN = reinterpret_cast<uint16_t*>(smem + 2 * DMA_STAGES * TB + (D == 64 ? 4096 * NW : 0));
  uint16_t* U1 = UN;                       // low rank: operand (rb, s) of U_cat^T K^T: [2][4][64 lanes][8]
  uint16_t* AP = UN;                       // dense: operand (s_out, half, ks) of (g P) K^T: [NP][D/32][2][D/32][64 lanes][8]
  float* cvec = reinterpret_cast<float*>(UN + (DENSE ? (size_t)NP * D * D : (size_t)D * Rpad));   // [Rpad]
  unsigned char* zbuf = reinterpret_cast<unsigned char*>(cvec + Rpad);     // low rank: [2][4 blocks][64 lanes][8] coordinates
  unsigned char* qtbuf = zbuf + 2 * PIPE_Z_BYTES;                          // low rank: [NW][2][64 lanes][8] U^T q
  unsigned long long* hlbits = reinterpret_cast<unsigned long long*>(      // [tiles] (STEER)
      DENSE ? reinterpret_cast<unsigned char*>(cvec + Rpad) : qtbuf + NW * PIPE_QT_BYTES);

  const uint16_t* __restrict__ Qg = static_cast<const uint16_t*>(a.Q);
  const uint16_t* __restrict__ Kg = static_cast<const uint16_t*>(a.K);
  const uint16_t* __restrict__ Vg = static_cast<const uint16_t*>(a.V);
  uint16_t* __restrict__ Og = static_cast<uint16_t*>(a.O);

  const int Scap = a.S;                      // tokens per prompt in memory (strides, launch grid)
  const int G = a.Hq / a.Hkv;
  const int nHC = a.Hq / HPW;
  // A workgroup handles several blocks of query rows of one (batch, head group), one after the other.  A prompt's
  // blocks, latest (longest) first, are dealt to its W workgroups back and forth: slot 0 .. W-1, then W-1 .. 0 and so
  // on.  Two deals give every slot the same number of key tiles, so there is no imbalance from causality; the
  // steering set-up is done once for all of a workgroup's blocks, and a block's first loads overlap the output stores
  // of the one before.  W comes from the launcher (see pipe_width there).
  // blockIdx = (prompt, slot, head chunk), head chunk fastest: workgroups are dispatched round-robin over the
  // XCDs in index order, so with 8 head chunks an XCD's L2 serves one KV head, and the workgroups resident at the
  // same time walk the K / V tiles of the same prompt from tile 0 on, at the same pace.
  const int hc = (int)(blockIdx.x % nHC);
  const int item = (int)(blockIdx.x / nHC);
  const int hq0 = hc * HPW;
  const int h = hq0 / G;
  int b, slot, W = a.width;
  if (a.slots) {
    if (!pipe_ragged_item<BQ, D>(a, item, b, slot, W)) return;
  } else {
    b = item / a.width;
    slot = item % a.width;
  }
  size_t tok0;                               // first token of this prompt in the tensors
  int S;                                     // this prompt's length: rows and keys beyond it do not exist
  prompt_extent(a, b, tok0, S);
  const int nblocks = (S + BQ - 1) / BQ;
  if (!a.slots && (a.cu || a.lens)) W = (nblocks + 1) / 2;
  if (slot >= W || slot >= nblocks) return;  // workgroup-uniform, before any barrier
  int qb = nblocks - 1 - slot;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4;
  const int hq = hq0 + wave / RBW;
  // Waves w and w + 4 share a SIMD: their row blocks are chosen to end on different tiles or halves of a tile.
  const int rb = RBW == 1 ? 0 : RBW == 2 ? (wave ^ (wave >> 2)) & 1 : RBW == 4 ? (wave & 3) ^ (wave >> 2 ? 3 : 0) : wave < 4 ? wave : 11 - wave;
  int qw = qb * BQ + WR * rb;    // first query row of this wave
  int qi0 = qw + l16;                      // this lane's query row in row tile 0 (tile 1: + 16)

  const float gain = STEER ? st.gain[h] : 0.f;
  const float kscale = STEER ? st.kscale[h] : 1.f;
  const bool steer_on = STEER && gain != 0.f;

  int last_key = min(S, qb * BQ + BQ) - 1;
  int ntiles = last_key / BK + 1;          // the first block is the later one: its tile count bounds the second's

  // ---- tile loads: scalar tile base + per-lane offset fixed for the whole kernel ----
  // Slot s of a tile is LDS bytes [1024 s, 1024 s + 1024) = 4 rows (8 at D = 64); lane l lands at row l / CH of them,
  // chunk position l % CH, and fetches the logical chunk that the swizzle assigns to that position.
  const uint32_t rowbytes = (uint32_t)a.Hkv * D * 2;
  const uint32_t kst_base = (uint32_t)(uintptr_t)(dma_lds_void_ptr)Kst;
  const uint32_t vst_base = kst_base + DMA_STAGES * TB;      // (Vst itself, a generic pointer, would be compared with null at every request)
  // V travels in units of half a tile, one half tile behind K: "shifted tile" t = rows [64 t - 32, 64 t + 32) = the
  // 32-key blocks 2t - 1 and 2t, and block j lives at ring position j % 6 (HB bytes each; tile t = positions 2t % 6,
  // 2t % 6 + 1 as before).  The PV product of a block runs one step after its softmax (see `step`), so the last
  // block of tile t is still being read while the loads of iteration t + 1 are in flight; shifting the unit by
  // half a tile makes every load overwrite only blocks that all waves are done with.
  constexpr int HB = TB / 2;              // bytes of a 32-key block
  // Load n of a wave fills slot wave + NW n (surplus loads repeat the last slot, same bytes).
  auto slot_of = [&](int w, int n) __attribute__((always_inline)) { return SLOTS % NW == 0 ? w + NW * n : min(w + NW * n, SLOTS - 1); };
  auto slot_lds = [&](int w, int n) __attribute__((always_inline)) { return 1024u * slot_of(w, n); };
  // of a shifted tile of V: the block that slot n belongs to, and where it lies in it
  auto vslot_hi = [&](int w, int n) __attribute__((always_inline)) { return NW == SLOTS / 2 ? n == 1 : slot_of(w, n) >= SLOTS / 2; };
  auto vslot_lds = [&](int w, int n) __attribute__((always_inline)) { return NW == SLOTS / 2 ? 1024u * w : 1024u * (slot_of(w, n) & (SLOTS / 2 - 1)); };
  auto slot_row = [&](int n) __attribute__((always_inline)) { return (64 / CH) * slot_of(wave, n) + lane / CH; };   // this lane's row in it
  // (the wave's index passes through an opaque copy at every request: the LDS addresses of all stages would be kept in scalar registers)
  auto opaque_wave = [&]() __attribute__((always_inline)) {
    int w = wave;
    asm volatile("" : "+s"(w));
    return w;
  };
  uint32_t koff[SPW], voff[SPW];
#pragma unroll
  for (int n = 0; n < SPW; ++n) {
    const int row = slot_row(n);
    koff[n] = row * rowbytes + 16u * ((lane & (CH - 1)) ^ pipe_k_swizzle<D>(row));
    voff[n] = row * rowbytes + 16u * ((lane & (CH - 1)) ^ pipe_v_swizzle<D>(row));
  }
  const size_t head_off = (tok0 * a.Hkv + h) * D * 2;          // bytes to this (batch, KV head), token 0
  const unsigned char* Kbytes = reinterpret_cast<const unsigned char*>(Kg) + head_off;
  const unsigned char* Vbytes = reinterpret_cast<const unsigned char*>(Vg) + head_off;
  // ring position (byte offset inside the V ring) of 32-key block j >= -1
  auto vpos = [&](int j) __attribute__((always_inline)) -> uint32_t { return (uint32_t)((j + 6) % 6) * HB; };
  // K tile t into its ring stage.  `full`: every row of the tile exists (no clamping, offsets fixed per lane).
  // Otherwise rows past the prompt's end repeat its last key (finite data that the causal mask hides); offsets
  // are then taken from token 0 so that they never go negative.
  auto issue_k_to = [&](auto full_c, int t, uint32_t lds_stage_base) __attribute__((always_inline)) {
    const int w = opaque_wave();
    if (decltype(full_c)::value || t * BK + BK <= S) {
      // (a product of 32-bit factors: of 64-bit ones it took five scalar instructions more per tile)
      const unsigned char* tile = Kbytes + (uint64_t)(uint32_t)(t * BK) * rowbytes;
#pragma unroll
      for (int n = 0; n < SPW; ++n) pipe_load_16B(tile, koff[n], lds_stage_base + slot_lds(w, n));
    } else {
#pragma unroll
      for (int n = 0; n < SPW; ++n) {
        uint32_t ko = koff[n];
        int row = slot_row(n);
        asm volatile("" : "+v"(ko), "+v"(row));     // formed here, not hoisted out of the loops into a register (or scratch slot) of its own
        pipe_load_16B(Kbytes, ko + (uint32_t)(min(t * BK + row, S - 1) - row) * rowbytes,
                      lds_stage_base + slot_lds(w, n));
      }
    }
  };
  // Shifted V tile t: block 2t - 1 to ring byte offset posA, block 2t to posB.
  auto issue_v_to = [&](auto full_c, int t, uint32_t posA, uint32_t posB) __attribute__((always_inline)) {
    const int w = opaque_wave();
    const int first = t * BK - BK / 2;
    if (decltype(full_c)::value || (first >= 0 && first + BK <= S)) {
      const unsigned char* tile = Vbytes + (uint64_t)(uint32_t)first * rowbytes;
#pragma unroll
      for (int n = 0; n < SPW; ++n) pipe_load_16B(tile, voff[n], vst_base + (vslot_hi(w, n) ? posB : posA) + vslot_lds(w, n));
    } else {
#pragma unroll
      for (int n = 0; n < SPW; ++n) {
        uint32_t vo = voff[n];
        int row = slot_row(n);
        asm volatile("" : "+v"(vo), "+v"(row));
        pipe_load_16B(Vbytes, vo + (uint32_t)(min(max(first + row, 0), S - 1) - row) * rowbytes,
                      vst_base + (vslot_hi(w, n) ? posB : posA) + vslot_lds(w, n));
      }
    }
  };
  auto issue_k = [&](int t) __attribute__((always_inline)) { issue_k_to(std::false_type{}, t, kst_base + (t % 3) * TB); };
  auto issue_v = [&](int t) __attribute__((always_inline)) { issue_v_to(std::false_type{}, t, vpos(2 * t - 1), vpos(2 * t)); };

  // 4 KB per wave for turning Q rows into operands and the output accumulators into rows: the third stage of the K
  // ring and positions 3 and 4 of the V ring, which a block's first loads do not touch (at D = 64 an area of its own).  32 rows x 128 bytes; the
  // 16-byte chunk of a row is swizzled with the row (chunk ^ row % 8).
  static_assert(NW <= 8, "one 4 KB staging area per wave");
  unsigned char* const stg = D == 64    ? smem + 2 * DMA_STAGES * TB + 4096 * wave
                             : wave < 4 ? Kst + 2 * TB + 4096 * wave
                                        : Vst + 3 * HB + 4096 * (wave - 4);
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  // (the lane index passes through an opaque copy where they are used: addresses formed from it would be kept over the tile loops)
  auto opaque_lane = [&]() __attribute__((always_inline)) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    return ln;
  };
  auto stg_line = [&](int ln, int i) __attribute__((always_inline)) -> u32x4* {     // chunk ln % 8 of row 8 i + ln / 8
    return reinterpret_cast<u32x4*>(stg + 1024 * i + 128 * (ln >> 3) + 16 * ((ln & 7) ^ (ln >> 3)));
  };
  auto stg_row = [&](int ln, int rt, int chunk) __attribute__((always_inline)) -> unsigned char* {     // of row 16 rt + ln % 16
    return stg + 2048 * rt + 128 * (ln & 15) + 16 * (chunk ^ (ln & 7));
  };

  // ---- Q fragments: B operand of S^T = K Q^T, lane (col = row 16 rt + l16, k = 32 ks + 8 grp + e) at rt KS + ks ----
  bf16x8 qf[2 * KS];
  // First loads of a block of query rows: K tiles 0 and 1, V blocks -1 (a copy of row 0: the first step's PV
  // product multiplies it by zero probabilities, so it only has to be finite) to 2, then the wave's Q rows.
  auto begin_block = [&]() __attribute__((always_inline)) {
    issue_k(0);
    issue_v(0);
    if (ntiles > 1) issue_k(1);
    issue_v(1);
    // Raw order: register i of lane l holds 16-byte chunk (l % 8) + 8 (i / 4) of row 8 (i % 4) + l / 8, so every load
    // covers eight whole 128-byte lines; q_operands() turns them into operands through LDS.  (Fetched in operand
    // order, 32 rows x 32 bytes per load, the address unit took 3 cycles per row: 6000 cycles per block.)
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {    // rows past the end read row 0 (finite data, results never stored):
      const int qi = qw + 8 * (i & 3) + (lane >> 3);                                          // no branch, no wait here
      const uint16_t* qp = Qg + ((tok0 + (qi < S ? qi : 0)) * a.Hq + hq) * D + 64 * (i >> 2) + 8 * (lane & 7);
      qf[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(qp));
    }
  };
  auto q_operands = [&]() __attribute__((always_inline)) {
    bf16x8 qn[2 * KS];
    const int ln = opaque_lane();
#pragma unroll
    for (int half = 0; half < D / 64; ++half) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *stg_line(ln, i) = __builtin_bit_cast(u32x4, qf[4 * half + i]);
      asm volatile("" ::: "memory");       // a wave's LDS accesses complete in program order: no wait needed
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          qn[rt * KS + 2 * half + ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(stg_row(ln, rt, 4 * ks + (ln >> 4))));
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) qf[i] = qn[i];
  };
  begin_block();

  // ---- steering set-up: edit operands, per-column coefficients, highlight bitmap ----
  // Every global load of the set-up (mask bytes, U_cat, routing weights) is issued before the first of them is
  // waited for, with addresses clamped into range instead of branches around the loads: one memory round trip.
  if (STEER && steer_on) {
    const int R = st.M * st.r;
    const uint16_t* Uh = static_cast<const uint16_t*>(st.U) + (size_t)h * st.M * D * st.r;
    const int r8 = st.r / 8;
    const int total = st.M * D * r8;                  // 16-byte pieces of U_cat
    constexpr int UB = 4;                             // pieces per thread and turn

    // (1) mask bytes of tile `tid` (first turn of the bitmap loop), if the fast form applies
    const uint8_t* mrow = st.mask + tok0;
    const int nfull = S / BK;
    const bool wide = (reinterpret_cast<uintptr_t>(mrow) & 15) == 0 && nfull > 0;
    uint4 mv0[BK / 16];
    if (wide) {
      const uint4* mp = reinterpret_cast<const uint4*>(mrow + (size_t)min(tid, nfull - 1) * BK);
#pragma unroll
      for (int q = 0; q < BK / 16; ++q) mv0[q] = mp[q];
    }
    // The other tiles (the last one of most lengths; all of them where a packed prompt starts off a 16-byte boundary): a wave
    // takes a tile, a lane a byte, the word is a ballot.  First turn: MB tiles per wave.
    constexpr int MB = 4;
    const int ballot0 = (wide ? nfull : 0) + wave;
    uint8_t mb0[MB];
#pragma unroll
    for (int k = 0; k < MB; ++k) mb0[k] = mrow[min((ballot0 + NW * k) * BK + lane, S - 1)];
    // (2) first turn of U_cat.  Piece idx = (expert m, row d, 8-column group v); the divisions by run-time
    // constants are done in floating point (exact for these small operands: idx < 64 K, quotients < 2 K).
    const float inv_dr8 = 1.f / (float)(D * r8), inv_r8 = 1.f / (float)r8;
    auto split = [&](int idx, int& m, int& d, int& v) __attribute__((always_inline)) {
      m = (int)(((float)idx + 0.5f) * inv_dr8);
      const int rm = idx - m * (D * r8);
      d = (int)(((float)rm + 0.5f) * inv_r8);
      v = rm - d * r8;
    };
    uint4 uv[UB];
    int um[UB], ud[UB], uc[UB];
#pragma unroll
    for (int k = 0; k < UB; ++k) {
      uv[k] = make_uint4(0, 0, 0, 0);
      um[k] = ud[k] = uc[k] = 0;
      if (k * NT < total) {                          // workgroup-uniform
        split(min(tid + k * NT, total - 1), um[k], ud[k], uc[k]);
        uv[k] = *reinterpret_cast<const uint4*>(Uh + ((size_t)um[k] * D + ud[k]) * st.r + 8 * uc[k]);
      }
    }
    // (3) routing weight of column `tid`
    float cw = 1.f;
    if (st.w) cw = st.w[((size_t)b * a.Hkv + h) * st.M + min(tid, R - 1) / st.r];

    auto bits_of = [&](const uint4 (&mv)[BK / 16]) __attribute__((always_inline)) -> unsigned long long {
      unsigned long long bits = 0ull;
#pragma unroll
      for (int q = 0; q < BK / 16; ++q) {
        const uint32_t x4[4] = {mv[q].x, mv[q].y, mv[q].z, mv[q].w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          // non-zero test of the four bytes of x, gathered into four adjacent bits
          const uint32_t x = x4[w];
          const uint32_t y = ((x | ((x & 0x7f7f7f7fu) + 0x7f7f7f7fu)) & 0x80808080u) >> 7;
          const uint32_t nib = ((y * 0x00204081u) >> 21) & 0xfu;
          bits |= (unsigned long long)nib << (16 * q + 4 * w);
        }
      }
      return bits;
    };
    // one 64-bit word per tile: bit k = key 64 t + k is highlighted.  Whole tiles, one thread per tile:
    if (wide)
      for (int t = tid; t < min(ntiles, nfull); t += NT) {
        if (t == tid) {
          hlbits[t] = bits_of(mv0);
        } else {
          uint4 mv[BK / 16];
          const uint4* mp = reinterpret_cast<const uint4*>(mrow + (size_t)t * BK);
#pragma unroll
          for (int q = 0; q < BK / 16; ++q) mv[q] = mp[q];
          hlbits[t] = bits_of(mv);
        }
      }
    // The others.  (Byte by byte in one thread, 64 loads in a row, they cost 5 to 8 us per launch of an odd length: B=2 S=333
    // 32 / 8 heads rank 32 20.6 -> 15.9 us.)
    for (int t0 = ballot0; t0 < ntiles; t0 += MB * NW) {
      uint8_t mb[MB];
#pragma unroll
      for (int k = 0; k < MB; ++k) mb[k] = t0 == ballot0 ? mb0[k] : mrow[min((t0 + NW * k) * BK + lane, S - 1)];
#pragma unroll
      for (int k = 0; k < MB; ++k) {
        const int t = t0 + NW * k;
        const unsigned long long bits = __ballot(t * BK + lane < S && mb[k] != 0);
        if (t < ntiles && lane == 0) hlbits[t] = bits;
      }
    }
    if (tid < Rpad) cvec[tid] = tid < R ? gain * cw : 0.f;        // Rpad <= 128 < NT

    // where a 16-byte piece of U_cat goes
    constexpr int CPR = Rpad / 8;                    // dense form: chunks per staged row, 8 or 16
    auto ustage = [&](int d, int chunk) __attribute__((always_inline)) -> unsigned char* {
      const int sw = CPR == 16 ? (d & 15) : ((d >> 1) & 7);
      const int off = d * (Rpad * 2) + 16 * (chunk ^ sw);
      return off < TB ? Kst + 2 * TB + off : Vst + 3 * HB + (off - TB);
    };
    auto place = [&](int m, int d, int v, const uint4 val) __attribute__((always_inline)) {
      if (DENSE) {
        *reinterpret_cast<uint4*>(ustage(d, (m * st.r) / 8 + v)) = val;
      } else {
        const int r0 = m * st.r + 8 * v;              // concatenated column of the first of these 8 elements
        const uint16_t* e16 = reinterpret_cast<const uint16_t*>(&val);
        // operand (rb, s) of U_cat^T K^T: lane (g, j) holds U_cat[d = 32 s + 8 g + e][r = 16 rb + j], e = 0..7
        const int s1 = d >> 5, g1 = (d >> 3) & 3, e1 = d & 7;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int r = r0 + i;
          U1[((((r >> 4) * KS + s1) * 64) + g1 * 16 + (r & 15)) * 8 + e1] = e16[i];
        }
      }
    };
    if (!DENSE && R != Rpad) {
      for (int i = tid; i < D * Rpad / 8; i += NT) reinterpret_cast<uint4*>(UN)[i] = make_uint4(0, 0, 0, 0);
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < UB; ++k)
      if (tid + k * NT < total) place(um[k], ud[k], uc[k], uv[k]);
    for (int idx = tid + UB * NT; idx < total; idx += NT) {        // further turns (large rank and few waves only)
      int m, d, v;
      split(idx, m, d, v);
      place(m, d, v, *reinterpret_cast<const uint4*>(Uh + ((size_t)m * D + d) * st.r + 8 * v));
    }
    if (DENSE) {
      // Dense form.  U_cat (row d, r contiguous, zero-padded to Rpad columns) is staged in the third stage of
      // the K ring and positions 3 and 4 of the V ring, which no tile load touches before the main loop starts
      // (the first loads fill V positions 5, 0, 1 and 2); 16-byte chunks of a row are
      // swizzled so that sixteen consecutive rows can be read at one chunk index without bank conflicts.
      const int padc = CPR - R / 8;                    // R is a multiple of 8
      for (int idx = tid; idx < D * padc; idx += NT)
        *reinterpret_cast<uint4*>(ustage(idx / padc, R / 8 + idx % padc)) = make_uint4(0, 0, 0, 0);
      __syncthreads();
      // T = (U_cat diag(c)) U_cat^T in 16 x 16 blocks; wave w computes the rows 16 w .. 16 w + 15.  The block
      // element T[y][x] is stored where the edit expects (g P)[d_out = x][d' = y] (T is symmetric up to rounding).
      const int j = lane & 15, g = lane >> 4;
      for (int strip = wave; strip < D / 16; strip += NW) {
        bf16x8 af[NKR], al[NKR];      // A operand: lane (row = 16 strip + j, k = r = 32 kk + 8 g + e), scaled by c_r; al: its remainder
#pragma unroll
        for (int kk = 0; kk < NKR; ++kk) {
          const bf16x8 u = *reinterpret_cast<const bf16x8*>(ustage(16 * strip + j, 4 * kk + g));
          const f32x4 c0 = *reinterpret_cast<const f32x4*>(cvec + 32 * kk + 8 * g);
          const f32x4 c1 = *reinterpret_cast<const f32x4*>(cvec + 32 * kk + 8 * g + 4);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = (float)u[e] * (e < 4 ? c0[e & 3] : c1[e & 3]);
            af[kk][e] = (__bf16)x;
            if (NP == 2) al[kk][e] = (__bf16)(x - (float)af[kk][e]);
          }
        }
#pragma unroll
        for (int ct = 0; ct < D / 16; ++ct) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < NKR; ++kk) {
            const bf16x8 bfr = *reinterpret_cast<const bf16x8*>(ustage(16 * ct + j, 4 * kk + g));
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[kk], bfr, acc, 0, 0, 0);
            if (NP == 2) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[kk], bfr, acc, 0, 0, 0);
          }
          // this lane holds T[y = 16 strip + 4 g + i][x = 16 ct + j], i = 0..3
          const int x = 16 * ct + j, xl = x & 31, y0 = 16 * strip + 4 * g;
          const int frag = ((x >> 5) * 2 + ((xl >> 2) & 1)) * KS + (y0 >> 5);           // (s_out, half, ks)
          const int flane = 16 * ((y0 & 31) >> 3) + 4 * (xl >> 3) + (xl & 3);          // lane (g', j') of the edit
          bf16x4 o4;
#pragma unroll
          for (int i = 0; i < 4; ++i) o4[i] = (__bf16)acc[i];
          *reinterpret_cast<uint2*>(AP + (frag * 64 + flane) * 8 + (y0 & 7)) = __builtin_bit_cast(uint2, o4);
          if (NP == 2) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o4[i] = (__bf16)(acc[i] - (float)o4[i]);
            *reinterpret_cast<uint2*>(AP + D * D + (frag * 64 + flane) * 8 + (y0 & 7)) = __builtin_bit_cast(uint2, o4);
          }
        }
      }
      if (D == 128) dma_barrier();           // q_operands() stages its rows where the staged U_cat lies
    }
  }
  // Which of the 64 tiles [tile0, tile0 + 64) hold a highlighted key: kept in scalar registers so that the common
  // case (nothing to edit) costs no LDS access.  Valid once the bitmap is complete (after the first barrier).
  auto any_word = [&](int tile0) __attribute__((always_inline)) -> unsigned long long {
    const int idx = tile0 + lane;
    const unsigned long long v = (steer_on && idx < ntiles) ? hlbits[idx] : 0ull;
    return __ballot(v != 0ull);
  };

  // Dense form (rank > 32): edit the highlighted 16-key blocks of (swizzled) K tile `tile` at Kb in place; wave w < 4
  // owns block w.  Every block reads all of the matrix operand (32 KB at D = 128), so blocks are not split further.  The
  // output rows go in 2 KS groups of 16: the operand of a group is read while the group before it is multiplied, and a
  // group is finished (scaled, added) while the next one is multiplied; the wave's keys and the first operand are on their way
  // before it knows whether its block has highlighted keys.  (One group at a time, reads, products and the rest in a row, an
  // event cost an editing wave 2050 cycles, all of it latency.)  ahead_c false: one group at a time all the same, for the turns behind
  // a wave's last tile at D = 128, where the reads ahead spilled 17 to 25 registers (no slower: ratios of time for B=8 S=4096 32 / 8 heads rank 128, a ragged batch of rank 48
  // and one prompt of 32k tokens at rank 64 0.999 to 1.001; 110 shapes 0.998).
  auto edit_tile = [&](auto ahead_c, unsigned char* Kb, int tile) __attribute__((always_inline)) {
    // The lane index is re-derived behind an opaque copy so that none of the per-lane operand addresses below
    // is hoisted out of the tile loop: they would occupy registers the attention pipeline needs.
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int j = ln & 15, g = ln >> 4;
    const int kblk = opaque_wave();
    if (kblk >= BK / 16) return;                          // wave-uniform
    const unsigned long long bits = hlbits[tile];
    unsigned char* krow = Kb + (16 * kblk + j) * RB;
    bf16x8 kreg[KS];   // K^T as B operand: lane (col = key j, k = d = 32 s + 8 g + e) = logical chunk 4 s + g
#pragma unroll
    for (int s = 0; s < KS; ++s) kreg[s] = *reinterpret_cast<const bf16x8*>(krow + 16 * ((4 * s + g) ^ pipe_k_swizzle<D>(j)));
    struct Operand { bf16x8 u[NP][KS]; };     // of a group of 16 output rows
    auto part = [&](int g8, int p, int ks) __attribute__((always_inline)) {
      return *reinterpret_cast<const bf16x8*>(AP + p * D * D + ((g8 * KS + ks) * 64 + ln) * 8);
    };
    Operand ua;
#pragma unroll
    for (int i = 0; i < NP * KS; ++i) ua.u[i / KS][i % KS] = part(0, i / KS, i % KS);
    const unsigned bits16 = __builtin_amdgcn_readfirstlane((unsigned)((bits >> (16 * kblk)) & 0xffffull));
    if (bits16 == 0) return;                              // wave-uniform
    const bool lit = (bits16 >> j) & 1u;
    // k' = a k + (g P) k: output rows d are permuted so that each result lands in the lane that holds that
    // element of k, and the products are added to a k there.  Keys that are not highlighted keep their bits.
    f32x4 c[3];
    auto start = [&](int g8) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) c[g8 % 3][i] = (float)kreg[g8 >> 1][4 * (g8 & 1) + i] * kscale;
      if (g8 < 2) asm volatile("s_nop 1" : "+v"(c[g8 % 3]));      // behind the others comes a `finish` before their products
      else asm volatile("" : "+v"(c[g8 % 3]));
    };
    uint2 out[2];
    auto finish = [&](int g8) __attribute__((always_inline)) {
      const int s = g8 >> 1, half = g8 & 1;
      // 8 states and more: with the four products of the next group, and behind all but the last but one their reads and four multiplications
      if (g8 == 2 * KS - 2) asm volatile("s_nop 7" : "+v"(c[g8 % 3]));
      else asm volatile("s_nop 3" : "+v"(c[g8 % 3]));
      bf16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (__bf16)c[g8 % 3][i];
      const uint2 ob = __builtin_bit_cast(uint2, o);
      const uint4 kb = __builtin_bit_cast(uint4, kreg[s]);
      out[half] = make_uint2(lit ? ob.x : half ? kb.z : kb.x, lit ? ob.y : half ? kb.w : kb.y);
      if (half) *reinterpret_cast<uint4*>(krow + 16 * ((4 * s + g) ^ pipe_k_swizzle<D>(j))) = make_uint4(out[0].x, out[0].y, out[1].x, out[1].y);
    };
    if (!decltype(ahead_c)::value) {       // one group after the other
#pragma unroll
      for (int g8 = 0; g8 < 2 * KS; ++g8) {
        if (g8 > 0) {
#pragma unroll
          for (int i = 0; i < NP * KS; ++i) ua.u[i / KS][i % KS] = part(g8, i / KS, i % KS);
        }
        start(g8);
        asm volatile("s_nop 1" : "+v"(c[g8 % 3]));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int p = 0; p < NP; ++p) pipe_mfma(c[g8 % 3], ua.u[p][ks], kreg[ks]);
        asm volatile("s_nop 7" : "+v"(c[g8 % 3]));
        finish(g8);
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
    start(0);
#pragma unroll
    for (int g8 = 0; g8 < 2 * KS; ++g8) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          pipe_mfma(c[g8 % 3], ua.u[p][ks], kreg[ks]);
          __builtin_amdgcn_sched_barrier(0);
          if (g8 + 1 < 2 * KS) ua.u[p][ks] = part(g8 + 1, p, ks);
          __builtin_amdgcn_sched_barrier(0);
        }
      if (g8 + 1 < 2 * KS) start(g8 + 1);
      if (g8 > 0) finish(g8 - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_nop 7" : "+v"(c[(2 * KS - 1) % 3]));
    finish(2 * KS - 1);
  };

  // Score-side form (rank <= 32): the coordinates c .* (U_cat^T k) of the 64 keys of (swizzled, unchanged) K tile `tile`
  // at Kb, zero for keys that are not highlighted, into the buffer at zdst; wave w < 4 owns the 16-key block w
  // (a block without highlights only stores zeros).  A key's 32 coordinates are stored in the order the score
  // correction contracts them: lane group grp, slot e  <->  r = 16 (e / 4) + 4 grp + e % 4, which is the order in which
  // a lane of the 16 x 16 accumulators holds U^T q of its query row.  The operands are on their way before the wave knows
  // whether its block has highlighted keys.  What bounds an event is latency: of LDS, and of scalar registers that come back from
  // vector lanes.  With the operands read one after the other here and in `corr`, and the event's tests on 64-bit values whose
  // halves were spilled, short steered prompts at D = 64 took 3.8 % longer (12 shapes, few workgroups or many highlighted keys; 32 / 4 heads
  // S=1220 28.2 -> 27.2 us, 8 / 2 heads S=9875 165.4 -> 158.4).
  auto coords_tile = [&](const unsigned char* Kb, int tile, unsigned char* zdst) __attribute__((always_inline)) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int j = ln & 15, g = ln >> 4;
    const int kblk = opaque_wave();
    if (kblk >= BK / 16) return;                          // wave-uniform
    const unsigned long long bits = hlbits[tile];
    const unsigned char* krow = Kb + (16 * kblk + j) * RB;
    bf16x8 kreg[KS];   // K^T as B operand: lane (col = key j, k = d = 32 s + 8 g + e) = logical chunk 4 s + g
#pragma unroll
    for (int s = 0; s < KS; ++s) kreg[s] = *reinterpret_cast<const bf16x8*>(krow + 16 * ((4 * s + g) ^ pipe_k_swizzle<D>(j)));
    constexpr int AHEAD = D == 64 ? 2 * KS : KS;          // of the 2 KS operands (all of them at D = 128: 8 registers spilled)
    auto operand = [&](int i) __attribute__((always_inline)) { return *reinterpret_cast<const bf16x8*>(U1 + (i * 64 + ln) * 8); };
    bf16x8 ua[2 * KS];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) ua[i] = operand(i);
    auto coefficients = [&](int half) __attribute__((always_inline)) { return *reinterpret_cast<const f32x4*>(cvec + 16 * half + 4 * g); };
    f32x4 c4[2];
    if (D == 64) c4[0] = coefficients(0), c4[1] = coefficients(1);
    __builtin_amdgcn_sched_barrier(0);
    const unsigned bits16 = __builtin_amdgcn_readfirstlane((unsigned)((bits >> (16 * kblk)) & 0xffffull));
    // this lane's results: key 16 kblk + j, coordinates r = 16 half + 4 g + i  ->  lane of the operand, slots 4 half + i
    u32x4* const zrow = reinterpret_cast<u32x4*>(zdst + 1024 * kblk + 16 * ln);
    u32x4 z = {0u, 0u, 0u, 0u};
    if (bits16 != 0) {                                    // wave-uniform
      bf16x8 z8;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // two chains: even and odd slices of d
#pragma unroll
        for (int s = 0; s < KS; ++s) acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ua[half * KS + s], kreg[s], acc[s & 1], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (D == 128) c4[half] = coefficients(half);
#pragma unroll
        for (int i = AHEAD; i < (half == 0 ? 2 * KS : 0); ++i) ua[i] = operand(i);
#pragma unroll
        for (int i = 0; i < 4; ++i) z8[4 * half + i] = (__bf16)((acc[0][i] + acc[1][i]) * c4[half][i]);
      }
      const u32x4 w = __builtin_bit_cast(u32x4, z8);
      const bool lit = (bits16 >> j) & 1u;
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = lit ? w[i] : 0u;
    }
    *zrow = z;
  };

  for (int pass = 0;; ++pass) {      // one turn per block of query rows (indentation of the body kept flat)
  // ---- math pieces ----
  f32x4 oacc[DT][2], lacc[2];              // O^T tiles (16 columns x 16 rows) and, in all four elements alike, the row sums
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    lacc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  pipe_pin_acc(oacc, lacc);
  const float c2 = a.scale * 1.4426950408889634f;   // probabilities are exp2(s * c2 - m)
  // m_run: reference exponent of the row (in units of s * c2).  It follows the row maximum lazily.  A row's first one is put kLead
  // above the maximum of its first block.  It is put there again where a probability of any row of the wave reaches 2, and
  // then in every row of the wave whose maximum has moved more than kSlack since; so too in the wave's last tile, which
  // takes its maxima anyway.  So probabilities stay below 2 and the output accumulators are rescaled a handful of times
  // per row instead of once per block.
  constexpr float kLead = 11.f, kSlack = 8.f;
  float m_run[2] = {-1e30f, -1e30f};
  // The tile loops live in a (generic, always inlined) lambda of their own.  This changes nothing in what is
  // computed; the compiler allocates the loop's registers differently for it, and the launch is 3 % faster.
  auto run_block = [&](auto) __attribute__((always_inline)) {

  // LDS byte addresses of this lane's operands inside stage 0 (stage, key-tile and row offsets are immediates):
  // K: row l16 (+ 16), logical chunk 4 ks + grp
  // V: row 4 grp + (l16 >> 2) (+ 16), logical chunk 2 dt + ((l16 & 3) >> 1)
  uint32_t kaddr[KS], vaddr[DT];
  {
    const int kfix = l16 * RB + 16 * (grp ^ pipe_k_swizzle<D>(l16));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kaddr[ks] = kst_base + (uint32_t)(kfix ^ (ks << 6));
    const int vrow = 4 * grp + (l16 >> 2);
    const int vfix = vrow * RB + 16 * (((l16 & 3) >> 1) ^ pipe_v_swizzle<D>(vrow)) + 8 * (l16 & 1);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vaddr[dt] = vst_base + (uint32_t)(vfix ^ (dt << 5));
  }
  const bf16x8 zeros8 = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
  asm volatile("" : "+v"(ones));           // kept in registers

  // Scores of one 32-key block: S^T tiles [key tile][row tile]; off = LDS byte offset of the block's first row.
  auto kfrag = [&](int i, int off) __attribute__((always_inline)) -> bf16x8 {        // fragment i: slice i / 2, key tile i % 2
    return *(pipe_lds_bf16x8_ptr)(uintptr_t)(kaddr[i >> 1] + off + 16 * (i & 1) * RB);
  };
  auto qk_one = [&](int i, const bf16x8& k, f32x4 (&sn)[2][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      if (i < 2) pipe_mfma_first(sn[i & 1][rt], k, qf[rt * KS + (i >> 1)]);
      else pipe_mfma(sn[i & 1][rt], k, qf[rt * KS + (i >> 1)]);
    }
  };
  auto qk_block = [&](int off, f32x4 (&sn)[2][2]) __attribute__((always_inline)) {
    bf16x8 kf[2 * KS];
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) kf[i] = kfrag(i, off);
    __builtin_amdgcn_sched_barrier(0);     // all of them on their way before the first product
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) qk_one(i, kf[i], sn);
  };
  using IC0 = std::integral_constant<int, 0>;
  // causal mask of the 32-key block starting at key j0
  auto causal_mask = [&](int j0, f32x4 (&sv)[2][2]) __attribute__((always_inline)) {
    const int jbase = j0 + 4 * grp;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (jbase + 16 * kt + i > qi0 + 16 * rt) sv[kt][rt][i] = -INFINITY;
  };
  // Row maximum (of s * c2) over one 32-key block, all lanes of the row.
  auto block_max = [&](int rt, const f32x4 (&sv)[2][2]) __attribute__((always_inline)) -> float {
    float mx = pipe_max3(sv[0][rt][0], sv[0][rt][1], sv[0][rt][2]);
    mx = pipe_max3(mx, sv[0][rt][3], sv[1][rt][0]);
    mx = pipe_max3(mx, sv[1][rt][1], sv[1][rt][2]);
    mx = fmaxf(mx, sv[1][rt][3]) * c2;
    // the other 24 keys of this query row live in lanes ^ 16, ^ 32 and ^ 48
    const auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
    const auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
  };
  // Raise the reference exponent of the rows whose maximum over the block ran away from it, and rescale their outputs and sums
  // (every PV product whose probabilities were formed against the old reference has been accumulated).
  auto raise_reference = [&](const f32x4 (&sv)[2][2], bool empty = false) __attribute__((always_inline)) {
    const float mx[2] = {block_max(0, sv) + kLead, block_max(1, sv) + kLead};
    const bool need0 = mx[0] > m_run[0] + kSlack, need1 = mx[1] > m_run[1] + kSlack;
    if (__any(need0 | need1)) {    // a handful of times per row
      const float m0 = need0 ? mx[0] : m_run[0], m1 = need1 ? mx[1] : m_run[1];
      const float alpha[2] = {__builtin_amdgcn_exp2f(m_run[0] - m0), __builtin_amdgcn_exp2f(m_run[1] - m1)};
      m_run[0] = m0;
      m_run[1] = m1;
      if (empty) return;             // nothing accumulated yet
      // (the maxima and exponentials above lie between the last PV product and these)
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int i = 0; i < 4; ++i) oacc[dt][rt][i] *= alpha[rt];
#pragma unroll
        for (int i = 0; i < 4; ++i) lacc[rt][i] *= alpha[rt];
      }
      pipe_pin_acc(oacc, lacc);
    }
  };
  // Probabilities of one block, packed as P^T operands (lane group grp, slot e <-> key 16 (e / 4) + 4 grp + e % 4).
  auto block_exp = [&](const f32x4 (&sv)[2][2], bf16x8 (&pb)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const float mneg = -m_run[rt];
#pragma unroll
      for (int e = 0; e < 8; ++e) pb[rt][e] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sv[e >> 2][rt][e & 3], c2, mneg));
    }
  };
  // O^T += V^T P^T for one 32-key block, and the row sums of P^T (the rounded probabilities, those that the products use)
  // as one more output tile whose V^T is all ones; off = LDS byte offset of the block's first row
  auto pv_block = [&](int off, bf16x8 (&pb)[2]) __attribute__((always_inline)) {
    s16x4 lo[DT], hi[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      lo[dt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dma_lds_s16x4_ptr)(uintptr_t)(vaddr[dt] + off));
      hi[dt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dma_lds_s16x4_ptr)(uintptr_t)(vaddr[dt] + off + 16 * RB));
    }
    __builtin_amdgcn_sched_barrier(0);     // all of them on their way before the first product
    pipe_mfma_operand_guard(pb);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) pipe_mfma(lacc[rt], ones, pb[rt]);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x4 lo4 = __builtin_bit_cast(bf16x4, lo[dt]), hi4 = __builtin_bit_cast(bf16x4, hi[dt]);
      const bf16x8 va = __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) pipe_mfma(oacc[dt][rt], va, pb[rt]);
    }
  };

  const bool wave_rows_exist = qw < S;
  const int tw_last = wave_rows_exist ? min(ntiles - 1, (qw + WR - 1) / BK) : -1;   // last tile this wave computes on

  // ---- prologue: wait for the first tiles, edit K(0) and K(1), first block of S^T ----
  dma_wait_vmcnt<0>();   // also covers the Q, U and mask loads issued after the tile loads
  q_operands();
#pragma unroll
  for (int i = 0; i < 2 * KS; ++i) asm volatile("" : "+v"(qf[i]));   // pin the compiler's own wait for Q here, not in the loop
  dma_barrier();
  unsigned long long anyw = 0ull;      // bit i: tile 64 (t / 64) + i holds a highlighted key (0 when not steering)
  // Next tile index at which the loop has something to do besides attention: a tile with highlighted keys, or
  // the start of the next group of 64 tiles (summary reload).  Scalar; the loop compares one integer per tile.
  auto next_event = [&](int tile) __attribute__((always_inline)) -> int {     // first event strictly after `tile`
    const unsigned sh = tile & 63;
    const unsigned long long rest = sh == 63u ? 0ull : anyw >> (sh + 1);
    return rest != 0ull ? tile + 1 + __builtin_ctzll(rest) : (tile | 63) + 1;
  };
  int tile_evt = 0x7fffffff;
  int ztile = -1;                      // score-side form: the tile whose coordinates were computed last
  if (STEER && !DENSE) {
    // U^T q of this wave's 32 query rows: (U_cat^T Q^T)[r][row], A = the operand store of U_cat^T K^T as it stands, B = the Q
    // fragments.  A lane ends up with its query rows' coordinates r = 16 rb + 4 grp + i: converted to bf16 they are the
    // B operands of the score correction, kept in LDS (each lane reads back what it wrote: no barrier).
    if (steer_on) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        bf16x8 q8;
#pragma unroll
        for (int rb2 = 0; rb2 < 2; ++rb2) {
          f32x4 qt = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            qt = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(U1 + ((rb2 * KS + ks) * 64 + lane) * 8),
                                                         qf[rt * KS + ks], qt, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) q8[4 * rb2 + i] = (__bf16)qt[i];
        }
        *reinterpret_cast<bf16x8*>(qtbuf + wave * PIPE_QT_BYTES + 1024 * rt + lane * 16) = q8;
      }
    }
    anyw = any_word(0);
    if (anyw & 1ull) {
      coords_tile(Kst, 0, zbuf);
      dma_barrier();
      ztile = 0;
    }
    tile_evt = next_event(0);          // tile 1 is handled by iteration 0 like every later tile
  } else if (STEER) {
    anyw = any_word(0);
    if (anyw & 3ull) {
      if (anyw & 1ull) edit_tile(std::true_type{}, Kst, 0);
      if (anyw & 2ull) edit_tile(std::true_type{}, Kst + TB, 1);
      dma_barrier();
    }
    tile_evt = next_event(1);
  }
  // Score correction of one 32-key block of S^T (keys keyoff .. keyoff + 31 of `tile`): += Z (32 keys x 32 r) . (U^T q)^T,
  // four MFMAs; A = the keys' coordinates from the tile's buffer, B = this wave's U^T q operands.  before_step: the next vector
  // instruction that reads the scores is that of a step.
  auto corr = [&](auto before_step_c, int tile, int keyoff, f32x4 (&sv)[2][2]) __attribute__((always_inline)) {
    const unsigned char* zp = zbuf + (tile & 1) * PIPE_Z_BYTES + keyoff * 64 + lane * 16;
    const unsigned char* qp = qtbuf + wave * PIPE_QT_BYTES + lane * 16;
    const bf16x8 za[2] = {*reinterpret_cast<const bf16x8*>(zp), *reinterpret_cast<const bf16x8*>(zp + 1024)};
    const bf16x8 qb[2] = {*reinterpret_cast<const bf16x8*>(qp), *reinterpret_cast<const bf16x8*>(qp + 1024)};
    __builtin_amdgcn_sched_barrier(0);     // all four on their way before the first product
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) pipe_mfma(sv[kt][rt], za[kt], qb[rt]);
    // a step reads sv[0][0] behind its first product, the other tiles in this order four elements apart: with the three products behind
    // each, eight states and more
    if (decltype(before_step_c)::value) asm volatile("s_nop 3" : "+v"(sv[0][0]), "+v"(sv[0][1]), "+v"(sv[1][0]), "+v"(sv[1][1]));
    else pipe_mfma_result_guard(sv);
  };

  bf16x8 pb[2] = {zeros8, zeros8};   // probabilities (P^T operands) of the block whose PV product is next; none at first
  f32x4 sc0[2][2], sc1[2][2];  // scores of keys 0..31 / 32..63 of the current tile
#pragma unroll
  for (int i = 0; i < 4; ++i) sc0[i >> 1][i & 1] = sc1[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 kpre[2];              // first two K fragments of the block the next step scores (see `step`)
  if (0 <= tw_last) {
    qk_block(0, sc0);
    pipe_mfma_result_guard(sc0);
    // The first reference of rows that see the whole block: its maximum, with the score correction if it gets one (the largest
    // probability is then a power of two and is not rounded: from the maximum without the correction the outputs' error against 64
    // bits was 1 to 2 % larger).  Rows that start with a masked block take theirs after the mask.
    if (0 < tw_last) {
      auto first_reference = [&](const f32x4 (&sv)[2][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) m_run[rt] = fmaxf(block_max(rt, sv) + kLead, m_run[rt]);
      };
      if (STEER && !DENSE && ztile == 0) {
        f32x4 sv[2][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) sv[i >> 1][i & 1] = sc0[i >> 1][i & 1];
        asm volatile("s_nop 1" : "+v"(sv[0][0]), "+v"(sv[0][1]), "+v"(sv[1][0]), "+v"(sv[1][1]));
        corr(std::false_type{}, 0, 0, sv);
        first_reference(sv);
      } else {
        first_reference(sc0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) kpre[i] = kfrag(i, HB);

  // `top` of iteration t: request K(t+2), then the V blocks 2t+3 and 2t+4; their ring slots are free since the
  // barrier of iteration t - 1.  Bottom: everything but those two V blocks must have landed before the next
  // iteration (K(t+2) is edited there, see `events`).  The hot loop calls `top` between its two steps: requests
  // issued right after the barrier delayed the first step's operand reads (1-2 % of the kernel).
  // The hot loop only runs where tile t + 2 exists and is complete (`sure`): no tests there.
  auto top = [&](auto sure_c, auto stage_c, int t) __attribute__((always_inline)) {
    constexpr bool SURE = decltype(sure_c)::value;
    if (SURE) {
      constexpr int ST = decltype(stage_c)::value;          // = t % 3
      issue_k_to(std::true_type{}, t + 2, kst_base + ((ST + 2) % 3) * TB);
      issue_v_to(std::true_type{}, t + 2, ((2 * ST + 3) % 6) * HB, ((2 * ST + 4) % 6) * HB);
    } else if (t + 1 < ntiles) {
      if (t + 2 < ntiles) issue_k(t + 2);
      issue_v(t + 2);                                       // its first block belongs to tile t + 1
    }
  };
  auto bottom = [&](auto sure_c, int t) __attribute__((always_inline)) {
    if (decltype(sure_c)::value || t + 1 < ntiles) dma_wait_vmcnt<SPW>();   // all but the V loads of this iteration
    else dma_wait_vmcnt<0>();
    dma_barrier();
  };

  // Steering events of the tile that landed at the bottom of the previous iteration (tile t + 1 in iteration t):
  // handled between the two steps of an iteration, where a basic-block boundary exists anyway (the conditional
  // rescale).  Directly after the per-tile barrier the same branch kept the compiler from moving the next step's
  // first LDS reads up, which cost every iteration of the steered kernels 7-9 % even with nothing to edit.  The
  // second step is the first reader of that tile; after an edit in place (dense form) its two prefetched
  // fragments are read again.  In the score-side form the tile is not changed: the event leaves the tile's
  // coordinates in the buffer of its parity (the other buffer may still be read for the previous tile's second
  // block) and ztile tells the next iteration which scores to correct.  No barrier of its own: the coordinates are
  // first read after the barrier at the bottom of the iteration, by the corrections of the two score blocks of
  // that tile at the top of the next iteration and after its first step.
  auto events = [&](auto ahead_c, int t, int koff, bf16x8 (&kp)[2]) __attribute__((always_inline)) {
    if (!STEER) return;
    // one scalar compare in the common case; tiles past the end and unsteered heads have no bit set
    const int tn = t + 1;
    if (__builtin_expect(tn == tile_evt, 0)) {
      const unsigned sh = tn & 63;
      if (sh == 0u) anyw = any_word(tn);
      tile_evt = next_event(tn);
      if ((unsigned)(anyw >> sh) & 1u) {      // (of 32 bits: as a 64-bit test it kept four more scalar registers)
        if (!DENSE) {                    // score-side: the tile stays as it is, its coordinates go to a buffer
          coords_tile(Kst + koff, tn, zbuf + (tn & 1) * PIPE_Z_BYTES);
          ztile = tn;                    // first read after the barrier at the bottom of this iteration
        } else {
          edit_tile(ahead_c, Kst + koff, tn);
          dma_barrier();
#pragma unroll
          for (int i = 0; i < 2; ++i) kp[i] = kfrag(i, koff);
        }
      }
    }
  };

  // One software-pipelined step over three consecutive 32-key blocks: the S^T block at LDS offset KOFF is
  // produced into `next` and the PV products of the block before `cur` (probabilities pb, V rows at ring offset
  // VOFF) are accumulated while the softmax of `cur` runs on the vector ALU; pb then receives the probabilities
  // of `cur`.  Every MFMA of the step has vector work to share the issue port with.
  // The LDS offsets are std::integral_constant in the main loop (they become immediates) and int elsewhere.
  // kpre: the first two K fragments of the block at KOFF, read during the previous step (an LDS read issued right
  // before the MFMA that needs it leaves the wave waiting for the whole LDS latency); on return it holds those of
  // the block at KNEXT, the one the following step scores.
  //
  // No row maximum in the common case.  The probabilities of `cur` are formed against the row's reference exponent
  // as it stands, and their bits tell whether that was safe: they are not negative, so bit 14 or 30 of a packed pair is set if and
  // only if one of them is 2 or more (or not a number), and that
  // means some score ran far ahead of the reference, and only then is the block's maximum computed, the
  // reference raised and the block's probabilities formed again (a handful of times per row; not for its first block, whose
  // maximum the first reference was taken from before the loop, unless that was -inf).  The common case is 16 multiply-adds, 16
  // exponentials, 8 packings and 4 ors per 34 MFMAs: no three-input maxima, no cross-lane exchange, no raise test, and
  // the row sums are two of the MFMAs (as dot products with ones, eight per step, they took a ninth of the step's time).
  auto step = [&](auto koff_c, uint32_t knext, auto voff_c, f32x4 (&cur)[2][2], f32x4 (&next)[2][2], bf16x8 (&pb)[2],
                  bf16x8 (&kpre)[2]) __attribute__((always_inline)) {
    const int KOFF = koff_c, VOFF = voff_c;
    // Program order, one MFMA per slot: the scores of the next block (two per K fragment), the row sums and the outputs of the block before
    // (two per V fragment).  Behind an MFMA comes its share of the LDS reads, issued RA MFMAs ahead of their use, and of the softmax:
    // the multiply-add and the exponential of an element in turn (a run of exponentials stalls the wave in front of the next
    // MFMA), a packing for every second element.
    constexpr int NQ = 4 * KS, NM = NQ + 2 + 2 * DT;        // MFMAs: scores, all
    constexpr int RA = PIPE_RA;
    static_assert(RA <= NQ + 1, "reads start in the step itself");
    bf16x8 kf[2 * KS];
    s16x4 vlo[DT], vhi[DT];
    float x[16], pr[16];
    bf16x2 pk[8];
    kf[0] = kpre[0];
    kf[1] = kpre[1];
    __builtin_amdgcn_sched_barrier(0);
    pipe_static_for<NM>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      if constexpr (m < NQ) {
        constexpr int f = m >> 1, kt = f & 1, rt = m & 1;
        if constexpr (f < 2) pipe_mfma_first(next[kt][rt], kf[f], qf[rt * KS + (f >> 1)]);
        else pipe_mfma(next[kt][rt], kf[f], qf[rt * KS + (f >> 1)]);
      } else if constexpr (m < NQ + 2) {
        pipe_mfma(lacc[m - NQ], ones, pb[m - NQ]);
      } else {
        constexpr int dt = (m - NQ - 2) >> 1, rt = m & 1;
        const bf16x4 lo4 = __builtin_bit_cast(bf16x4, vlo[dt]), hi4 = __builtin_bit_cast(bf16x4, vhi[dt]);
        const bf16x8 va = __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
        pipe_mfma(oacc[dt][rt], va, pb[rt]);
      }
      constexpr int f = pipe_kfrag_at(m, KS, RA);
      if constexpr (f >= 0) kf[f] = kfrag(f, KOFF);
      constexpr int v = m - (NQ + 2 - RA - 1);
      if constexpr (v >= 0 && v < 2 * DT) {
        const uint32_t ad = vaddr[v >> 1] + VOFF;
        if constexpr (v & 1) vhi[v >> 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dma_lds_s16x4_ptr)(uintptr_t)(ad + 16 * RB));
        else vlo[v >> 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dma_lds_s16x4_ptr)(uintptr_t)ad);
      }
      if constexpr (m == NM - 4) kpre[0] = *(pipe_lds_bf16x8_ptr)(uintptr_t)knext;
      if constexpr (m == NM - 2) kpre[1] = *(pipe_lds_bf16x8_ptr)(uintptr_t)(knext + 16 * RB);
      constexpr int e0 = pipe_element_at(m, NM), e1 = pipe_element_at(m - 1, NM), e2 = pipe_element_at(m - 2, NM);
      // (volatile: the compiler would form all of them at the first one's place)
      if constexpr (e0 >= 0) asm volatile("v_fma_f32 %0, %1, %2, -%3" : "=v"(x[e0]) : "v"(cur[(e0 >> 2) & 1][e0 >> 3][e0 & 3]), "s"(c2), "v"(m_run[e0 >> 3]));
      if constexpr (e1 >= 0) pr[e1] = __builtin_amdgcn_exp2f(x[e1]);
      if constexpr (e2 >= 0 && (e2 & 1)) pk[e2 >> 1] = bf16x2{(__bf16)pr[e2 - 1], (__bf16)pr[e2]};
      __builtin_amdgcn_sched_barrier(0);
    });
    bf16x8 pn[2];
    uint32_t bits = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) pn[e >> 3][e & 7] = pk[e >> 1][e & 1];
#pragma unroll
    for (int k = 0; k < 8; k += 2) bits = __builtin_bit_cast(uint32_t, pk[k]) | __builtin_bit_cast(uint32_t, pk[k + 1]) | bits;
    // The probabilities are first used by the next step: without a use here their whole computation is sunk
    // into that step, away from the MFMAs it is meant to share the issue port with.
    asm volatile("" : "+v"(pn[0]), "+v"(pn[1]), "+v"(bits));
    __builtin_amdgcn_sched_barrier(0);
    if (__builtin_expect(__any((bits & 0x40004000u) != 0u), 0)) {
      // `cur` was produced by the previous step's MFMAs: far enough behind for the inline-assembly maxima
      raise_reference(cur);    // after this step's PV product, whose probabilities were formed against the old reference
      block_exp(cur, pn);
    }
    pb[0] = pn[0];
    pb[1] = pn[1];
  };
  // One tile every row of this wave sees in full; ST = t % 3 is compile-time so that every LDS read address is
  // a register plus an immediate.  Enters with S(t, keys 0..31) in sc0 and the probabilities of the block before
  // it in pb; leaves with the same for tile t + 1.
  auto hot = [&](auto st_c, int t) __attribute__((always_inline)) {
    constexpr int ST = decltype(st_c)::value;
    using std::integral_constant;
    // The operand addresses pass through an opaque copy once per tile: otherwise every "address + stage offset"
    // below is hoisted out of the loop into a register of its own (dozens), instead of being an immediate.
    if (STEER && !DENSE && __builtin_expect(ztile == t, 0)) corr(std::true_type{}, t, 0, sc0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kaddr[ks]));
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) asm volatile("" : "+v"(vaddr[dt]));
    step(integral_constant<int, ST * TB + HB>{}, kaddr[0] + ((ST + 1) % 3) * TB, integral_constant<int, ((2 * ST + 5) % 6) * HB>{}, sc0, sc1, pb, kpre);
    if (STEER && !DENSE && __builtin_expect(ztile == t, 0)) corr(std::true_type{}, t, 32, sc1);
    top(std::true_type{}, st_c, t);
    if (kEventsInHot) events(std::true_type{}, t, ((ST + 1) % 3) * TB, kpre);
    step(integral_constant<int, ((ST + 1) % 3) * TB>{}, kaddr[0] + ((ST + 1) % 3) * TB + HB, integral_constant<int, 2 * ST * HB>{}, sc1, sc0, pb, kpre);
    bottom(std::true_type{}, t);
  };

  // A step at run-time ring offsets.  The operand addresses are moved there before the step and back after it: an
  // address formed inside the step is a vector instruction that the order asked for has no place for, and the
  // step's MFMAs then end up in a row in front of its exponentials (4100 cycles per tile instead of the loop's 2700, with 32 x 32 x 16
  // products).
  auto move_addr = [&](uint32_t dk, uint32_t dv) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kaddr[ks] += dk;
      asm volatile("" : "+v"(kaddr[ks]));
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      vaddr[dt] += dv;
      asm volatile("" : "+v"(vaddr[dt]));
    }
  };
  auto ring_step = [&](int koff, int knext, int voff, f32x4 (&cur)[2][2], f32x4 (&next)[2][2]) __attribute__((always_inline)) {
    uint32_t k0 = kaddr[0] + knext;
    asm volatile("" : "+v"(k0));
    move_addr(koff, voff);
    __builtin_amdgcn_sched_barrier(0);
    step(IC0{}, k0, IC0{}, cur, next, pb, kpre);
    move_addr(-koff, -voff);
  };

  // Hot iterations: tile t is seen in full by every row of this wave and tile t + 2 exists and is complete.  They
  // run in whole turns of the ring with a single loop exit (exits after every tile made the compiler park what
  // the code after the loop needs in scratch memory, inside the loop).  Everything else before the wave's last
  // tile runs the same pipelined step with run-time ring offsets and guarded loads (a slower tile).
  // Steering events (a tile to edit, a summary word to reload) are handled inside the hot loop, except in the
  // one shape where that measured slower than leaving the loop for the slower tile: the dense edit with seven
  // waves (Hq=28, Hkv=4, rank 64: 3 % faster outside; dense with eight waves: 3 % faster inside).
  const int t_hot = min(tw_last, min(ntiles, S / BK) - 2);
  int t = 0;
#pragma nounroll
  while (t < tw_last) {
    if (t % 3 == 0) {
      using std::integral_constant;
      // what the loop reads is in registers here (a reload from scratch memory that is first used in the loop is waited for in
      // every turn of it, and with it the tile loads)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kaddr[ks]));
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) asm volatile("" : "+v"(vaddr[dt]));
#pragma unroll
      for (int n = 0; n < SPW; ++n) asm volatile("" : "+v"(koff[n]), "+v"(voff[n]));
      asm volatile("" : "+v"(ones), "+v"(m_run[0]), "+v"(m_run[1]));
#pragma nounroll
      for (; t + 3 <= t_hot && (!STEER || kEventsInHot || tile_evt > t + 3); t += 3) {
        hot(integral_constant<int, 0>{}, t);
        hot(integral_constant<int, 1>{}, t + 1);
        hot(integral_constant<int, 2>{}, t + 2);
      }
      if (t >= tw_last) break;
    }
    top(std::false_type{}, IC0{}, t);
    const int off = (t % 3) * TB, offn = ((t + 1) % 3) * TB;
    if (STEER && !DENSE && ztile == t) corr(std::true_type{}, t, 0, sc0);
    ring_step(off + HB, offn, (int)vpos(2 * t - 1), sc0, sc1);
    if (STEER && !DENSE && ztile == t) corr(std::true_type{}, t, 32, sc1);
    events(std::true_type{}, t, offn, kpre);
    ring_step(offn, offn + HB, (int)vpos(2 * t), sc1, sc0);
    bottom(std::false_type{}, t);
    ++t;
  }
  // ---- the wave's last tile (causal mask, nothing further to score), then idle turns while other waves finish.
  // The second block of that tile may still be in flight during its own iteration (V runs half a tile behind), so
  // its PV product waits for the barrier at the bottom: it is done one turn later, or after the loop. ----
  bool owed = false;                       // wave-uniform: pb holds probabilities whose PV product is outstanding
  int owed_off = 0;
#pragma nounroll
  for (; t < ntiles; ++t) {
    top(std::false_type{}, IC0{}, t);
    const bool zt = STEER && !DENSE && ztile == t;     // before the event of tile t + 1 moves ztile on
    events(std::bool_constant<D == 64>{}, t, ((t + 1) % 3) * TB, kpre);                     // this wave scores nothing further; other waves may (kpre is dead here)
    if (owed) {
      pv_block(owed_off, pb);
      owed = false;
    }
    if (t == tw_last) {
      // A wave whose rows are the first 32 of the tile sees nothing of its second block; one whose rows are the
      // last 32 sees all of its first.
      const int off = (t % 3) * TB;
      const bool second = (qw & 32) != 0;      // wave-uniform
      if (second) qk_block(off + HB, sc1);
      if (zt) {
        corr(std::false_type{}, t, 0, sc0);
        if (second) corr(std::false_type{}, t, 32, sc1);
      }
      if (t > 0) pv_block((int)vpos(2 * t - 1), pb);     // the block before this tile (its softmax ran in the last step)
      auto last_block = [&](bool masked, bool empty, int j0, f32x4 (&sv)[2][2]) __attribute__((always_inline)) {
        if (masked) causal_mask(j0, sv);
        raise_reference(sv, empty);
        block_exp(sv, pb);
      };
      last_block(!second, t == 0, t * BK, sc0);
      pv_block((int)vpos(2 * t), pb);
      if (second) {
        last_block(true, false, t * BK + 32, sc1);
        owed = true;
        owed_off = (int)vpos(2 * t + 1);
      }
    }
    bottom(std::false_type{}, t);
  }
  if (owed) pv_block(owed_off, pb);
  };
  run_block(std::false_type{});

  // ---- next block's first loads (after a barrier: the last PV product above still read the V ring), then this
  // block's output ----
  const int qw_out = qw;
  const int dealt = (pass + 1) * W + (pass & 1 ? slot : W - 1 - slot);    // the next deal's block for this slot
  const bool more = dealt < nblocks;
  if (more) {
    dma_barrier();
    qb = nblocks - 1 - dealt;
    qw = qb * BQ + WR * rb;
    qi0 = qw + l16;
    last_key = min(S, qb * BQ + BQ) - 1;
    ntiles = last_key / BK + 1;
    begin_block();
  }
  if (!more) dma_barrier();    // the staging areas belong to the rings
  // Output: through the staging area, 64 of the 128 columns at a time, so that every store covers eight whole
  // 128-byte lines (straight from the accumulators a store is 32 pieces of 16 bytes: 13000 cycles per block).
  asm volatile("s_nop 15" ::: "memory");   // the last PV product
  pipe_pin_acc(oacc, lacc);
  const int ln = opaque_lane();
  const float inv[2] = {1.f / lacc[0][0], 1.f / lacc[1][0]};
#pragma unroll
  for (int half = 0; half < D / 64; ++half) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int c = 0; c < 4; ++c) {        // columns 64 half + 16 c + 4 grp .. + 3
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(oacc[4 * half + c][rt][e] * inv[rt]);
        *reinterpret_cast<uint2*>(stg_row(ln, rt, 2 * c + (ln >> 5)) + 8 * ((ln >> 4) & 1)) = __builtin_bit_cast(uint2, o4);
      }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int qi = qw_out + 8 * i + (ln >> 3);
      const u32x4 line = *stg_line(ln, i);
      if (qi < S) *reinterpret_cast<u32x4*>(Og + ((tok0 + qi) * a.Hq + hq) * D + 64 * half + 8 * (ln & 7)) = line;
    }
    asm volatile("" ::: "memory");
  }
  // m_run is the reference exponent in units of s * scale * log2(e); the sums are relative to it
  if (a.lse && grp < 2) {                  // lane group rt writes row tile rt
    const int qi = qw_out + lane;
    if (qi < S) a.lse[lse_index(a, b, hq, tok0, qi)] = (grp ? m_run[1] : m_run[0]) * 0.6931471805599453f + logf(grp ? lacc[1][0] : lacc[0][0]);
  }
  if (!more) break;
  }   // for pass
}

}  // namespace seka
