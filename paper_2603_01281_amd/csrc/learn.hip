// Offline stage of SEKA for one layer (paper Sec. 3.1 and 3.4): per KV head, the cross-covariance
// Omega = h^T h_signal / n of token key embeddings, its left singular vectors and singular values, the rank k
// that keeps a fraction gamma of the singular-value mass (Eq. 3), and the head score D_h = mean ||h+ - h-||_2.
//
// Not on the inference path; deterministic throughout (every sum has a fixed order).
//   cov_partial_f32_kernel, cov_partial_mfma_kernel   Omega on the matrix cores, the token range split into chunks (fp32
//                        products and accumulation; exact products of bf16 values).
//   cov_reduce_kernel, gram_kernel   Omega from its partial sums, Omega Omega^T in fp64.
//   tridiag_kernel, eig_kernel   (learn_eig.h) eigenvalues and vectors of the Gram matrix in fp64: singular values and left
//                        singular vectors of Omega.
//   svd_kernel           order, rank rule and packed basis; and where two singular values are too close for the above, or the
//                        samples few (learn_few), the vectors from a pivoted Cholesky factor (fp64) and one-sided (Hestenes) Jacobi: plane rotations
//                        from the right make the factor's columns orthogonal, L V = U Sigma, whatever the gaps are.
//   head_distance_*      token ranges per workgroup, 16-byte loads, partial sums merged in a fixed order.
#include "common.h"
#include "learn_eig.h"

namespace seka {

namespace {

constexpr int kLearnThreads = 256;
constexpr int kCovTokens = 16;          // fp32: tokens per turn
constexpr int kMaxSweeps = 30;
constexpr float kRotateTol = 2e-6f;     // sweeps go on while |a_p . a_q| > tol |a_p| |a_q| (fp32 dot products of length d)
// Few samples: they rotate what is above this as well, so that the last one leaves the columns orthogonal to the rounding of the
// sums (2.7e-7 instead of 2e-6, for less than a microsecond; 3 to 8 % of a sweep over all columns).
constexpr float kRotateFewTol = 2e-7f;
constexpr float kZeroSigma = 1e-5f;     // sigma_c <= this share of sigma_1 is rounding noise: its direction is not determined

__host__ __device__ inline int learn_token_splits(int n) {
  int s = n / 256;
  return s < 1 ? 1 : (s > 32 ? 32 : s);
}

// Omega's partial sums of fp32 tensors: part[((split * Hkv + h) * D + i) * D + j] = sum over the split's tokens of
// hn[t,h,i] hs[t,h,j].  grid ((D / 64)^2, Hkv, splits), four waves with a block of 32 x 32 each, on v_mfma_f32_32x32x2_f32: both
// operands are a row of a block from each of two tokens, 128 bytes in a line, so they go from global memory straight into
// operand registers (two loads per 64-cycle product), 16 tokens ahead of the products.  Bound by latency for a few hundred
// samples (n = 717, 12 heads, D = 128: 77 us with vector FMAs and both views staged in LDS, 18 now), by the fp32 matrix
// rate beyond.
template <int D>
__global__ __launch_bounds__(kLearnThreads) void cov_partial_f32_kernel(const float* __restrict__ hn, const float* __restrict__ hs,
                                                                        int n, int Hkv, int splits, float* __restrict__ part) {
  constexpr int QUADS = D / 64, STEPS = kCovTokens / 2;
  const int h = blockIdx.y, split = blockIdx.z;
  const int per = (n + splits - 1) / splits;
  const int t0 = split * per, t1 = min(n, t0 + per);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5;
  const int i0 = 64 * (blockIdx.x / QUADS) + 32 * (wave >> 1), j0 = 64 * (blockIdx.x % QUADS) + 32 * (wave & 1);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  struct Tokens { float a[STEPS], b[STEPS]; };
  auto fetch = [&](int tb, Tokens& x) __attribute__((always_inline)) {     // past the range: zeros, from a row that exists
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int t = tb + 2 * s + hf;
      const size_t row = ((size_t)min(t, n - 1) * Hkv + h) * D + l32;
      const float a = hn[row + i0], b = hs[row + j0];
      x.a[s] = t < t1 ? a : 0.f;
      x.b[s] = t < t1 ? b : 0.f;
    }
  };
  auto multiply = [&](const Tokens& x) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < STEPS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.a[s], x.b[s], acc, 0, 0, 0);
  };
  Tokens x0, x1;
  fetch(t0, x0);
  for (int tb = t0; tb < t1; tb += 2 * kCovTokens) {
    fetch(tb + kCovTokens, x1);
    multiply(x0);
    fetch(tb + 2 * kCovTokens, x0);
    multiply(x1);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {                 // element r of lane (l32, hf): row 8 (r / 4) + 4 hf + r % 4, column l32
    const int i = i0 + 8 * (r >> 2) + 4 * hf + (r & 3), j = j0 + l32;
    part[(((size_t)split * Hkv + h) * D + i) * D + j] = acc[r];
  }
}

// The same partial sums for bf16 tensors on the matrix cores.  A product of two bf16 values is exact in fp32, so
// v_mfma_f32_32x32x16_bf16 with its fp32 accumulation computes what the fp32 kernel above computes (up to the
// order of the additions) and the kernel is a single pass over both views: grid (splits, Hkv), a workgroup
// stages 64 tokens x D of both views in LDS with 16-byte loads and every wave owns D*D/4096 blocks of 32 x 32 of
// Omega.  Both MFMA operands run along the token axis, the strided one of the row-major [token][d] tiles, hence
// the transposing LDS reads (rows padded by 64 bytes: four consecutive rows, of which 16 lanes read 32 bytes each, fall
// into different banks).
typedef __attribute__((address_space(3))) s16x4* learn_lds_s16x4_ptr;
template <int D>
__global__ __launch_bounds__(kLearnThreads) void cov_partial_mfma_kernel(const uint16_t* __restrict__ hn,
                                                                         const uint16_t* __restrict__ hs, int n, int Hkv,
                                                                         int splits, float* __restrict__ part) {
  constexpr int TOK = 64, LD = D + 32, NB = D / 32, NBW = NB * NB / 4, CPR = D / 8;
  static_assert(NBW >= 1, "at least one block per wave");
  __shared__ __attribute__((aligned(16))) uint16_t a_s[TOK * LD];
  __shared__ __attribute__((aligned(16))) uint16_t b_s[TOK * LD];
  const int split = blockIdx.x, h = blockIdx.y;
  const int per = (n + splits - 1) / splits;
  const int t0 = split * per, t1 = min(n, t0 + per);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, hf = lane >> 5, li = lane & 15, grp = lane >> 4;
  f32x16 acc[NBW];
#pragma unroll
  for (int q = 0; q < NBW; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
  // transposing read of an operand fragment: lanes address row 4 hf + li / 4 (+ 8) of a 16-token slab, columns
  // 16 (grp & 1) + 4 (li & 3) of a 32-column block; the result is lane (column l32, tokens 8 hf .. 8 hf + 7)
  const int frag_off = (4 * hf + (li >> 2)) * LD + 16 * (grp & 1) + 4 * (li & 3);
  auto frag = [&](const uint16_t* tile, int slab, int blk) __attribute__((always_inline)) -> bf16x8 {
    const uint16_t* p = tile + frag_off + (16 * slab) * LD + 32 * blk;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((learn_lds_s16x4_ptr)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((learn_lds_s16x4_ptr)(p + 8 * LD));
    return __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi), 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // the next 64 tokens travel through registers while the current ones are multiplied
  constexpr int NLD = TOK * CPR / kLearnThreads;
  static_assert(TOK * CPR % kLearnThreads == 0, "whole turns");
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  u32x4 ra[NLD], rb[NLD];
  auto fetch = [&](int tb) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int idx = threadIdx.x + k * kLearnThreads, tt = idx / CPR, c = idx % CPR, t = tb + tt;
      ra[k] = u32x4{0, 0, 0, 0};
      rb[k] = u32x4{0, 0, 0, 0};
      if (t < t1) {
        ra[k] = *reinterpret_cast<const u32x4*>(hn + ((size_t)t * Hkv + h) * D + 8 * c);
        rb[k] = *reinterpret_cast<const u32x4*>(hs + ((size_t)t * Hkv + h) * D + 8 * c);
      }
    }
  };
  if (t0 < t1) fetch(t0);
  for (int tb = t0; tb < t1; tb += TOK) {
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int idx = threadIdx.x + k * kLearnThreads, tt = idx / CPR, c = idx % CPR;
      *reinterpret_cast<u32x4*>(a_s + tt * LD + 8 * c) = ra[k];
      *reinterpret_cast<u32x4*>(b_s + tt * LD + 8 * c) = rb[k];
    }
    __syncthreads();
    if (tb + TOK < t1) fetch(tb + TOK);
#pragma unroll
    for (int slab = 0; slab < TOK / 16; ++slab) {
#pragma unroll
      for (int q = 0; q < NBW; ++q) {
        const int blk = wave * NBW + q, ib = blk / NB, jb = blk % NB;
        acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a_s, slab, ib), frag(b_s, slab, jb), acc[q], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  // accumulator element r of lane (l32, hf): row 8 (r / 4) + 4 hf + r % 4 of the block, column l32
#pragma unroll
  for (int q = 0; q < NBW; ++q) {
    const int blk = wave * NBW + q, ib = blk / NB, jb = blk % NB;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 32 * ib + 8 * (r >> 2) + 4 * hf + (r & 3), j = 32 * jb + l32;
      part[(((size_t)split * Hkv + h) * D + i) * D + j] = acc[q][r];
    }
  }
}

// Omega = (sum of the token splits, in order) / n, over the first split's slots.  grid-stride over 4-element pieces.
__global__ __launch_bounds__(kLearnThreads) void cov_reduce_kernel(float* __restrict__ part, size_t elems, int splits, float inv_n) {
  const size_t e = ((size_t)blockIdx.x * kLearnThreads + threadIdx.x) * 4;
  if (e >= elems) return;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int sp = 0; sp < splits; ++sp) s += *reinterpret_cast<const f32x4*>(part + (size_t)sp * elems + e);
  *reinterpret_cast<f32x4*>(part + e) = s * inv_n;
}

// B = Omega Omega^T in fp64 (a product of two fp32 values is exact there).  grid (D / 8, D / 64, Hkv): 8 rows x 64
// columns of B per workgroup, which needs 72 rows of Omega in LDS (rows padded by 16 bytes: 16-byte reads down a
// column of rows without bank conflicts).
template <int D>
__global__ __launch_bounds__(kLearnThreads) void gram_kernel(const float* __restrict__ omega, double* __restrict__ gram) {
  constexpr int LD = D + 4, P = D / 4;                           // 16-byte pieces per row
  constexpr int NLD = (72 * P + kLearnThreads - 1) / kLearnThreads;     // surplus threads repeat the last piece
  __shared__ __attribute__((aligned(16))) float om[72 * LD];     // rows c0 .. c0 + 63, then r0 .. r0 + 7
  const int h = blockIdx.z, r0 = 8 * blockIdx.x, c0 = 64 * blockIdx.y;
  f32x4 v[NLD];
#pragma unroll
  for (int k = 0; k < NLD; ++k) {
    const int idx = min((int)threadIdx.x + k * kLearnThreads, 72 * P - 1), row = idx / P;
    v[k] = *reinterpret_cast<const f32x4*>(omega + ((size_t)h * D + (row < 64 ? c0 + row : r0 + row - 64)) * D + 4 * (idx % P));
  }
#pragma unroll
  for (int k = 0; k < NLD; ++k) {
    const int idx = min((int)threadIdx.x + k * kLearnThreads, 72 * P - 1);
    *reinterpret_cast<f32x4*>(om + (idx / P) * LD + 4 * (idx % P)) = v[k];
  }
  __syncthreads();
  const int c = threadIdx.x & 63, r = 2 * (threadIdx.x >> 6);    // one column, rows r and r + 1
  double acc0 = 0.0, acc1 = 0.0;
#pragma unroll 4
  for (int j = 0; j < D; j += 4) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(om + c * LD + j);
    const f32x4 y0 = *reinterpret_cast<const f32x4*>(om + (64 + r) * LD + j), y1 = *reinterpret_cast<const f32x4*>(om + (65 + r) * LD + j);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc0 = __builtin_fma((double)y0[e], (double)x[e], acc0);
      acc1 = __builtin_fma((double)y1[e], (double)x[e], acc1);
    }
  }
  double* g = gram + ((size_t)h * D + r0 + r) * D + c0 + c;
  g[0] = acc0;
  g[D] = acc1;
}

// value of lane (l + DPP pattern) within the 16-lane row
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// Eight sums over the 64 lanes at once: lane l receives the total of v[l / 8].
__device__ __forceinline__ float reduce8(const float (&v)[8], int lane) {
  float a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 4]), false, false);
    a[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[i]), __float_as_uint(a[i + 2]), false, false);
    b[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
  const bool up = (lane & 8) != 0;
  float r = (up ? b[1] : b[0]) + dpp<0x128>(up ? b[0] : b[1]);   // row_ror:8
  r += dpp<0xB1>(r);                                             // lane ^ 1
  r += dpp<0x4E>(r);                                             // lane ^ 2
  r += dpp<0x141>(r);                                            // mirrored in 8
  return r;
}

// Rank rule and packed basis of one head, and its singular values and vectors where the tridiagonal path cannot tell two
// directions apart: squares closer than 1e-13 of the largest one (they come with about 1e-15) or than 1e-7 of themselves
// (its vectors are then orthogonal to 1e-7 at worst).  Values of samples with noise are further apart by orders of magnitude
// (smallest gap in 128 of them: 3e-3 of the value); equal ones are what the iteration is for.
// grid (Hkv), one workgroup of D / 16 waves per head.  8 heads, D = 128: 12 us, and 107 + 54 for the two kernels before it;
// with the iteration for every head, as it was: 654.
//
// Phase 1, Cholesky with diagonal pivoting, B = L L^T, in fp64: Omega and L have the same left singular vectors and
// singular values (up to rotations from the right), and L, whose columns come out nearly sorted and nearly
// orthogonal, needs about half the Jacobi sweeps that Omega needs.  fp64 because B holds squares: what falls below 1e-14
// of its largest element is below 1e-7 of sigma_1, and is dropped.  B lives in registers (a thread has a tile of
// D / 16 x 4 or 4 x 4); every wave keeps the diagonal and finds the pivot by itself, so a step has one barrier.
//
// Phase 2, one-sided Jacobi on L in fp32 in blocks of 8 columns: a wave holds two blocks (16 columns, D / 64 rows per
// lane) in registers and rotates all pairs across them (8 rounds of 8 disjoint pairs, registers named at compile
// time, the 8 dot products of a round reduced together); then blocks change partners through LDS (a round-robin
// tournament of the blocks: D / 8 - 1 exchanges per sweep instead of one barrier per round of pairs).  Pairs inside a
// block are rotated once per sweep.  A rotation is applied as three shears.  Sweeps repeat until one finds nothing above kRotateTol.
// What bounds it: vector issue on the head's CU (about 140 instructions per round and wave, two waves per SIMD: 11 k
// cycles per exchange of blocks; 8 or 9 sweeps).
template <typename T, int D>
__global__ __launch_bounds__(4 * D) void svd_kernel(const double* __restrict__ gram, const float* __restrict__ omega, float gamma, float* __restrict__ U_out,
                                                    float* __restrict__ sigma_out, int* __restrict__ k_out,
                                                    T* __restrict__ U_packed, int r_pad, int few) {
  constexpr int NW = D / 16, NT = 64 * NW;
  constexpr int RPL = D / 64;                     // rows per lane
  constexpr int LD = D + RPL;                     // column stride in floats
  typedef float rows_t __attribute__((ext_vector_type(RPL)));
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* A = lds;                                 // [D columns][LD]
  double* colbuf = reinterpret_cast<double*>(lds + D * LD);      // [2][D]
  float* sig = lds + D * LD + 4 * D;              // [D]
  float* sorted_s = sig + D;                      // [D]
  int* by_rank = reinterpret_cast<int*>(sorted_s + D);           // [D] column of the r-th largest value
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto store_packed = [&](int i, int r, float v) __attribute__((always_inline)) {      // row i, column r < r_pad
    const size_t at = ((size_t)h * D + i) * r_pad + r;
    if (sizeof(T) == 2) {
      const __bf16 bv = (__bf16)v;
      reinterpret_cast<uint16_t*>(U_packed)[at] = __builtin_bit_cast(uint16_t, bv);
    } else {
      reinterpret_cast<float*>(U_packed)[at] = v;
    }
  };

  // ---- what the tridiagonal path found ----
  typedef EigWork<D> W;
  const double* work = reinterpret_cast<const double*>(omega + (size_t)h * D * D);
  const bool known = !few && work[W::kStatus] == 0.0;              // it ran, on an Omega that is finite
  bool alike = !known;                            // two directions that it cannot tell apart
  if (known) {
    if (tid < D) {                                // thread r: the r-th largest
      const double top = work[W::kLambda + D - 1], me = work[W::kLambda + D - 1 - tid];
      const double next = tid < D - 1 ? work[W::kLambda + D - 2 - tid] : -top;
      const bool kept = me > (double)kZeroSigma * kZeroSigma * top;
      alike = !is_finite(me) || (kept && (me - next < fmax(1e-13 * top, 1e-7 * me) || reinterpret_cast<const int*>(work + W::kBad)[D - 1 - tid] != 0));
      sig[tid] = me > 1e-14 * top ? (float)sqrt(me) : 0.f;         // below: rounding of the squares
    }
    alike = __syncthreads_or(alike);
  }
  float unit = known ? (float)work[W::kUnit] : 0.f;
  if (alike) {
  // ---- phase 1 ----
  // unit: sqrt of B's largest element, L is scaled by its inverse
  int ncols = D;
  {
    constexpr int TR = D * D / NT / 4;            // a thread holds TR rows x 4 columns (8 or 4 rows)
    const int tr = TR * (tid / (D / 4)), tc = 4 * (tid % (D / 4));
    const double* Bh = gram + (size_t)h * D * D;
    double a[TR][4], d[RPL];
#pragma unroll
    for (int i = 0; i < TR; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {               // the lower triangle: reflectors stand in the other, if there are any
        const int r = tr + i, c = tc + j;
        a[i][j] = Bh[few ? r * D + c : max(r, c) * D + min(r, c)];
      }
#pragma unroll
    for (int x = 0; x < RPL; ++x) d[x] = Bh[(size_t)(lane + 64 * x) * (D + 1)];
    unsigned top = 0;                             // high word of the largest diagonal element (they are sums of squares)
#pragma unroll
    for (int x = 0; x < RPL; ++x) top = max(top, (unsigned)(__builtin_bit_cast(unsigned long long, d[x]) >> 32) & 0x7fffffffu);
    top = wave_max(top);
    if (top >= 0x7ff00000u) {                     // Omega is not finite: neither is what is made of it (the same in every wave)
      const float nan = __builtin_nanf("");
      for (int idx = tid; idx < D * D; idx += NT) U_out[(size_t)h * D * D + idx] = nan;
      if (tid < D) sigma_out[(size_t)h * D + tid] = nan;
      if (tid == 0) k_out[h] = D;
      if (U_packed)
        for (int idx = tid; idx < D * r_pad; idx += NT) store_packed(idx / r_pad, idx % r_pad, nan);
      return;
    }
    // The factorisation runs on 2^-e B, e even, whose largest element lies in [1, 4): B's own, from 2^-298 to 2^263, and
    // their reciprocals leave fp32, in which the pivots are compared and L is stored.  Powers of two: no bit changes.
    const int e = top ? ((int)(top >> 20) - 1023) & ~1 : 0;
    const double down = __builtin_bit_cast(double, (unsigned long long)(1023 - e) << 52);
    const double up_half = __builtin_bit_cast(double, (unsigned long long)(1023 + e / 2) << 52);
#pragma unroll
    for (int i = 0; i < TR; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) a[i][j] *= down;
#pragma unroll
    for (int x = 0; x < RPL; ++x) d[x] *= down;
    double floor_d = 0.0;
    float key_scale = 1.f;
    unit = 0.f;
    for (int k = 0; k < D; ++k) {
      // pivot: the largest remaining diagonal element (to 17 bits; the lower ones carry its index)
      unsigned key = 0;
#pragma unroll
      for (int x = 0; x < RPL; ++x)
        key = max(key, d[x] > 0.0 ? (__float_as_uint((float)d[x] * key_scale) & ~127u) | (unsigned)(lane + 64 * x) : 0u);
      const int p = (int)(wave_max(key) & 127u);
      double dp = d[0];
#pragma unroll
      for (int x = 1; x < RPL; ++x) dp = (p >> 6) == x ? d[x] : dp;
      dp = lane_double(dp, p & 63);
      if (k == 0) {
        floor_d = 1e-14 * dp;
        unit = (float)(sqrt(dp) * up_half);
        key_scale = dp > 0.0 ? (float)(1.0 / dp) : 0.f;
      }
      if (!(dp > floor_d)) { ncols = k; break; }  // the same in every wave: same data, same operations
      // row p of what is left of B, as it stands: l_k = row / sqrt(dp)
      double* row = colbuf + (k & 1) * D;
      if (tr == (p & ~(TR - 1))) {
#pragma unroll
        for (int i = 0; i < TR; ++i)
          if ((p & (TR - 1)) == i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) row[tc + j] = a[i][j];
          }
      }
      double inv = __builtin_amdgcn_rcp(dp);      // 1 / dp: hardware estimate and two Newton steps
      inv = __builtin_fma(__builtin_fma(-dp, inv, 1.0), inv, inv);
      inv = __builtin_fma(__builtin_fma(-dp, inv, 1.0), inv, inv);
      __syncthreads();
      double rv[TR], cv[4], dv[RPL];
#pragma unroll
      for (int j = 0; j < 4; ++j) cv[j] = row[tc + j] * inv;
#pragma unroll
      for (int i = 0; i < TR; ++i) rv[i] = row[tr + i];
#pragma unroll
      for (int x = 0; x < RPL; ++x) dv[x] = row[lane + 64 * x];
#pragma unroll
      for (int x = 0; x < RPL; ++x) d[x] = lane + 64 * x == p || d[x] <= 0.0 ? 0.0 : __builtin_fma(-dv[x] * inv, dv[x], d[x]);
#pragma unroll
      for (int i = 0; i < TR; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) a[i][j] = __builtin_fma(-rv[i], cv[j], a[i][j]);
      if (wave == (k & (NW - 1))) {               // one wave writes the column of L
        const float rho = (float)dp * key_scale;  // of the largest element
        float f = __builtin_amdgcn_rsqf(rho);
        f = f * __builtin_fmaf(-0.5f * rho * f, f, 1.5f) * key_scale;
#pragma unroll
        for (int x = 0; x < RPL; ++x) A[k * LD + lane + 64 * x] = (float)dv[x] * f;
      }
    }
    for (int idx = tid; idx < (D - ncols) * LD; idx += NT) A[ncols * LD + idx] = 0.f;
    __syncthreads();
  }

  // ---- phase 2 ----
  const int nblk = max(2, ((ncols + 7) / 8 + 1) & ~1);           // blocks that take part (even)
  const float rotate_tol2 = few ? kRotateFewTol * kRotateFewTol : kRotateTol * kRotateTol;
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    int rotated = 0;
    for (int step = 0; step < nblk - 1; ++step) {
      if (wave < nblk / 2) {
        auto at = [&](int pos) {                  // round-robin: position 0 stays, the others rotate
          if (pos == 0) return 0;
          const int x = pos - 1 + step;
          return (x >= nblk - 1 ? x - (nblk - 1) : x) + 1;
        };
        float* base[2] = {A + 8 * at(wave) * LD, A + 8 * at(nblk - 1 - wave) * LD};
        rows_t x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = *reinterpret_cast<const rows_t*>(base[j / 8] + (j & 7) * LD + RPL * lane);
        auto dot = [&](int p, int q) __attribute__((always_inline)) -> float {
          float s = x[p][0] * x[q][0];
#pragma unroll
          for (int i = 1; i < RPL; ++i) s = __builtin_fmaf(x[p][i], x[q][i], s);
          return s;
        };
        // rotation of the lane's pair from its norms and dot product; returns t (0: leave the pair alone), sine and
        // tangent of half the angle, and whether another sweep is asked for
        auto angle = [&](float al, float be, float ga, float& sn, float& th, int& more) __attribute__((always_inline)) -> float {
          const bool rot = ga * ga > rotate_tol2 * (al * be);      // norms are 0 or in [1e-7, 1]
          more |= __any(ga * ga > (kRotateTol * kRotateTol) * (al * be));
          const float df = be - al, g2 = ga + ga;
          float t = g2 * __builtin_amdgcn_rcpf(df + copysignf(__builtin_amdgcn_sqrtf(__builtin_fmaf(df, df, g2 * g2)), df));
          t = rot ? t : 0.f;
          const float w = __builtin_fmaf(t, t, 1.f);
          float c = __builtin_amdgcn_rsqf(w);
          c = c * __builtin_fmaf(-0.5f * w * c, c, 1.5f);
          sn = c * t;
          th = sn * __builtin_amdgcn_rcpf(1.f + c);
          return t;
        };
        auto apply = [&](int p, int q, float sn, float th) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < RPL; ++i) {
            const float x1 = __builtin_fmaf(-th, x[q][i], x[p][i]);
            x[q][i] = __builtin_fmaf(sn, x1, x[q][i]);
            x[p][i] = __builtin_fmaf(-th, x[q][i], x1);
          }
        };
        auto lane_value = [&](float v, int j) __attribute__((always_inline)) {
          return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 8 * j));
        };
        if (step == 0) {                          // pairs inside the blocks: 7 rounds of 4 pairs in each
#pragma unroll
          for (int r = 0; r < 7; ++r) {
            // round-robin of 8: player 7 stays; pairs (7, r), (r + k, r - k) mod 7
            float va[8], vb[8], vg[8];
            int P[8], Q[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int k = j & 3, o = 8 * (j >> 2);
              P[j] = o + (k == 0 ? 7 : (r + k) % 7);
              Q[j] = o + (k == 0 ? r : (r - k + 7) % 7);
              va[j] = dot(P[j], P[j]);
              vb[j] = dot(Q[j], Q[j]);
              vg[j] = dot(P[j], Q[j]);
            }
            const float al = reduce8(va, lane), be = reduce8(vb, lane), ga = reduce8(vg, lane);
            float sn, th;
            angle(al, be, ga, sn, th, rotated);
#pragma unroll
            for (int j = 0; j < 8; ++j) apply(P[j], Q[j], lane_value(sn, j), lane_value(th, j));
          }
        }
        // pairs across the blocks: in round r lanes 8 p .. 8 p + 7 look after columns p and 8 + (p + r) % 8; the norms
        // are formed once and updated with each rotation
        float va[8], vb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) { va[j] = dot(j, j); vb[j] = dot(8 + j, 8 + j); }
        float al = reduce8(va, lane), be = reduce8(vb, lane);
        const int next_lane = ((lane + 8) & 63) * 4;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          float vg[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) vg[j] = dot(j, 8 + ((j + r) & 7));
          const float ga = reduce8(vg, lane);
          float sn, th;
          const float t = angle(al, be, ga, sn, th, rotated);
          if (__any(t != 0.f)) {                  // the last sweeps rotate few pairs
            al = fmaxf(__builtin_fmaf(-t, ga, al), 0.f);
            be = fmaxf(__builtin_fmaf(t, ga, be), 0.f);
#pragma unroll
            for (int j = 0; j < 8; ++j) apply(j, 8 + ((j + r) & 7), lane_value(sn, j), lane_value(th, j));
          }
          be = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(next_lane, __builtin_bit_cast(int, be)));
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) *reinterpret_cast<rows_t*>(base[j / 8] + (j & 7) * LD + RPL * lane) = x[j];
      }
      __syncthreads();                            // a block is read and written by the wave that holds it only
    }
    if (!__syncthreads_or(rotated)) break;
  }

  // ---- singular values = column norms; order them (descending, ties by column index) ----
  for (int c = wave; c < D; c += NW) {
    const rows_t v = *reinterpret_cast<const rows_t*>(A + c * LD + RPL * lane);
    float s2 = v[0] * v[0];
#pragma unroll
    for (int i = 1; i < RPL; ++i) s2 = __builtin_fmaf(v[i], v[i], s2);
#pragma unroll
    for (int s = 1; s < 64; s *= 2) s2 += __shfl_xor(s2, s);
    if (lane == 0) sig[c] = sqrtf(s2);
  }
  __syncthreads();
  }
  if (tid < D) {
    // compared as bits, which order non-negative values and leave no two of them unordered: every rank is written,
    // whatever the values are
    const unsigned me = __float_as_uint(sig[tid]);
    int r = 0;
#pragma unroll 8
    for (int k = 0; k < D; ++k) {
      const unsigned other = __float_as_uint(sig[k]);
      r += (other > me) || (other == me && k < tid);
    }
    by_rank[r] = tid;
    sorted_s[r] = sig[tid];
    sigma_out[(size_t)h * D + r] = sig[tid] * unit;
  }
  __syncthreads();
  // Rank rule of Eq. 3: the smallest k whose leading values reach gamma of the sum; every wave works it out by itself.
  // One chain of additions in index order: its sums never decrease and stay at the total from the last value that counts
  // on, so at gamma = 1 the zeros behind it are not asked for.  (Sums in another association differ in the last bit.)
  int k_sel;
  {
#pragma clang fp reassociate(off)
    float run[RPL], total = 0.f;                  // lane l keeps the sums up to l and up to 64 + l
#pragma unroll 8
    for (int k = 0; k < D; ++k) {
      total += sorted_s[k];
#pragma unroll
      for (int x = 0; x < RPL; ++x) run[x] = k == 64 * x + lane ? total : run[x];
    }
    int below = 0;
#pragma unroll
    for (int x = 0; x < RPL; ++x) below += __popcll(__ballot(!(run[x] >= gamma * total)));
    k_sel = min(below + 1, D);
    if (tid == 0) k_out[h] = k_sel;
  }
  static_assert(NT % D == 0, "a thread keeps its output column");
  const int r = tid % D, j = by_rank[r];
  const float s = sorted_s[r], s_inv = s > kZeroSigma * sorted_s[0] ? 1.f / s : 0.f;
  if (!alike) {                                   // the columns are there
    if (s_inv == 0.f)
      for (int i = tid / D; i < D; i += NT / D) U_out[((size_t)h * D + i) * D + r] = 0.f;
    if (U_packed) {
#pragma unroll 4
      for (int idx = tid; idx < D * r_pad; idx += NT) {
        const int i = idx / r_pad, c = idx % r_pad;
        const float u = U_out[((size_t)h * D + i) * D + c];
        store_packed(i, c, c < k_sel && sorted_s[c] > kZeroSigma * sorted_s[0] ? u : 0.f);
      }
    }
    return;
  }
#pragma unroll 8
  for (int i = tid / D; i < D; i += NT / D) {
    const float u = A[j * LD + i] * s_inv;
    U_out[((size_t)h * D + i) * D + r] = u;
    if (U_packed && r < r_pad) store_packed(i, r, r < k_sel ? u : 0.f);
  }
}

// Samples up to which every head goes straight to the iteration.  Omega of n samples has no more than n directions, columns of
// the pivoted factor that the iteration's time grows with; that of the tridiagonal form grows with the rounds that eig_kernel's D / 4
// workgroups per head make on the 256 compute units.  Rounding Omega to fp32 leaves fp32 samples further columns, bf16 samples
// fewer; the line for fp32 lies between that of samples whose spectrum decays (first figure) and of gaussian ones.  us,
// iteration / tridiagonal form: D = 128, 8 heads fp32 n = 1 38 / 184, n = 28 161, 185 / 185, n = 32 165, 227 / 185, bf16 n = 44
// 187, 173 / 185; 12 heads fp32 n = 32 177, 228 / 230, n = 40 187, 261 / 232; 32 heads fp32 n = 44 242, 410 / 336, bf16 n = 64 250, 249 /
// 336; 64 heads fp32 n = 64 416, 539 / 530, bf16 n = 80 490, 492 / 532; D = 64, 8 heads fp32 n = 16 79, 80 / 85, 64 heads bf16 n = 48
// 146, 146 / 165.
inline int learn_few(int Hkv, int D, bool bf16) {
  const int rounds = (Hkv * (D / 4) + 255) / 256;
  if (D == 64) return bf16 ? 12 + 10 * rounds : 10 + 8 * rounds;
  return bf16 ? 40 + 6 * rounds : 26 + 5 * rounds;
}

// grid (splits, Hkv): part[h * splits + split] = sum over the split's tokens of || hp[t,h,:] - hm[t,h,:] ||_2.
// A row is D / 8 (bf16) or D / 4 (fp32) consecutive lanes with one 16-byte load each; fixed-order merges throughout.
template <typename T, int D>
__global__ __launch_bounds__(kLearnThreads) void head_distance_partial_kernel(const T* __restrict__ hp, const T* __restrict__ hm,
                                                                              int n, int Hkv, int splits, float* __restrict__ part) {
  constexpr int EPL = 16 / sizeof(T);               // elements per lane
  constexpr int LPR = D / EPL;                      // lanes per row (8, 16 or 32)
  constexpr int RPT = kLearnThreads / LPR;          // rows per workgroup turn
  __shared__ float wsum[kLearnThreads / 64];
  const int split = blockIdx.x, h = blockIdx.y;
  const int per = (n + splits - 1) / splits;
  const int t0 = split * per, t1 = min(n, t0 + per);
  const int c = threadIdx.x % LPR, rr = threadIdx.x / LPR;
  float acc = 0.f;
  for (int tb = t0; tb < t1; tb += RPT) {           // workgroup-uniform trip count
    const int t = tb + rr;
    const bool ok = t < t1;
    const size_t off = ((size_t)(ok ? t : t1 - 1) * Hkv + h) * D + c * EPL;      // clamped: loads stay inside the tensors
    const uint4 a = *reinterpret_cast<const uint4*>(hp + off), b = *reinterpret_cast<const uint4*>(hm + off);
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
    float s2 = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (sizeof(T) == 2) {
        const float d0 = __uint_as_float(aw[i] << 16) - __uint_as_float(bw[i] << 16);
        const float d1 = __uint_as_float(aw[i] & 0xffff0000u) - __uint_as_float(bw[i] & 0xffff0000u);
        s2 = fmaf(d0, d0, s2);
        s2 = fmaf(d1, d1, s2);
      } else {
        const float d0 = __uint_as_float(aw[i]) - __uint_as_float(bw[i]);
        s2 = fmaf(d0, d0, s2);
      }
    }
#pragma unroll
    for (int d = 1; d < LPR; d *= 2) s2 += __shfl_xor(s2, d);
    if (ok && c == 0) acc += sqrtf(s2);
  }
#pragma unroll
  for (int d = 1; d < 64; d *= 2) acc += __shfl_xor(acc, d);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float s = 0.f;
    for (int w = 0; w < kLearnThreads / 64; ++w) s += wsum[w];
    part[(size_t)h * splits + split] = s;
  }
}

// grid (Hkv), one wave: D_h = (sum of the head's partials, in a fixed order) / n
__global__ void head_distance_finish_kernel(const float* __restrict__ part, int splits, float inv_n, float* __restrict__ D_out) {
  float s = 0.f;
  for (int i = threadIdx.x; i < splits; i += 64) s += part[(size_t)blockIdx.x * splits + i];
#pragma unroll
  for (int d = 1; d < 64; d *= 2) s += __shfl_xor(s, d);
  if (threadIdx.x == 0) D_out[blockIdx.x] = s * inv_n;
}

template <typename T, int D>
hipError_t launch_learn_td(const void* hn, const void* hs, int n, int Hkv, float gamma, float* U_out, float* sigma_out,
                           int* k_out, void* U_packed, int r_pad, float* part, hipStream_t s) {
  const int splits = learn_token_splits(n);
  if constexpr (sizeof(T) == 2)
    hipLaunchKernelGGL((cov_partial_mfma_kernel<D>), dim3(splits, Hkv), dim3(kLearnThreads), 0, s,
                       static_cast<const uint16_t*>(hn), static_cast<const uint16_t*>(hs), n, Hkv, splits, part);
  else
    hipLaunchKernelGGL((cov_partial_f32_kernel<D>), dim3((D / 64) * (D / 64), Hkv, splits), dim3(kLearnThreads), 0, s,
                       static_cast<const float*>(hn), static_cast<const float*>(hs), n, Hkv, splits, part);
  const size_t elems = (size_t)Hkv * D * D;
  double* gram = reinterpret_cast<double*>(part + elems);          // over the other splits' slots (learn_workspace_bytes has room)
  hipLaunchKernelGGL(cov_reduce_kernel, dim3((unsigned)((elems / 4 + kLearnThreads - 1) / kLearnThreads)), dim3(kLearnThreads), 0, s,
                     part, elems, splits, 1.0f / (float)n);
  hipLaunchKernelGGL((gram_kernel<D>), dim3(D / 8, D / 64, Hkv), dim3(kLearnThreads), 0, s, part, gram);
  const size_t smem = ((size_t)D * (D + D / 64) + 7 * D) * sizeof(float);
  auto kernel = svd_kernel<T, D>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  const bool few = n <= learn_few(Hkv, D, sizeof(T) == 2);
  if (!few) {
    hipLaunchKernelGGL((tridiag_kernel<D>), dim3(Hkv), dim3(256), 0, s, gram, part);
    hipLaunchKernelGGL((eig_kernel<D>), dim3(D / 4, Hkv), dim3(kEigThreads), 0, s, gram, part, U_out, 0.9 * kZeroSigma * kZeroSigma);
  }
  hipLaunchKernelGGL(kernel, dim3(Hkv), dim3(4 * D), smem, s, gram, part, gamma, U_out, sigma_out, k_out, static_cast<T*>(U_packed), r_pad, (int)few);
  return hipGetLastError();
}

}  // namespace

// token ranges of the head-distance pass: about 2048 workgroups in all, at least 256 tokens each
static inline int distance_splits(int n, int Hkv) {
  int want = (2048 + Hkv - 1) / Hkv;
  const int cap = n / 256 > 1 ? n / 256 : 1;
  if (want > cap) want = cap;
  return want > 1024 ? 1024 : want;
}

size_t learn_workspace_bytes(int Hkv, int D, int n) {
  const int splits = learn_token_splits(n);                        // at least Omega (fp32) and its Gram matrix (fp64)
  const size_t cov = (size_t)(splits > 3 ? splits : 3) * Hkv * D * D * sizeof(float);
  const size_t dist = ((size_t)distance_splits(n, Hkv) * Hkv * sizeof(float) + 15) / 16 * 16;
  return cov > dist ? cov : dist;
}

hipError_t launch_learn(const void* hn, const void* hs, int n, int Hkv, int D, int dtype, float gamma, float* U_out,
                        float* sigma_out, int* k_out, void* U_packed, int r_pad, void* workspace, hipStream_t s) {
  float* part = static_cast<float*>(workspace);
  if (dtype == SEKA_BF16)
    return D == 128 ? launch_learn_td<uint16_t, 128>(hn, hs, n, Hkv, gamma, U_out, sigma_out, k_out, U_packed, r_pad, part, s)
                    : launch_learn_td<uint16_t, 64>(hn, hs, n, Hkv, gamma, U_out, sigma_out, k_out, U_packed, r_pad, part, s);
  return D == 128 ? launch_learn_td<float, 128>(hn, hs, n, Hkv, gamma, U_out, sigma_out, k_out, U_packed, r_pad, part, s)
                  : launch_learn_td<float, 64>(hn, hs, n, Hkv, gamma, U_out, sigma_out, k_out, U_packed, r_pad, part, s);
}

hipError_t launch_head_distance(const void* hp, const void* hm, int n, int Hkv, int D, int dtype, float* D_out,
                                void* workspace, hipStream_t s) {
  const int splits = distance_splits(n, Hkv);
  float* part = static_cast<float*>(workspace);
#define SEKA_HD_CASE(T, DD) \
  hipLaunchKernelGGL((head_distance_partial_kernel<T, DD>), dim3(splits, Hkv), dim3(kLearnThreads), 0, s, \
                     static_cast<const T*>(hp), static_cast<const T*>(hm), n, Hkv, splits, part)
  if (dtype == SEKA_BF16) { if (D == 128) SEKA_HD_CASE(uint16_t, 128); else SEKA_HD_CASE(uint16_t, 64); }
  else { if (D == 128) SEKA_HD_CASE(float, 128); else SEKA_HD_CASE(float, 64); }
#undef SEKA_HD_CASE
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(head_distance_finish_kernel, dim3(Hkv), dim3(64), 0, s, part, splits, 1.0f / (float)n, D_out);
  return hipGetLastError();
}

}  // namespace seka
