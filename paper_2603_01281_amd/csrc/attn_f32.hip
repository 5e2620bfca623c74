// fp32 causal GQA attention with the key edit fused in (paper Sec. 2: scores q.k'/sqrt(d_k); k' = a k + g P k
// on highlighted tokens).  The exact-arithmetic path: every product is an fp32 multiply-add with fp32 accumulation,
// on the matrix cores (v_mfma_f32_16x16x4_f32; their fp32 rate is twice what plain vector FMAs reach, and an operand
// is one register per lane instead of an LDS broadcast per multiply).
//
// Mapping: one unit of work = 16 query rows of one head, held by a wave as B operands.  Keys are taken 16 at a time:
// S^T = K Q^T, so a lane owns query row l % 16 and the keys 4 (l / 16) + i, which is already the operand order of
// O^T += V^T P^T.  K and V go from global memory straight into operand registers with 16-byte loads (the order of
// the contraction over d, and of the rows of V^T, is permuted so that a lane's four elements are contiguous), one
// step ahead of the products; nothing is staged in LDS.  The step of 64 products covers the L2 latency.
//
// The edit is applied to the scores (Sec. 2, the equivalence of key-side and score-side control):
// s_ij = a q_i.k_j + (U^T q_i).(c .* U^T k_j) for highlighted j.  U^T k of a block with highlights is one more product
// against operands already in registers; in the accumulator layout it is the A operand of the correction as it stands.
//
// What bounds it: small problems, latency: few waves exist, so the keys of a unit are split over the four waves of
// a workgroup (KSPLIT = 4) and merged through LDS at the end.  Large ones, the operand loads from L1 / L2 (16 KB per 64
// products): four units that share their keys form a workgroup (KSPLIT = 1), and a wave takes the four parts of its keys
// one after the other, which gives the bits of the split form (0 to 5 % of a short launch, none of a long one).  The form before this one (scalar FMAs, keys
// and probabilities broadcast from LDS, the edit as dependent global loads) took 134 us at B=1 S=256 Hq=4 D=64 (one
// call among others), this one 8.3; B=15 S=549 Hq=32 D=64 1898 -> 306 us; B=2 S=1446 Hq=6 D=128 1706 -> 118 us.
#include <algorithm>

#include "common.h"

namespace seka {

namespace {

constexpr int kThreads = 256;
constexpr int kUnitRows = 16;

// maximum / sum over the four lanes (l % 16, 0..3) that share a query row
__device__ __forceinline__ float row_max(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float row_sum(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// x a1 + y a2 with the roundings fixed: the two ways of handing out units have to give the same bits.
__device__ __forceinline__ float fold(float x, float a1, float y, float a2) {
#pragma clang fp reassociate(off) contract(off)
  const float t = y * a2;
  return __builtin_fmaf(x, a1, t);
}
// log-sum-exp of a row from its reference exponent (base 2) and its sum, likewise
__device__ __forceinline__ float row_lse(float m, float l) {
#pragma clang fp reassociate(off) contract(off)
  const float log_l = logf(l);
  return __builtin_fmaf(m, 0.6931471805599453f, log_l);
}

__host__ __device__ inline int f32_rank_blocks(const SteerArgs& st) { return (st.M * st.r + 15) / 16; }

// LDS: U_cat as operands [rank block][D/16][64 lanes] of four floats, U^T q [wave][rank block][64 lanes] of four floats, the column
// coefficients; then a state per wave.  KSPLIT = 4: the states take the place of the rest after the key loop.
__host__ __device__ inline size_t attention_f32_steer_bytes(int D, int rank_blocks) {
  return (size_t)rank_blocks * (D / 16 + 4) * 1024 + (size_t)rank_blocks * 64;
}
inline size_t attention_f32_smem_bytes(int D, int rank_blocks, int ksplit) {
  const size_t steer = attention_f32_steer_bytes(D, rank_blocks), states = (size_t)4 * (D / 4 + 2) * 256;
  return ksplit == 1 ? steer + states : steer > states ? steer : states;
}

template <int D, bool STEER, int KSPLIT>
__global__ __launch_bounds__(kThreads, 2) void attention_f32_kernel(AttnArgs a, SteerArgs st) {
  static_assert(KSPLIT == 1 || KSPLIT == 4, "a unit is one wave's, or shared by the workgroup's four waves");
  constexpr int NB = D == 64 ? 2 : 1;            // 16-key blocks per step: 64 products either way
  constexpr int KI = D / 16;                     // 16-byte pieces of a K row per lane
  constexpr int VH = D / 64;                     // 16-byte pieces of a V row per lane
  extern __shared__ __attribute__((aligned(16))) float lds[];

  const float* __restrict__ Q = static_cast<const float*>(a.Q);
  const float* __restrict__ K = static_cast<const float*>(a.K);
  const float* __restrict__ V = static_cast<const float*>(a.V);
  float* __restrict__ O = static_cast<float*>(a.O);

  const int b = blockIdx.z, h = blockIdx.y, G = a.Hq / a.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  // units of one (prompt, KV head): row block slowest and longest first, so that neighbours read the same keys
  const int nrb = (a.S + kUnitRows - 1) / kUnitRows, units = nrb * G;
  const int unit = KSPLIT == 1 ? (int)blockIdx.x * 4 + wave : (int)blockIdx.x;
  const int rb = nrb - 1 - min(unit, units - 1) / G;
  const int hq = h * G + min(unit, units - 1) % G;
  size_t tok0;                                   // first token of this prompt in the tensors
  int Sb;                                        // this prompt's length
  prompt_extent(a, b, tok0, Sb);
  const int q0 = rb * kUnitRows;
  const bool live = unit < units && q0 < Sb;
  if (KSPLIT == 4 && !live) return;              // workgroup-uniform, before any barrier
  if (Sb == 0) return;                           // the same for the whole workgroup
  const int qi = q0 + l16;
  const int nkeys = live ? min(Sb, q0 + kUnitRows) : 0;
  const int nsteps = (nkeys + 16 * NB - 1) / (16 * NB);

  // operand registers of one step; a row past the end repeats the last one (finite, hidden by the causal mask)
  struct Step { f32x4 k[NB][KI]; f32x4 v[NB][4][VH]; int m[NB]; };
  const float gain = STEER ? st.gain[h] : 0.f;
  const bool steer_on = STEER && gain != 0.f;
  auto fetch = [&](int step, Step& s) __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int k0 = (step * NB + nb) * 16;
      const size_t row = tok0 + min(k0 + l16, Sb - 1);
      const float* kp = K + (row * a.Hkv + h) * D + 4 * g;
#pragma unroll
      for (int i = 0; i < KI; ++i) s.k[nb][i] = *reinterpret_cast<const f32x4*>(kp + 16 * i);
      if (STEER) s.m[nb] = steer_on && k0 + l16 < Sb ? st.mask[row] : 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float* vp = V + ((tok0 + min(k0 + 4 * g + i, Sb - 1)) * a.Hkv + h) * D + 4 * l16;
#pragma unroll
        for (int hh = 0; hh < VH; ++hh) s.v[nb][i][hh] = *reinterpret_cast<const f32x4*>(vp + 64 * hh);
      }
    }
  };
  const int step0 = KSPLIT == 1 ? 0 : wave;
  Step s0, s1;
  f32x4 q[KI];
  {
    const float* qp = Q + ((tok0 + min(qi, Sb - 1)) * a.Hq + hq) * D + 4 * g;
#pragma unroll
    for (int i = 0; i < KI; ++i) q[i] = *reinterpret_cast<const f32x4*>(qp + 16 * i);
  }
  if (step0 < nsteps) fetch(step0, s0);

  // ---- steering set-up: U_cat as operands, U^T q of this wave's rows ----
  const int NR = STEER ? f32_rank_blocks(st) : 0;
  f32x4* Uop = reinterpret_cast<f32x4*>(lds);
  f32x4* qt = Uop + NR * KI * 64 + wave * NR * 64;
  float* cvec = lds + (size_t)NR * (KI + 4) * 256;
  const float kscale = STEER ? st.kscale[h] : 1.f;
  if (STEER && steer_on) {
    const int R = st.M * st.r;
    const float* Uh = static_cast<const float*>(st.U) + (size_t)h * st.M * D * st.r;
    for (int idx = tid; idx < NR * KI * 64; idx += kThreads) {       // lane's d = 16 i + 4 g + e, column 16 blk + l % 16
      const int ln = idx & 63, i = (idx >> 6) % KI, blk = (idx >> 6) / KI;
      const int col = 16 * blk + (ln & 15), d0 = 16 * i + 4 * (ln >> 4);
      f32x4 u = {0.f, 0.f, 0.f, 0.f};
      if (col < R) {
        const int m = col / st.r, rr = col - m * st.r;
        const float* up = Uh + ((size_t)m * D + d0) * st.r + rr;
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = up[e * st.r];
      }
      Uop[idx] = u;
    }
    if (tid < 16 * NR) {
      float c = 0.f;
      if (tid < R) c = gain * (st.w ? st.w[((size_t)b * a.Hkv + h) * st.M + tid / st.r] : 1.f);
      cvec[tid] = c;
    }
    __syncthreads();
    for (int blk = 0; blk < NR; ++blk) {
      f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < KI; ++i) {
        const f32x4 u = Uop[(blk * KI + i) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) t = __builtin_amdgcn_mfma_f32_16x16x4f32(u[e], q[i][e], t, 0, 0, 0);
      }
      qt[blk * 64 + lane] = t;                   // read back by the lane that wrote it
    }
  }

  f32x4 o[D / 16];
#pragma unroll
  for (int x = 0; x < D / 16; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -1e30f, l_run = 0.f;             // l_run: this lane's keys only, until the end
  const float c2 = a.scale * 1.4426950408889634f;

  auto process = [&](int step, const Step& s) __attribute__((always_inline)) {
#pragma clang fp reassociate(off)
    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.k[nb][i][e], q[i][e], acc[nb], 0, 0, 0);
    if (STEER) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const unsigned bits = (unsigned)(__ballot(s.m[nb] != 0) & 0xffffull);
        if (__builtin_expect(bits != 0, 0)) {
          const f32x4 as_stored = acc[nb];
          if (kscale != 1.f) {
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[nb][i] *= (bits >> (4 * g + i)) & 1u ? kscale : 1.f;
          }
          for (int blk = 0; blk < NR; ++blk) {
            f32x4 z0 = {0.f, 0.f, 0.f, 0.f}, z1 = {0.f, 0.f, 0.f, 0.f};   // two chains
#pragma unroll
            for (int i = 0; i < KI; ++i) {
              const f32x4 u = Uop[(blk * KI + i) * 64 + lane];
#pragma unroll
              for (int e = 0; e < 4; e += 2) {
                z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(u[e], s.k[nb][i][e], z0, 0, 0, 0);
                z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(u[e + 1], s.k[nb][i][e + 1], z1, 0, 0, 0);
              }
            }
            // lane: key l % 16, columns 16 blk + 4 g + i: the A operand of the correction
            const f32x4 c4 = *reinterpret_cast<const f32x4*>(cvec + 16 * blk + 4 * g);
            const f32x4 t = qt[blk * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i)
              acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32((z0[i] + z1[i]) * c4[i], t[i], acc[nb], 0, 0, 0);
          }
          // the other keys of the block keep their scores, whatever the correction came to (weights that are not finite)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[nb][i] = (bits >> (4 * g + i)) & 1u ? acc[nb][i] : as_stored[i];
        }
      }
    }
    if ((step + 1) * (16 * NB) > q0) {           // wave-uniform: the diagonal block
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if ((step * NB + nb) * 16 + 4 * g + i > qi) acc[nb][i] = -INFINITY;
    }
    float mx = fmaxf(fmaxf(acc[0][0], acc[0][1]), fmaxf(acc[0][2], acc[0][3]));
    if (NB == 2) mx = fmaxf(mx, fmaxf(fmaxf(acc[NB - 1][0], acc[NB - 1][1]), fmaxf(acc[NB - 1][2], acc[NB - 1][3])));
    mx = row_max(mx) * c2;
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int x = 0; x < D / 16; ++x) o[x] *= alpha;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[nb][i], c2, -m_run));
        l_run += p;
#pragma unroll
        for (int hh = 0; hh < VH; ++hh)
#pragma unroll
          for (int db = 0; db < 4; ++db)
            o[4 * hh + db] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.v[nb][i][hh][db], p, o[4 * hh + db], 0, 0, 0);
      }
    }
  };
  // A state, this lane's part: D/16 x 4 values, m, l; value v of lane l at [v][l].
  constexpr int RS = D / 4 + 2;
  auto keep_state = [&](float* st) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < D / 16; ++x)
#pragma unroll
      for (int i = 0; i < 4; ++i) st[(4 * x + i) * 64] = o[x][i];
    st[(RS - 2) * 64] = m_run;
    st[(RS - 1) * 64] = l_run;
  };
  if (KSPLIT == 1) {
    // The steps of a row are four chains, w, w + 4, w + 8 ... for w = 0 .. 3, and the result is their states folded in
    // that order.  With KSPLIT = 4 each chain is a wave's; here the wave takes them one after the other.  So a row
    // has the same bits in either form, and they do not depend on the batch it is in.
    float* kept = lds + attention_f32_steer_bytes(D, NR) / 4 + (size_t)wave * RS * 64 + lane;
    auto after = [&](int step) __attribute__((always_inline)) {       // nsteps: none
      return step + 4 < nsteps ? step + 4 : (step & 3) < 3 ? min((step & 3) + 1, nsteps) : nsteps;
    };
    auto end_chain = [&](int step, bool last) __attribute__((always_inline)) {
      if (step + 4 < nsteps) return;
      l_run = row_sum(l_run);
      if ((step & 3) != 0) {
        const float m1 = kept[(RS - 2) * 64], l1 = kept[(RS - 1) * 64], mm = fmaxf(m1, m_run);
        const float a1 = __builtin_amdgcn_exp2f(m1 - mm), a2 = __builtin_amdgcn_exp2f(m_run - mm);
        m_run = mm;
        l_run = fold(l1, a1, l_run, a2);
#pragma unroll
        for (int x = 0; x < D / 16; ++x)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[x][i] = fold(kept[(4 * x + i) * 64], a1, o[x][i], a2);
      }
      if (last) return;
      keep_state(kept);                          // read back by the lane that wrote it
#pragma unroll
      for (int x = 0; x < D / 16; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
      m_run = -1e30f;
      l_run = 0.f;
    };
    for (int step = 0; step < nsteps;) {
      const int next = after(step);
      if (next < nsteps) fetch(next, s1);
      process(step, s0);
      end_chain(step, next >= nsteps);
      if (next >= nsteps) break;
      step = after(next);
      if (step < nsteps) fetch(step, s0);
      process(next, s1);
      end_chain(next, step >= nsteps);
    }
  } else {
    for (int step = step0; step < nsteps; step += 2 * KSPLIT) {
      if (step + KSPLIT < nsteps) fetch(step + KSPLIT, s1);
      process(step, s0);
      if (step + KSPLIT >= nsteps) break;
      if (step + 2 * KSPLIT < nsteps) fetch(step + 2 * KSPLIT, s0);
      process(step + KSPLIT, s1);
    }
    l_run = row_sum(l_run);
  }

  // ---- output: lane (row l % 16, g) holds d = 64 hh + 16 g + 4 i + db in o[4 hh + db][i] ----
  if (KSPLIT == 1) {
    if (!live || qi >= Sb) return;
    const float inv = 1.f / l_run;
    float* op = O + ((tok0 + qi) * a.Hq + hq) * D + 16 * g;
#pragma unroll
    for (int hh = 0; hh < VH; ++hh)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(op + 64 * hh + 4 * i) = f32x4{o[4 * hh][i], o[4 * hh + 1][i], o[4 * hh + 2][i], o[4 * hh + 3][i]} * inv;
    if (a.lse && g == 0) a.lse[lse_index(a, b, hq, tok0, qi)] = row_lse(m_run, l_run);
    return;
  }
  // fold the four waves' states; wave w finishes the values i = w
  __syncthreads();                               // the steering operands are dead
  keep_state(lds + (size_t)wave * RS * 64 + lane);
  __syncthreads();
  float m_all = lds[(size_t)(RS - 2) * 64 + lane], l_all = lds[(size_t)(RS - 1) * 64 + lane], r[D / 16];
#pragma unroll
  for (int x = 0; x < D / 16; ++x) r[x] = lds[(size_t)(4 * x + wave) * 64 + lane];
#pragma unroll
  for (int w = 1; w < 4; ++w) {                  // a wave without a step changes nothing: its a2 is zero and so is its state
    const float* other = lds + (size_t)w * RS * 64 + lane;
    const float m2 = other[(RS - 2) * 64], mm = fmaxf(m_all, m2);
    const float a1 = __builtin_amdgcn_exp2f(m_all - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
    m_all = mm;
    l_all = fold(l_all, a1, other[(RS - 1) * 64], a2);
#pragma unroll
    for (int x = 0; x < D / 16; ++x) r[x] = fold(r[x], a1, other[(4 * x + wave) * 64], a2);
  }
  if (qi >= Sb) return;
  const float inv = 1.f / l_all;
  float* op = O + ((tok0 + qi) * a.Hq + hq) * D + 16 * g + 4 * wave;
#pragma unroll
  for (int hh = 0; hh < VH; ++hh)
    *reinterpret_cast<f32x4*>(op + 64 * hh) = f32x4{r[4 * hh], r[4 * hh + 1], r[4 * hh + 2], r[4 * hh + 3]} * inv;
  if (a.lse && wave == 0 && g == 0) a.lse[lse_index(a, b, hq, tok0, qi)] = row_lse(m_all, l_all);
}

template <int D, bool STEER, int KSPLIT>
hipError_t launch_cfg(const AttnArgs& a, const SteerArgs& st, int units, hipStream_t s) {
  const size_t smem = attention_f32_smem_bytes(D, STEER ? f32_rank_blocks(st) : 0, KSPLIT);
  auto kernel = attention_f32_kernel<D, STEER, KSPLIT>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  const dim3 grid(KSPLIT == 1 ? (units + 3) / 4 : units, a.Hkv, a.B);
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), smem, s, a, st);
  return hipGetLastError();
}

template <int D, bool STEER>
hipError_t launch_d(const AttnArgs& a, const SteerArgs& st, hipStream_t s) {
  const int units = (a.S + kUnitRows - 1) / kUnitRows * (a.Hq / a.Hkv);      // per (prompt, KV head)
  // One wave per unit or four; the results are the same.  Whole units win where they fill the 1024 SIMDs once, just, or often
  // enough for their length that the last ones do not matter; a little over 1024 a second wave shares a few SIMDs and sets
  // the time.  The fewer steps a unit has, the more the split form's merge weighs: up to 4 steps at D = 64 and 7 at D = 128 whole
  // units win over 1024 as well.  `whole` counts the idle waves of a last workgroup.
  // Measured, us, whole / split, units x steps.  D = 64: 544 x 1 5.4 / 9.6, 480 x 3 10.7 / 8.1, 600 x 3 10.6 / 12.5, 588 x 4 13.6 / 13.8,
  // 1136 x 2 12.3 / 18.4, 1056 x 6 22 / 20, 1140 x 10 36 / 27, 2024 x 12 42 / 45, 2160 x 45 138 / 107, 4320 x 45 229 / 201.  D = 128: 576 x 3
  // 13.0 / 16.2, 800 x 10 25 / 28, 1140 x 5 25 / 28, 1728 x 6 28 / 38, 1056 x 12 38 / 32, 2016 x 12 40 / 55, 2016 x 36 104 / 93, 4032 x 56
  // 283 / 264, 4320 x 90 407 / 371, 5632 x 44 266 / 288, 7920 x 90 637 / 664.
  const int steps = (a.S + 2048 / D - 1) / (2048 / D);      // 32 keys at D = 64, 16 at D = 128
  const long long total = (long long)units * a.Hkv * a.B, whole = (long long)((units + 3) / 4 * 4) * a.Hkv * a.B;
  const int rise = D == 64 ? std::min(60 * std::min(steps - 4, 11) + 350 * std::max(steps - 15, 0), 6800)
                           : std::min(55 * std::min(steps - 7, 41) + 320 * std::max(steps - 48, 0), 5800);
  const long long least = whole <= 1024 ? (D == 64 ? 375 + 70 * steps : 400 + 35 * steps) : rise <= 0 ? 0 : rise + (D == 64 ? 1215 : 1180);
  return (whole <= 1024 ? total : whole) >= least ? launch_cfg<D, STEER, 1>(a, st, units, s) : launch_cfg<D, STEER, 4>(a, st, units, s);
}

}  // namespace

hipError_t launch_attention_f32(const AttnArgs& a, const SteerArgs* steer, hipStream_t s) {
  SteerArgs none;
  none.U = nullptr; none.w = nullptr; none.mask = nullptr; none.M = 0; none.r = 0;
  if (steer) return a.D == 128 ? launch_d<128, true>(a, *steer, s) : launch_d<64, true>(a, *steer, s);
  return a.D == 128 ? launch_d<128, false>(a, none, s) : launch_d<64, false>(a, none, s);
}

}  // namespace seka
