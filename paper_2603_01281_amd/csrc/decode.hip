// seka_attention_decode: the generation step that follows a steered prefill.  The edited keys persist in the
// KV cache (the hook of Algorithm 1 ran at prefill, seka_edit_keys in place), so one new query per (prompt,
// head) attends to the cached keys as they are: logits q . k'_j / sqrt(d_k) over the first len[b] tokens,
// softmax, weighted sum of V (paper Sec. 2).
//
// HBM-bound: every cached key and value is read once (2 * B * S * Hkv * D elements), a few flops per byte.
// Stage 1: grid (splits, KV head x head chunk, prompt); a workgroup streams its range of cached tokens with
// 16-byte loads (a row is 16 consecutive lanes for bf16 at D = 128, so one wave instruction fetches whole
// rows) and scores them against all the query heads of its KV head (the GQA group shares every byte read),
// keeping one online-softmax state per head with a lazily raised reference exponent: on the matrix cores for
// bf16 caches (decode_partial_mfma_kernel) and fp32 ones of larger groups (decode_partial_f32_kernel), on the vector
// unit for the other fp32 ones (decode_partial_kernel).  Partial
// states are merged across lanes, waves (LDS) and splits (stage 2, fixed order, so the result does not depend on
// scheduling).
#include <algorithm>
#include <mutex>

#include "common.h"

namespace seka {

namespace {

// Library-owned partial-state buffer of seka_attention_decode_static (callers that cannot allocate).  One copy per
// GPU that loads the library, held until the process ends; host code never uses this name as an address (it is
// a host-side stand-in there): decode_static_scratch() resolves the device address once per device.
static __device__ __align__(256) unsigned char scratch[kDecodeStaticScratchBytes];

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / 64;
constexpr float kDecSlack = 8.f;        // a head's reference exponent trails its maximum by at most this
constexpr float kNegBig = -1e30f;
// split policy (measured on MI355X: more, smaller splits lose to the merge stage; fewer leave CUs idle)
constexpr int kDecTargetWG = 4096, kDecMinRows = 512, kDecMinElemsF32 = 8192, kDecMaxSplits = 64;

// Query heads that one stage-1 workgroup serves: up to kDecMaxHeads of a KV head's group.
constexpr int kDecMaxHeads = 16;
inline int decode_heads_per_wg(int G) {
  if (G <= kDecMaxHeads) return G;
  for (int hp = kDecMaxHeads; hp > 1; --hp)
    if (G % hp == 0) return hp;
  return 1;
}

// Heads that count as one workgroup where fp32 ranges are cut: up to 8.
inline int decode_heads_f32(int G) {
  if (G <= 8) return G;
  for (int hp = 8; hp > 1; --hp)
    if (G % hp == 0) return hp;
  return 1;
}

// Splits of the cached range per (prompt, head group): about kDecTargetWG workgroups in all, at least min_rows tokens each.
inline int decode_splits(int groups, int S, int min_rows) {
  int want = (kDecTargetWG + groups - 1) / groups;
  const int cap = S / min_rows > 1 ? S / min_rows : 1;
  if (want > cap) want = cap;
  if (want > kDecMaxSplits) want = kDecMaxSplits;
  return want < 1 ? 1 : want;
}

// A 16-byte load of the cache.  NT: without keeping a place for it in the caches (decode_streams).
template <bool NT, typename V>
__device__ __forceinline__ V dec_load(const V* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

template <typename T> struct DecElem;
template <> struct DecElem<uint16_t> {
  __device__ static void store(uint16_t* p, float v) {
    const __bf16 b = (__bf16)v;
    *p = __builtin_bit_cast(uint16_t, b);
  }
};
__device__ __forceinline__ float dec_dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}

template <> struct DecElem<float> {
  static constexpr int EPL = 4;
  template <bool NT = false>
  __device__ static void load(const float* p, float (&out)[4]) {
    const f32x4 v = dec_load<NT>(reinterpret_cast<const f32x4*>(p));
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = v[i];
  }
  __device__ static void store(float* p, float v) { *p = v; }
};

// Maximum and sum over the lanes with the same index in a half (HALVES = 2) or a row of 16 (4); the same bits in all of them.
// Lane swaps on the vector unit: a shuffle through LDS is some 120 cycles in a chain that every step of a range waits for
// (us, shuffles / swaps, kernels of a graph on one cache: bf16 32 / 8 heads B=1 S=1000 D = 128 6.8 / 6.7, D = 64 7.0 / 6.8; fp32 D = 64
// S=600 7.4 / 7.2).
template <int PARTS, typename F>
__device__ __forceinline__ float across(float v, F join) {
  if (PARTS == 4) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = join(__uint_as_float(a[0]), __uint_as_float(a[1]));
  }
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return join(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <int PARTS>
__device__ __forceinline__ float across_max(float v) {
  return across<PARTS>(v, [](float x, float y) __attribute__((always_inline)) { return fmaxf(x, y); });
}
template <int PARTS>
__device__ __forceinline__ float across_sum(float v) {
  return across<PARTS>(v, [](float x, float y) __attribute__((always_inline)) { return x + y; });
}

// Sum over the LPR consecutive lanes that hold one row; every one of them receives the total.
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));    // lane ^ 1
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xf, 0xf, true));    // lane ^ 2
  if (LPR >= 8)
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xf, 0xf, true)); // mirror in 8
  if (LPR >= 16)
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xf, 0xf, true)); // mirror in 16
  if (LPR >= 32) v += __shfl_xor(v, 16);
  return v;
}

// Merge online-softmax state (m2, l2, o2) into (m, l, o); exponents are base 2.
template <int N>
__device__ __forceinline__ void merge_state(float& m, float& l, float (&o)[N], float m2, float l2, const float (&o2)[N]) {
  const float mm = fmaxf(m, m2);
  const float a1 = __builtin_amdgcn_exp2f(m - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
  m = mm;
  l = l * a1 + l2 * a2;
#pragma unroll
  for (int i = 0; i < N; ++i) o[i] = o[i] * a1 + o2[i] * a2;
}

// The range of the cache that a stage-1 workgroup takes.  Workgroups go to the eight XCDs in index order, so with a
// multiple of four ranges an XCD has the same ranges of every prompt and head, and the first ranges, the only ones that
// short caches have, pile up on a few (16 caches of 536 to 8192 tokens, 8 KV heads: 23 ranges per head on one XCD, 8 on
// another; 68 -> 53 us with nothing cached).  Ragged batches therefore turn the order with the head and the prompt; equal
// lengths keep it (an XCD then reads all heads of the same tokens).
__device__ __forceinline__ int decode_split_index(const int* lens, int splits) {
  const unsigned turn = lens && splits % 4 == 0 ? blockIdx.y + blockIdx.z : 0u;
  return (int)((blockIdx.x + turn) % (unsigned)splits);
}

// What a stage-1 workgroup does with the merged state (mm, ll, oo) of output element d of query head hq: with
// several splits it goes to the partial-state buffer for stage 2; with a single split it IS the result, and the
// workgroup writes the output and the log-sum-exp itself (the same arithmetic as stage 2 on one split, which is
// then not launched: short caches take one kernel instead of two).
template <typename T, int D>
__device__ __forceinline__ void decode_emit(float mm, float ll, float oo, int b, int hq, int d, int Hq, int splits,
                                            int split, float* __restrict__ part, T* __restrict__ O,
                                            float* __restrict__ lse) {
  if (splits == 1) {
    DecElem<T>::store(O + ((size_t)b * Hq + hq) * D + d, ll > 0.f ? oo / ll : 0.f);
    if (lse && d == 0) lse[(size_t)b * Hq + hq] = ll > 0.f ? mm * 0.6931471805599453f + logf(ll) : -INFINITY;
    return;
  }
  float* dst = part + (((size_t)b * Hq + hq) * splits + split) * (D + 2);
  dst[d] = oo;
  if (d == 0) {
    dst[D] = mm;
    dst[D + 1] = ll;
  }
}

// Partial state of one (prompt, query head, split): D unnormalised outputs, then m (base-2 exponent), then l.
// Stage 1 for fp32 caches and groups of few heads: every product on the vector unit.
template <int D, int GP, bool NT>
__global__ __launch_bounds__(kDecThreads) void decode_partial_kernel(const float* __restrict__ q, const float* __restrict__ K,
                                                                     const float* __restrict__ V, const int* __restrict__ lens,
                                                                     int S, int Hq, int Hkv, float c2, int splits,
                                                                     float* __restrict__ part, float* __restrict__ O,
                                                                     float* __restrict__ lse) {
  constexpr int EPL = DecElem<float>::EPL;
  constexpr int LPR = D / EPL;            // lanes per cached row
  constexpr int KPW = 64 / LPR;           // rows per wave load
  constexpr int UNR = 4;                  // row groups in flight per lane
  __shared__ float sm_o[kDecWaves][GP][D];
  __shared__ float sm_ml[kDecWaves][GP][2];

  const int G = Hq / Hkv;
  const int chunks = G / GP;
  const int b = blockIdx.z, h = blockIdx.y / chunks, hq0 = h * G + (blockIdx.y % chunks) * GP;
  const int split = decode_split_index(lens, splits);
  const int n = lens ? min(max(lens[b], 0), S) : S;
  const int per = (S + splits - 1) / splits;
  const int k0 = split * per, k1 = min(n, k0 + per);
  if (k0 >= k1 && splits > 1) return;      // workgroup-uniform; stage 2 knows which ranges are empty

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane % LPR, kk = lane / LPR;

  float qv[GP][EPL];
#pragma unroll
  for (int g = 0; g < GP; ++g) DecElem<float>::load(q + ((size_t)b * Hq + hq0 + g) * D + c * EPL, qv[g]);

  float m[GP], l[GP], o[GP][EPL];
#pragma unroll
  for (int g = 0; g < GP; ++g) {
    m[g] = kNegBig;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[g][e] = 0.f;
  }

  const size_t rowstride = (size_t)Hkv * D;
  const float* Kb = K + ((size_t)b * S * Hkv + h) * D + c * EPL;
  const float* Vb = V + ((size_t)b * S * Hkv + h) * D + c * EPL;
  const int step = kDecWaves * KPW;                      // rows per workgroup turn
  for (int turn = k0; turn < k1; turn += UNR * step) {      // workgroup-uniform trip count
    const int base = turn + wave * KPW + kk;
    bool ok[UNR];
    {
      float kf[UNR][EPL], vf[UNR][EPL];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int row = base + u * step;
        ok[u] = row < k1;
        const size_t r = (size_t)(ok[u] ? row : k1 - 1) * rowstride;
        DecElem<float>::load<NT>(Kb + r, kf[u]);
        DecElem<float>::load<NT>(Vb + r, vf[u]);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
#pragma unroll
        for (int g = 0; g < GP; ++g) {
          float s = 0.f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) s = fmaf(qv[g][e], kf[u][e], s);
          s = row_sum<LPR>(s) * c2;
          if (!ok[u]) s = -INFINITY;
          if (s > m[g] + kDecSlack) {                      // raise the reference exponent (rare after the first rows)
            const float alpha = __builtin_amdgcn_exp2f(m[g] - s);
            m[g] = s;
            l[g] *= alpha;
#pragma unroll
            for (int e = 0; e < EPL; ++e) o[g][e] *= alpha;
          }
          const float p = __builtin_amdgcn_exp2f(s - m[g]);
          l[g] += p;
#pragma unroll
          for (int e = 0; e < EPL; ++e) o[g][e] = fmaf(p, vf[u][e], o[g][e]);
        }
      }
    }
  }

  // ---- merge the row groups of a wave (lanes c, c + LPR, ...), then the waves ----
#pragma unroll
  for (int g = 0; g < GP; ++g) {
#pragma unroll
    for (int d = LPR; d < 64; d *= 2) {
      float o2[EPL];
      const float m2 = __shfl_xor(m[g], d), l2 = __shfl_xor(l[g], d);
#pragma unroll
      for (int e = 0; e < EPL; ++e) o2[e] = __shfl_xor(o[g][e], d);
      merge_state(m[g], l[g], o[g], m2, l2, o2);
    }
    if (kk == 0) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) sm_o[wave][g][c * EPL + e] = o[g][e];
      if (c == 0) {
        sm_ml[wave][g][0] = m[g];
        sm_ml[wave][g][1] = l[g];
      }
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < GP * D; idx += kDecThreads) {
    const int g = idx / D, d = idx % D;
    float mm = sm_ml[0][g][0];
#pragma unroll
    for (int w = 1; w < kDecWaves; ++w) mm = fmaxf(mm, sm_ml[w][g][0]);
    float ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      const float aw = __builtin_amdgcn_exp2f(sm_ml[w][g][0] - mm);
      ll += sm_ml[w][g][1] * aw;
      oo += sm_o[w][g][d] * aw;
    }
    decode_emit<float, D>(mm, ll, oo, b, hq0 + g, d, Hq, splits, split, part, O, lse);
  }
}

// Stage 1 for fp32 caches where decode_on_matrix_cores says so, on v_mfma_f32_16x16x4_f32 (fp32 products and
// accumulation).  The query heads of a group (HP <= 16 of them, padded to the instruction's 16 columns) take the place that
// 16 query rows have in the fp32 prefill kernel:
//   S^T (16 keys x heads)  = K q^T        lane (head l % 16, g = l / 16) gets keys 4 g + i,
//   O^T (D x heads)       += V^T P^T      for which it has the operand, and ends with d = 64 hh + 16 g + 4 i + db.
// K and V go from global memory straight into operand registers with 16-byte loads, those of a wave's next 16 keys as soon
// as its products with these are issued.  On the vector unit every head is a multiplication and an addition per element and
// lane, and a token cost a workgroup 8.6 ns per head; the matrix cores take a whole group for what two or three heads cost
// there.  us before / after (nothing cached): 28 / 4 heads, D = 128, B=1 S=100 15.3 / 6.6, S=9078 25.4 / 14.8, B=12 S=3000
// 51.2 / 37.7 (3.9 TB/s); D = 64, B=1 S=777 13.5 / 8.6; 16 / 1 heads, D = 128, B=40 S=1137 43.6 / 18.4.
// A score is shared by NCH accumulators and an output by two, so that the error against 64 bits is not above that of the vector
// unit's sums (1.9e-7 against 2.0e-7 relative at S = 1137; one chain of 128 products per score 4.2e-7).  The registers for that
// leave 2 waves per SIMD at D = 128 and 4 at D = 64 (where holding the compiler to 4 made it spill: B=40 S=1137 32 / 8 heads
// 46.8 us instead of 44.3).
template <int D, bool NT>
__global__ __launch_bounds__(kDecThreads, D == 64 ? 3 : 2) void decode_partial_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ K, const float* __restrict__ V, const int* __restrict__ lens, int S,
    int Hq, int Hkv, int HP, float c2, int splits, float* __restrict__ part, float* __restrict__ O, float* __restrict__ lse) {
  constexpr int NCH = 8;
  constexpr int KI = D / 16, VH = D / 64;        // 16-byte pieces of a K row, of a V row per lane
  constexpr int BK = 16, OLD = D + 4;            // keys per step; row stride of the merge area
  __shared__ __attribute__((aligned(16))) float sm_o[kDecWaves][kDecMaxHeads][OLD];
  __shared__ float sm_ml[kDecWaves][kDecMaxHeads][2];

  const int G = Hq / Hkv, chunks = G / HP;
  const int b = blockIdx.z, h = blockIdx.y / chunks, hq0 = h * G + (blockIdx.y % chunks) * HP;
  const int split = decode_split_index(lens, splits);
  const int n = lens ? min(max(lens[b], 0), S) : S;
  const int per = (S + splits - 1) / splits;
  const int k0 = split * per, k1 = min(n, k0 + per);
  if (k0 >= k1 && splits > 1) return;            // workgroup-uniform; stage 2 knows which ranges are empty

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
  f32x4 qv[KI];
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    qv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (l16 < HP) qv[i] = *reinterpret_cast<const f32x4*>(q + ((size_t)b * Hq + hq0 + l16) * D + 16 * i + 4 * g);
  }
  const size_t rowstride = (size_t)Hkv * D;
  const float* Kb = K + ((size_t)b * S * Hkv + h) * D + 4 * g;
  const float* Vb = V + ((size_t)b * S * Hkv + h) * D + 4 * l16;
  f32x4 kv[KI], vv[4][VH];
  // rows clamped into the range: loads stay inside the cache
  auto fetch_k = [&](int kb) __attribute__((always_inline)) {
    const float* kp = Kb + (size_t)min(kb + l16, k1 - 1) * rowstride;
#pragma unroll
    for (int i = 0; i < KI; ++i) kv[i] = *reinterpret_cast<const f32x4*>(kp + 16 * i);
  };
  auto fetch_v = [&](int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* vp = Vb + (size_t)min(kb + 4 * g + i, k1 - 1) * rowstride;
#pragma unroll
      for (int hh = 0; hh < VH; ++hh) vv[i][hh] = dec_load<NT>(reinterpret_cast<const f32x4*>(vp + 64 * hh));
    }
  };

  f32x4 o[2][D / 16];                            // keys 4 g + i of even and of odd i
#pragma unroll
  for (int x = 0; x < D / 16; ++x) o[0][x] = o[1][x] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = kNegBig, l = 0.f;                    // l: this lane's keys only, until the end
  constexpr int TURN = kDecWaves * BK;
  int kb = k0 + wave * BK;
  if (kb < k1) {
    fetch_k(kb);
    fetch_v(kb);
  }
  for (; kb < k1; kb += TURN) {
    const bool more = kb + TURN < k1;
    f32x4 acc[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[(4 * i + e) % NCH] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[i][e], qv[i][e], acc[(4 * i + e) % NCH], 0, 0, 0);
    if (more) fetch_k(kb + TURN);
#pragma unroll
    for (int half = NCH / 2; half; half /= 2)
#pragma unroll
      for (int c = 0; c < half; ++c) acc[c] += acc[c + half];
    f32x4 t = acc[0] * c2;
    float bmax = kNegBig;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (kb + 4 * g + i >= k1) t[i] = -INFINITY;
      bmax = fmaxf(bmax, t[i]);
    }
    bmax = across_max<4>(bmax);
    const bool raise = bmax > m + kDecSlack;     // the same in a head's four lanes
    if (__any(raise)) {                          // rare after the first steps
      const float alpha = raise ? __builtin_amdgcn_exp2f(m - bmax) : 1.f;
      if (raise) m = bmax;
      l *= alpha;
#pragma unroll
      for (int x = 0; x < D / 16; ++x) {
        o[0][x] *= alpha;
        o[1][x] *= alpha;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = __builtin_amdgcn_exp2f(t[i] - m);
      l += p;
#pragma unroll
      for (int x = 0; x < D / 16; ++x)
        o[i & 1][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[i][x / 4][x % 4], p, o[i & 1][x], 0, 0, 0);
    }
    if (more) fetch_v(kb + TURN);
  }

  // ---- merge the waves ----
  l = across_sum<4>(l);
#pragma unroll
  for (int x = 0; x < D / 16; ++x) o[0][x] += o[1][x];
  if (l16 < HP) {
#pragma unroll
    for (int hh = 0; hh < VH; ++hh)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(&sm_o[wave][l16][64 * hh + 16 * g + 4 * i]) = 
            f32x4{o[0][4 * hh][i], o[0][4 * hh + 1][i], o[0][4 * hh + 2][i], o[0][4 * hh + 3][i]};
    if (g == 0) {
      sm_ml[wave][l16][0] = m;
      sm_ml[wave][l16][1] = l;
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < HP * D; idx += kDecThreads) {
    const int hd = idx / D, d = idx % D;
    float mm = sm_ml[0][hd][0];
#pragma unroll
    for (int w = 1; w < kDecWaves; ++w) mm = fmaxf(mm, sm_ml[w][hd][0]);
    float ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      const float aw = __builtin_amdgcn_exp2f(sm_ml[w][hd][0] - mm);
      ll += sm_ml[w][hd][1] * aw;
      oo += sm_o[w][hd][d] * aw;
    }
    decode_emit<float, D>(mm, ll, oo, b, hq0 + hd, d, Hq, splits, split, part, O, lse);
  }
}

// Stage 1 for bf16 caches on the matrix cores.  Same grid, split ranges and partial-state layout as the kernel
// above; what changes is who does the arithmetic.  The query heads of the group (HP <= 16 of them, padded to the 32
// columns of the instruction) take the place that a tile of queries has in the prefill kernel:
//   S^T (32 keys x heads)   = K (32 keys x D) q^T        D/16 x v_mfma_f32_32x32x16_bf16
//   O^T (D x heads)        += V^T (D x 32 keys) P^T      2 D/32 of them
// Keys and values are loaded as whole rows (every cache line requested once; fragments fetched straight from
// global memory, 32 bytes per lane pair, cost twice the time) and pass through a wave-private LDS tile with padded
// rows (no bank conflicts): K comes back with 16-byte reads, then V takes the tile over and comes back through transposing reads,
// so that the vector unit is left with the softmax alone (one fma, one exponential and half a conversion per key
// and lane) instead of every product, and a wave's next 32 keys and values (16 KB) are in flight while it works
// on the current ones.  Waves take the 32-key blocks of the workgroup's range in turn and never synchronise
// before the final merge.  Probabilities are rounded to bf16 once; that value feeds the row sum and the product.
typedef __attribute__((address_space(3))) s16x4* dec_lds_s16x4_ptr;
template <int D, int NW, bool NT>
__global__ __launch_bounds__(64 * NW, 2) void decode_partial_mfma_kernel(const uint16_t* __restrict__ q,
                                                                          const uint16_t* __restrict__ K,
                                                                          const uint16_t* __restrict__ V,
                                                                          const int* __restrict__ lens, int S, int Hq,
                                                                          int Hkv, int HP, float c2, int splits,
                                                                          float* __restrict__ part, uint16_t* __restrict__ O,
                                                                          float* __restrict__ lse) {
  constexpr int BK = 32;                   // keys per block
  // LDS row strides (elements).  K rows are read back 16 bytes per lane by 16 consecutive rows: a stride of 16 bytes
  // mod 256 spreads them over all banks.  V rows come back through transposing reads, where 16 lanes take 32 bytes
  // of each of four consecutive rows: a stride of 64 bytes mod 256 keeps those apart.
  constexpr int LDK = D + 8, LD = D + 32;
  constexpr int OLD = D + 4;               // row stride of the merge area (floats)
  constexpr int KS = D / 16, NB = D / 32;
  constexpr int CPR = D / 8, RPI = 64 / CPR, NV = BK / RPI;   // V rows: 16-byte chunks per row, rows per load, loads
  constexpr int kTileBytes = BK * LD * 2;
  constexpr int kMergeBytes = kDecMaxHeads * OLD * 4;
  __shared__ __attribute__((aligned(16))) unsigned char smem[NW * (kTileBytes > kMergeBytes ? kTileBytes : kMergeBytes)];
  __shared__ float sm_ml[NW][kDecMaxHeads][2];

  const int G = Hq / Hkv;
  const int chunks = G / HP;
  const int b = blockIdx.z, h = blockIdx.y / chunks, hq0 = h * G + (blockIdx.y % chunks) * HP;
  const int split = decode_split_index(lens, splits);
  const int n = lens ? min(max(lens[b], 0), S) : S;
  const int per = (S + splits - 1) / splits;
  const int k0 = split * per, k1 = min(n, k0 + per);
  if (k0 >= k1 && splits > 1) return;      // workgroup-uniform; stage 2 knows which ranges are empty

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, hf = lane >> 5, li = lane & 15, grp = lane >> 4;
  uint16_t* vt = reinterpret_cast<uint16_t*>(smem + (size_t)wave * kTileBytes);

  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;   // (a plain vector type: arrays of it stay in registers)
  // B operand of the score product: lane (head l32, hf) holds q[head][16 s + 8 hf ..][0..7]; padding heads are zero
  bf16x8 qf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    u32x4 t = {0, 0, 0, 0};
    if (l32 < HP) t = *reinterpret_cast<const u32x4*>(q + ((size_t)b * Hq + hq0 + l32) * D + 16 * s + 8 * hf);
    qf[s] = __builtin_bit_cast(bf16x8, t);
  }

  const size_t rowstride = (size_t)Hkv * D;
  const uint16_t* Kb = K + ((size_t)b * S * Hkv + h) * D;
  const uint16_t* Vb = V + ((size_t)b * S * Hkv + h) * D;
  // both tiles arrive as whole rows (a row is CPR consecutive lanes: every cache line is requested once)
  u32x4 kr[NV], vr[NV];
  auto fetch = [&](int kb) __attribute__((always_inline)) {       // rows clamped into the range: loads stay inside the cache
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const size_t rv = (size_t)min(kb + RPI * i + lane / CPR, k1 - 1) * rowstride + 8 * (lane % CPR);
      kr[i] = dec_load<NT>(reinterpret_cast<const u32x4*>(Kb + rv));
      vr[i] = dec_load<NT>(reinterpret_cast<const u32x4*>(Vb + rv));
    }
  };
  // transposing read of a V^T fragment (32 values of d x 16 keys): lanes address key 4 hf + li / 4 (+ 8) of the
  // 16-key slab, columns 16 (grp & 1) + 4 (li & 3) of the 32-column block; lane (d l32, hf) receives the keys in
  // the order in which the score accumulator holds them (element e: key 8 (e / 4) + 4 hf + e % 4)
  const int frag_off = (4 * hf + (li >> 2)) * LD + 16 * (grp & 1) + 4 * (li & 3);
  auto vfrag = [&](int slab, int blk) __attribute__((always_inline)) -> bf16x8 {
    const uint16_t* p = vt + frag_off + (16 * slab) * LD + 32 * blk;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dec_lds_s16x4_ptr)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dec_lds_s16x4_ptr)(p + 8 * LD));
    return __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi), 0, 1, 2, 3, 4, 5, 6, 7);
  };

  // state of head l32 (both halves hf keep the same m; l is this lane's share of the row sum)
  float m = kNegBig, l = 0.f;
  f32x16 oacc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;

  int kb = k0 + wave * BK;
  if (kb < k1) fetch(kb);
  for (; kb < k1; kb += NW * BK) {
    // K rows to the wave's tile, back as A fragments (lane (key l32, hf): 16 bytes at d = 16 s + 8 hf); then the V
    // rows take the tile over.  A wave's LDS operations execute in program order; the fences are for the compiler.
#pragma unroll
    for (int i = 0; i < NV; ++i)
      *reinterpret_cast<u32x4*>(vt + (RPI * i + lane / CPR) * LDK + 8 * (lane % CPR)) = kr[i];
    asm volatile("" ::: "memory");
    f32x16 sacc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[r] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bf16x8 kf = *reinterpret_cast<const bf16x8*>(vt + l32 * LDK + 16 * s + 8 * hf);
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], sacc, 0, 0, 0);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < NV; ++i)
      *reinterpret_cast<u32x4*>(vt + (RPI * i + lane / CPR) * LD + 8 * (lane % CPR)) = vr[i];
    asm volatile("" ::: "memory");
    const int kb_next = kb + NW * BK;
    const bool full = kb + BK <= k1;
    if (kb_next < k1) fetch(kb_next);      // the registers are free again: next block's loads fly during the softmax

    float t[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r] = sacc[r] * c2;
    if (!full) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (kb + 16 * (r >> 3) + 8 * ((r >> 2) & 1) + 4 * hf + (r & 3) >= k1) t[r] = -INFINITY;
    }
    float bmax = t[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) bmax = fmaxf(bmax, t[r]);
    bmax = across_max<2>(bmax);
    const bool raise = bmax > m + kDecSlack;
    if (__any(raise)) {                    // rare after the first blocks
      const float alpha = raise ? __builtin_amdgcn_exp2f(m - bmax) : 1.f;
      if (raise) m = bmax;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
    }
    bf16x8 pb[2];
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const bf16x2 p2 = {(__bf16)__builtin_amdgcn_exp2f(t[8 * sl + e] - m), (__bf16)__builtin_amdgcn_exp2f(t[8 * sl + e + 1] - m)};
        pb[sl][e] = p2[0];
        pb[sl][e + 1] = p2[1];
        l = dec_dot2(__builtin_bit_cast(uint32_t, p2), 0x3f803f80u, l);
      }
    }
#pragma unroll
    for (int sl = 0; sl < 2; ++sl)
#pragma unroll
      for (int i = 0; i < NB; ++i) oacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfrag(sl, i), pb[sl], oacc[i], 0, 0, 0);
    asm volatile("" ::: "memory");         // the tile is rewritten only after these reads
  }

  // ---- merge the waves: lane (head l32, hf) holds O[head][32 i + 8 (r / 4) + 4 hf + r % 4] ----
  l = across_sum<2>(l);
  __syncthreads();                         // every wave is done with its V tile: the area becomes the merge area
  float* sm_o = reinterpret_cast<float*>(smem) + (size_t)wave * kDecMaxHeads * OLD;
  if (l32 < HP) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        *reinterpret_cast<f32x4*>(sm_o + l32 * OLD + 32 * i + 8 * r4 + 4 * hf) =
            f32x4{oacc[i][4 * r4], oacc[i][4 * r4 + 1], oacc[i][4 * r4 + 2], oacc[i][4 * r4 + 3]};
    if (hf == 0) {
      sm_ml[wave][l32][0] = m;
      sm_ml[wave][l32][1] = l;
    }
  }
  __syncthreads();
  const float* sm_all = reinterpret_cast<const float*>(smem);
  for (int idx = threadIdx.x; idx < HP * D; idx += 64 * NW) {
    const int g = idx / D, d = idx % D;
    float mm = sm_ml[0][g][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) mm = fmaxf(mm, sm_ml[w][g][0]);
    float ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float aw = __builtin_amdgcn_exp2f(sm_ml[w][g][0] - mm);
      ll += sm_ml[w][g][1] * aw;
      oo += sm_all[((size_t)w * kDecMaxHeads + g) * OLD + d] * aw;
    }
    decode_emit<uint16_t, D>(mm, ll, oo, b, hq0 + g, d, Hq, splits, split, part, O, lse);
  }
}

// grid (Hq, B), block kFinThreads: thread (j, d) merges splits j, j + NJ, ... in that order, then the NJ partial
// states are merged in index order: a fixed order, whatever the launch.  The kernel is pure latency (a few tens of
// kilobytes per workgroup), so every load of a thread is issued before the first is used; NI, the states a thread
// takes, is what the number of splits needs.
constexpr int kFinThreads = 1024;
template <typename T, int D, int NI>
__global__ __launch_bounds__(kFinThreads) void decode_finish_kernel(const float* __restrict__ part, const int* __restrict__ lens,
                                                                    int S, int Hq, int splits, T* __restrict__ O,
                                                                    float* __restrict__ lse) {
  constexpr int NJ = kFinThreads / D;
  __shared__ float sm[NJ][D + 2];
  const int hq = blockIdx.x, b = blockIdx.y, d = threadIdx.x % D, j = threadIdx.x / D;
  const float* src = part + ((size_t)b * Hq + hq) * splits * (D + 2);
  const int per = (S + splits - 1) / splits;             // tokens per range, as in stage 1; a shorter cache has fewer
  const int live = lens ? (min(max(lens[b], 0), S) + per - 1) / per : splits;
  float mv[NI], lv[NI], ov[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int s = j + NJ * i;
    const float* ps = src + (size_t)(s < splits ? s : 0) * (D + 2);     // clamped: the value is dropped below
    mv[i] = ps[D];
    lv[i] = ps[D + 1];
    ov[i] = ps[d];
  }
  float mm = kNegBig;
#pragma unroll
  for (int i = 0; i < NI; ++i)
    if (j + NJ * i < live) mm = fmaxf(mm, mv[i]);
  float ll = 0.f, oo = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i)
    if (j + NJ * i < live) {
      const float aw = __builtin_amdgcn_exp2f(mv[i] - mm);
      ll += lv[i] * aw;
      oo += ov[i] * aw;
    }
  sm[j][d] = oo;
  if (d == 0) {
    sm[j][D] = mm;
    sm[j][D + 1] = ll;
  }
  __syncthreads();
  if (j == 0) {
    float m2 = sm[0][D];
#pragma unroll
    for (int k = 1; k < NJ; ++k) m2 = fmaxf(m2, sm[k][D]);
    float l2 = 0.f, o2 = 0.f;
#pragma unroll
    for (int k = 0; k < NJ; ++k) {
      const float aw = __builtin_amdgcn_exp2f(sm[k][D] - m2);
      l2 += sm[k][D + 1] * aw;
      o2 += sm[k][d] * aw;
    }
    DecElem<T>::store(O + ((size_t)b * Hq + hq) * D + d, l2 > 0.f ? o2 / l2 : 0.f);
    if (lse && d == 0) lse[(size_t)b * Hq + hq] = l2 > 0.f ? m2 * 0.6931471805599453f + logf(l2) : -INFINITY;
  }
}

template <typename T, int D>
void launch_decode_finish(const float* part, const int* lens, int B, int S, int Hq, int splits, T* O, float* lse, hipStream_t s) {
  constexpr int NJ = kFinThreads / D;
  const dim3 grid(Hq, B), block(kFinThreads);
  if (splits <= NJ) hipLaunchKernelGGL((decode_finish_kernel<T, D, 1>), grid, block, 0, s, part, lens, S, Hq, splits, O, lse);
  else if (splits <= 2 * NJ) hipLaunchKernelGGL((decode_finish_kernel<T, D, 2>), grid, block, 0, s, part, lens, S, Hq, splits, O, lse);
  else hipLaunchKernelGGL((decode_finish_kernel<T, D, (kDecMaxSplits + NJ - 1) / NJ>), grid, block, 0, s, part, lens, S, Hq, splits, O, lse);
}

// Whether an fp32 call goes to the matrix cores.  Groups of five heads and more do; one or two heads are too few for an
// instruction of 16 (32 / 16 heads, D = 128, B=1 S=9078: vector unit 33.9 us, matrix cores 37.0; D = 64, B=6 S=1137 16.2 /
// 17.1); three and four do while the call is a chain of loads and products and not yet memory's: up to 64 MB of cache at
// D = 128, 128 MB at D = 64 (24 / 8 heads, D = 128: B=6 S=1137, 56 MB, 20.2 / 16.6, B=16 S=560, 73 MB, 20.4 / 22.8; 32 / 8
// heads: B=6 S=1137 22.4 / 16.6, B=100 S=400 69.5 / 72.8; D = 64, B=16 S=560, 37 MB, 14.4 / 12.8, B=100 S=400, 164 MB,
// 43.1 / 44.4).
// `ranges` of `turns` times 64 tokens for each of B Hkv chunks groups: above one workgroup per compute unit three heads, and four
// in ranges of a single turn, are not always enough either.  Three lose where the last workgroups share only a few compute
// units, where a range is a single turn, and at D = 64 with two to a unit.  us, vector unit / matrix cores, 3 heads: D = 128,
// S=128 264 groups 11.5 / 13.9, S=300 96 groups 10.8 / 12.3, 160 groups 15.4 / 14.0, 184 groups 16.5 / 18.7, S=600 72 groups
// 15.1 / 13.5; D = 64, S=100 640 groups 7.3 / 8.1, S=300 144 groups 9.5 / 10.2, 300 groups 15.8 / 15.1, S=900 84 groups
// 13.2 / 11.1; 4 heads, D = 128, S=384 84 groups 11.1 / 10.3, 112 groups 14.4 / 15.8.
bool decode_on_matrix_cores(int B, int S, int Hkv, int chunks, int D, int hp, int ranges, int turns) {
  if (hp <= 2 || hp > 4) return hp > 4;
  if (2.0 * sizeof(float) * B * S * Hkv * D * D > 64e6 * 128) return false;
  const int wg = B * Hkv * chunks * ranges;
  if (wg <= 256) return true;
  if (hp == 4) return D == 64 || turns > 1 || wg <= 512;
  if (D == 64) return S >= 128 && wg > 448 - std::max(S - 600, 0) / 10;
  return turns > 1 && (S < 120 || S >= 192) && (wg - 1) % 256 >= (S < 350 ? 80 : 60);
}

// Whether a call reads past the caches: each byte once, and so many of them that the next call over the same cache would find
// little of them in the 256 MB of the memory-side cache either.  The line is at 300 MB, with the call repeated on one cache: up
// to 290 MB plain loads are the better by up to 10 %, from 310 MB on nontemporal ones, by 1 to 14 %.  us, plain / nontemporal,
// D = 128: bf16 32 / 8 heads B=16, 290 MB, 49.8 / 50.7, 310 MB 55.2 / 54.0; 32 / 32 heads B=6 S=9078, 892 MB, 154.4 / 137.6
// (6.5 TB/s); fp32 28 / 4 heads B=4 S=32000, 524 MB, 104.5 / 81.9; 32 / 16 heads B=40 S=1137, 745 MB, 136.6 / 123.0.
// The lengths of a ragged batch are on the device: a quarter of the allocation is taken for them (lengths spread over 1 : 16
// by ratio fill a third).  One kind of loads stays plain whatever this says: K in decode_partial_f32_kernel, whose lines are asked
// for by two loads each (us, plain / nontemporal K: 40 / 8 heads B=15 S=4050 D = 128 84.4 / 95.5, 16 / 1 B=148 S=3417 91.8 / 110.2,
// 32 / 4 B=222 S=1114 192.9 / 200.7; up to 20 % slower, never faster).
bool decode_streams(int B, int S, int Hkv, int D, int dtype, bool ragged, int chunks) {
  const double bytes = 2.0 * (dtype == SEKA_BF16 ? 2 : 4) * B * S * Hkv * D;
  return chunks == 1 && bytes * (ragged ? 0.25 : 1.0) > 300e6;
}

template <int D, bool NT>
hipError_t launch_decode_f32(const float* q, const float* K, const float* V, float* O, float* lse, const int* lens, int B, int S,
                             int Hq, int Hkv, float scale, float* part, int splits, bool on_matrix_cores, hipStream_t s) {
  const int G = Hq / Hkv, hp = decode_heads_per_wg(G);
  const float c2 = scale * 1.4426950408889634f;
  const dim3 grid(splits, Hkv * (G / hp), B);
  if (on_matrix_cores) {
    hipLaunchKernelGGL((decode_partial_f32_kernel<D, NT>), grid, dim3(kDecThreads), 0, s, q, K, V, lens, S, Hq, Hkv, hp, c2, splits, part, O,
                       lse);
  } else {
    auto kernel = hp == 1 ? decode_partial_kernel<D, 1, NT> : hp == 2 ? decode_partial_kernel<D, 2, NT>
                : hp == 3 ? decode_partial_kernel<D, 3, NT> : decode_partial_kernel<D, 4, NT>;
    hipLaunchKernelGGL(kernel, grid, dim3(kDecThreads), 0, s, q, K, V, lens, S, Hq, Hkv, c2, splits, part, O, lse);
  }
  if (splits > 1) launch_decode_finish<float, D>(part, lens, B, S, Hq, splits, O, lse, s);
  return hipGetLastError();
}

}  // namespace

hipError_t decode_static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptrs[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptrs[dev]) {                         // first call on this device, with it current: its own copy's address
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptrs[dev] = p;
  }
  *out = ptrs[dev];
  return hipSuccess;
}

// fp32: ranges of 64 tokens (128 at D = 64) where there are workgroups to spare; 64 tokens are one turn of the matrix-core
// kernel's waves.  Nothing changes where the groups alone are enough.  Not more than the library's own buffer holds, unless
// the 512-token ranges need that much.
static int decode_least_splits(int B, int S, int Hq, int Hkv, int D, int dtype) {
  const int G = Hq / Hkv, groups = B * Hkv * (G / (dtype == SEKA_BF16 ? decode_heads_per_wg(G) : decode_heads_f32(G)));
  const int splits = decode_splits(groups, S, kDecMinRows);
  if (dtype == SEKA_BF16) return splits;
  const size_t fit = kDecodeStaticScratchBytes / ((size_t)B * Hq * (D + 2) * sizeof(float));
  return std::max(splits, (int)std::min((size_t)decode_splits(groups, S, kDecMinElemsF32 / D), fit));
}

static size_t decode_state_bytes(int B, int Hq, int D, int splits) { return (size_t)B * Hq * splits * (D + 2) * sizeof(float); }

// bf16 caches of few groups at D = 128: as many ranges as give every compute unit a workgroup, down to 64 tokens each (a chain
// of 512 tokens is 8 us by itself).  us, 512-token ranges / these, in a graph on caches that are not cached: 32 / 8 heads B=1 S=1000
// 15.5 / 8.2 (on one cache over and over 10.6 / 6.7; called one by one from the host 14.4 / 9.8, the host's time for two launches),
// S=2500 14.8 / 10.1, S=10000 17.4 / 15.9; B=3 S=1500 16.7 / 11.2; B=10 S=1000 18.7 / 15.0; 8 / 2 heads B=10 S=1500 15.7 / 10.1;
// 32 / 32 B=1 S=1000 16.1 / 9.5.  Not for a second range alone (28 / 4 heads B=30 S=1000 18.6 / 19.5), nor up to about 700 tokens and at
// D = 64, where one range is one launch: called one by one on one cache S=600 7.9 / 9.9, D = 64 B=1 S=1000 7.5 / 9.8, while in a graph on
// caches that are not cached 11.0 / 8.1 and 10.8 / 6.9.  A workspace that was sized for the longer ranges gets those.
constexpr int kDecOneRange = 700, kDecFineRows = 64, kDecFineWG = 256;
static int decode_splits_of(int B, int S, int Hq, int Hkv, int D, int dtype, size_t workspace_bytes) {
  const int least = decode_least_splits(B, S, Hq, Hkv, D, dtype);
  if (dtype != SEKA_BF16 || D != 128 || S <= kDecOneRange) return least;
  const int groups = B * Hkv * (Hq / Hkv / decode_heads_per_wg(Hq / Hkv));
  const int fine = std::min({S / kDecFineRows, kDecFineWG / groups, kDecMaxSplits});
  return fine > std::max(least, 2) && decode_state_bytes(B, Hq, D, fine) <= workspace_bytes ? fine : least;
}

// bf16 caches whose groups alone give more than half of the compute units a workgroup of eight waves, and none two: one range
// up to S = 1535, and up to 2047 from 192 groups on.  Two or three ranges are workgroups of four waves, of which some compute
// units get two and others one.  us, ranges / one, in a graph on caches that are not cached, 32 / 8 heads: D = 128 S=1100 160 groups
// 28.1 / 22.8, 256 groups 34.0 / 29.3; S=2000 192 groups 45.6 / 41.3, 256 60.0 / 50.2; D = 64 S=1300 160 groups 21.6 / 16.8; ragged B=32
// S=1100 23.6 / 19.3.  Not at 128 groups (S=1300 23.4 / 23.8, S=2000 32.1 / 34.0) nor longer (192 groups S=3500 61.9 / 67.1), nor for a
// few prompts of their own lengths, where the longest is all (B=6 32 / 32 heads S=2000 29.6 / 33.2).
static bool decode_one_range(int B, int S, int groups, bool ragged) {
  return groups <= 256 && (groups >= 192 ? S < 2048 : groups > 128 && S < 1536) && (!ragged || B >= 8);
}

size_t decode_least_bytes(int B, int S, int Hq, int Hkv, int D, int dtype) {
  return decode_state_bytes(B, Hq, D, decode_least_splits(B, S, Hq, Hkv, D, dtype));
}

// A workspace that serves any smaller batch and any shorter cache too.  Fewer prompts may be cut into so many more ranges that
// they need more than B do (fp32, 32 / 8 heads, D = 128, S = 1408: 22 prompts more than 23), hence the largest
// need up to B; beyond kDecTargetWG prompts it only grows with B.  The need never falls with S.
size_t decode_workspace_bytes(int B, int S, int Hq, int Hkv, int D, int dtype) {
  auto need = [=](int b) { return decode_state_bytes(b, Hq, D, decode_splits_of(b, S, Hq, Hkv, D, dtype, SIZE_MAX)); };
  size_t most = need(B);
  for (int b = std::min(B - 1, kDecTargetWG); b > 0; --b) most = std::max(most, need(b));
  return most;
}

hipError_t launch_decode(const void* q, const void* K, const void* V, void* O, float* lse, const int* lens, int B, int S,
                         int Hq, int Hkv, int D, int dtype, float scale, void* workspace, size_t workspace_bytes, hipStream_t s) {
  const int G = Hq / Hkv, hp = decode_heads_per_wg(G);
  int splits = decode_splits_of(B, S, Hq, Hkv, D, dtype, workspace_bytes);
  const int groups = B * Hkv * (G / hp);
  if (dtype == SEKA_BF16 && splits > 1 && decode_one_range(B, S, groups, lens != nullptr)) splits = 1;
  bool on_matrix_cores = false;
  if (dtype != SEKA_BF16) {
    // the four waves of that kernel take 64 tokens per turn: whole turns, in fewer ranges (D = 128, S=1137 in 13 ranges of 88
    // or 9 of 127: 32 / 8 heads B=6 21.9 -> 16.6 us, 28 / 4 B=40 52.2 -> 44.3, 16 / 1 B=40 26.6 -> 18.4)
    constexpr int kTurn = kDecWaves * 16;
    const int turns = ((S + splits - 1) / splits + kTurn - 1) / kTurn;
    const int ranges = splits > 1 ? (S + turns * kTurn - 1) / (turns * kTurn) : 1;
    on_matrix_cores = decode_on_matrix_cores(B, S, Hkv, G / hp, D, hp, ranges, turns);
    if (on_matrix_cores) splits = ranges;
  }
  float* part = static_cast<float*>(workspace);
  const bool streams = decode_streams(B, S, Hkv, D, dtype, lens != nullptr, G / hp);
  if (dtype == SEKA_BF16) {
    const float c2 = scale * 1.4426950408889634f;
    const dim3 grid(splits, Hkv * (G / hp), B);
    const uint16_t *q16 = static_cast<const uint16_t*>(q), *K16 = static_cast<const uint16_t*>(K), *V16 = static_cast<const uint16_t*>(V);
    uint16_t* O16 = static_cast<uint16_t*>(O);
#define SEKA_DEC_LAUNCH(DD, NW, NT)                                                                                              \
    hipLaunchKernelGGL((decode_partial_mfma_kernel<DD, NW, NT>), grid, dim3(64 * NW), 0, s, q16, K16, V16, lens, S, Hq, Hkv, hp, \
                       c2, splits, part, O16, lse)
    if (splits > 1) {
      if (D == 128) {
        if (streams) SEKA_DEC_LAUNCH(128, 4, true); else SEKA_DEC_LAUNCH(128, 4, false);
        launch_decode_finish<uint16_t, 128>(part, lens, B, S, Hq, splits, O16, lse, s);
      } else {
        if (streams) SEKA_DEC_LAUNCH(64, 4, true); else SEKA_DEC_LAUNCH(64, 4, false);
        launch_decode_finish<uint16_t, 64>(part, lens, B, S, Hq, splits, O16, lse, s);
      }
    } else if (S > 128 && groups <= 256) {
      // A short cache is one workgroup's chain of blocks, half as long with twice the waves: 12.0 -> 10.3 us at S = 1000,
      // 32 / 8 heads.  Only one such workgroup fits a compute unit (LDS): at 512 workgroups 17.5 us became 20.1.
      if (D == 128) SEKA_DEC_LAUNCH(128, 8, false); else SEKA_DEC_LAUNCH(64, 8, false);
    } else {
      if (D == 128) {
        if (streams) SEKA_DEC_LAUNCH(128, 4, true); else SEKA_DEC_LAUNCH(128, 4, false);
      } else {
        if (streams) SEKA_DEC_LAUNCH(64, 4, true); else SEKA_DEC_LAUNCH(64, 4, false);
      }
    }
#undef SEKA_DEC_LAUNCH
    return hipGetLastError();
  }
  const float *q32 = static_cast<const float*>(q), *K32 = static_cast<const float*>(K), *V32 = static_cast<const float*>(V);
  auto launch = D == 128 ? (streams ? launch_decode_f32<128, true> : launch_decode_f32<128, false>)
                         : (streams ? launch_decode_f32<64, true> : launch_decode_f32<64, false>);
  return launch(q32, K32, V32, static_cast<float*>(O), lse, lens, B, S, Hq, Hkv, scale, part, splits, on_matrix_cores, s);
}

}  // namespace seka
