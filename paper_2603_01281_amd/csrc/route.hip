// seka_route: AdaSEKA expert coefficients (paper Sec. 3.3, Eq. 6; benchmark rule softmax of cosines).
//
// HBM-bound: one pass over Q[B, t0:t1, Hq, D].  Stage 1 splits the token range of every
// (batch, KV head) into chunks so that the launch has enough workgroups to fill 256 CUs; each
// workgroup streams its chunk with 16-byte loads (the G query heads of a KV head are contiguous,
// so a token contributes one contiguous G*D run) and writes D fp32 partial sums to the
// workspace.  Stage 2 (one small workgroup per (batch, KV head)) adds the partials in a fixed
// order, so the result is deterministic, then forms the M alignments and normalises them.
#include <type_traits>

#include "common.h"
#include "project_tile.h"
#include "project_wide.h"

namespace seka {

namespace {

constexpr int kRouteThreads = 256;
constexpr int kMaxChunks = 256;
constexpr int kFinishThreads = 512;
constexpr int kRouteAllRows = 128;

// Chunks per (batch, KV head): enough workgroups for the whole chip (about 2048) even when B * Hkv is small,
// at least 32 tokens per chunk, at most kMaxChunks partial sums for the second stage to add.
__host__ __device__ inline int route_chunks(int T, int BH) {
  int want = (2048 + BH - 1) / BH;
  if (want < 16) want = 16;
  if (want > kMaxChunks) want = kMaxChunks;
  int c = (T + 31) / 32;
  return c < 1 ? 1 : (c > want ? want : c);
}

template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  __device__ static void load(const float* p, float (&out)[4]) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
  }
};
template <> struct Vec16<uint16_t> {
  static constexpr int N = 8;
  __device__ static void load(const uint16_t* p, float (&out)[8]) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = __uint_as_float(w[i] << 16);
      out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

// Sum over the 64 lanes, the same value in all of them.
__device__ __forceinline__ float wave_total(float v) {
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0xB1, 0xf, 0xf, true));    // lane ^ 1
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x4E, 0xf, 0xf, true));    // lane ^ 2
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x141, 0xf, 0xf, true));   // mirrored in 8
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x140, 0xf, 0xf, true));   // mirrored in 16
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Tokens [t0, t1) that prompt b contributes, and the tensor row of its first token.  With length arrays: its last
// `window` tokens.
__device__ __forceinline__ size_t route_range(int b, int S, const int* lens, const int* cu, int total, int window, int& t0, int& t1) {
  if (lens == nullptr && cu == nullptr) return (size_t)b * S;
  size_t row_base = (size_t)b * S;
  int len;
  if (cu != nullptr) {
    const int start = min(max(cu[b], 0), total);
    len = min(cu[b + 1] - start, total - start);
    row_base = (size_t)start;
  } else {
    len = lens[b];
  }
  t1 = min(max(len, 0), S);
  t0 = max(0, t1 - window);
  return row_base;
}

// The expert prototypes of a KV head as the waves of a workgroup take them: wave w has experts w, w + NW, ...,
// element lane + 64 x.  Loaded ahead of the sums they are multiplied with.
template <int D, int NW>
struct RouteProto {
  static constexpr int N = (SEKA_MAX_EXPERTS + NW - 1) / NW, X = D / 64;
  float p[N][X];
  __device__ __forceinline__ void load(const float* proto, int h, int M, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int x = 0; x < X; ++x) {
        const int m = wave + NW * i;
        p[i][x] = m < M ? proto[((size_t)h * M + m) * D + lane + 64 * x] : 0.f;
      }
  }
};

// Expert coefficients from the mean query (qbar, in LDS behind a barrier).  Every dot product is one wave's, the rule
// is 16 lanes' of wave 0; sums are trees of a fixed shape.  (One thread per expert and one for the rule: 3 us.)
template <int D, int NW>
__device__ __forceinline__ void route_weights(const float* qbar, const RouteProto<D, NW>& pr, int M, int mode, float tau,
                                              float (&dots)[SEKA_MAX_EXPERTS], float (&pnorm2)[SEKA_MAX_EXPERTS], int wave,
                                              int lane, float* out) {
  float q[D / 64], q2 = 0.f;
#pragma unroll
  for (int x = 0; x < D / 64; ++x) {
    q[x] = qbar[lane + 64 * x];
    q2 += q[x] * q[x];
  }
  q2 = wave_total(q2);
#pragma unroll
  for (int i = 0; i < RouteProto<D, NW>::N; ++i) {
    const int m = wave + NW * i;
    if (m < M) {                                 // wave-uniform
      float d = 0.f, n2 = 0.f;
#pragma unroll
      for (int x = 0; x < D / 64; ++x) {
        d += q[x] * pr.p[i][x];
        n2 += pr.p[i][x] * pr.p[i][x];
      }
      d = wave_total(d);
      n2 = wave_total(n2);
      if (lane == 0) {
        dots[m] = d;
        pnorm2[m] = n2;
      }
    }
  }
  __syncthreads();
  if (wave != 0) return;
  const bool live = lane < M;
  const float dot = live ? dots[lane] : 0.f;
  float value;
  if (mode == SEKA_ROUTE_SOFTMAX_COS) {
    const float nn = live ? sqrtf(q2) * sqrtf(pnorm2[lane]) : 0.f;
    const float z = live ? tau * (nn >= 1e-30f ? dot / nn : 0.f) : -INFINITY;
    float zmax = z;
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, m));
    const float e = live ? expf(z - zmax) : 0.f;
    float den = e;
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) den += __shfl_xor(den, m);
    value = e / den;
  } else {
    float big = fabsf(dot);
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) big = fmaxf(big, __shfl_xor(big, m));
    value = big >= 1e-30f ? dot / big : 0.f;
  }
  if (live) out[lane] = value;
}
static_assert(SEKA_MAX_EXPERTS <= 16, "the rule runs in 16 lanes");

// grid = (chunks, B*Hkv); workspace[(bh*chunks + c)*D + d] = sum over the chunk's tokens and the G heads.
// ALL: one chunk, and the workgroup goes on to the coefficients itself (no second kernel; the workspace is not used).
template <typename T, int D, bool ALL>
__global__ __launch_bounds__(kRouteThreads) void route_partial_kernel(const T* __restrict__ Q, int S, int Hq, int Hkv,
                                                                       int t0, int t1, int chunks,
                                                                       const int* __restrict__ lens,
                                                                       const int* __restrict__ cu, int total, int window,
                                                                       float* __restrict__ workspace,
                                                                       const float* __restrict__ proto, int M, int mode,
                                                                       float tau, float* __restrict__ w_out) {
  constexpr int VE = Vec16<T>::N;
  constexpr int VPR = D / VE;                    // 16-byte vectors per (token, head) row
  constexpr int RPP = kRouteThreads / VPR;       // rows per pass
  __shared__ float red[RPP][D];
  const int G = Hq / Hkv;
  const int bh = blockIdx.y, b = bh / Hkv, h = bh % Hkv;
  const int c = blockIdx.x;
  RouteProto<D, kRouteThreads / 64> pr;
  if (ALL) pr.load(proto, h, M, threadIdx.x >> 6, threadIdx.x & 63);
  const size_t row_base = route_range(b, S, lens, cu, total, window, t0, t1);
  const int T_total = t1 - t0;
  const int per = (T_total + chunks - 1) / chunks;
  const int ta = t0 + c * per;
  const int tb = min(t1, ta + per);
  const int col = threadIdx.x % VPR, lane_row = threadIdx.x / VPR;
  float acc[VE];
#pragma unroll
  for (int i = 0; i < VE; ++i) acc[i] = 0.f;
  const int nrows = max(0, tb - ta) * G;
  // four independent 16-byte loads per thread and turn keep enough bytes in flight
  for (int row0 = lane_row; row0 < nrows; row0 += 4 * RPP) {
    float v[4][VE];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = row0 + u * RPP;
      if (row < nrows) {
        const int t = ta + row / G, g = row % G;
        Vec16<T>::load(Q + ((row_base + t) * Hq + (size_t)h * G + g) * D + col * VE, v[u]);
      } else {
#pragma unroll
        for (int i = 0; i < VE; ++i) v[u][i] = 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < VE; ++i) acc[i] += v[u][i];
  }
#pragma unroll
  for (int i = 0; i < VE; ++i) red[lane_row][col * VE + i] = acc[i];
  __syncthreads();
  __shared__ float qbar[ALL ? D : 1], dots[SEKA_MAX_EXPERTS], pnorm2[SEKA_MAX_EXPERTS];
  if (threadIdx.x < D) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < RPP; ++r) s += red[r][threadIdx.x];
    if (ALL)
      qbar[threadIdx.x] = nrows > 0 ? s * (1.0f / (float)nrows) : 0.f;
    else
      workspace[((size_t)bh * chunks + c) * D + threadIdx.x] = s;
  }
  if (ALL) {
    __syncthreads();
    route_weights<D, kRouteThreads / 64>(qbar, pr, M, mode, tau, dots, pnorm2, threadIdx.x >> 6, threadIdx.x & 63,
                                         w_out + (size_t)bh * M);
  }
}

// grid = B*Hkv, block = kFinishThreads: thread (j, d) adds the partials of chunks j, j + NJ, ... in that order, then
// the NJ sums are added in index order: a fixed order, whatever the launch.
template <int D>
__global__ __launch_bounds__(kFinishThreads) void route_finish_kernel(const float* __restrict__ workspace, int chunks, float inv_count,
                                                           const float* __restrict__ proto, int Hkv, int M, int mode,
                                                           float tau, const int* __restrict__ lens, const int* __restrict__ cu,
                                                           int total, int S, int window, int G, float* __restrict__ w_out) {
  __shared__ float qbar[D], dots[SEKA_MAX_EXPERTS], pnorm2[SEKA_MAX_EXPERTS];
  constexpr int NJ = kFinishThreads / D;
  __shared__ float part[NJ][D];
  const int bh = blockIdx.x, h = bh % Hkv;
  RouteProto<D, kFinishThreads / 64> pr;
  pr.load(proto, h, M, threadIdx.x >> 6, threadIdx.x & 63);
  if (lens != nullptr || cu != nullptr) {        // tokens this prompt contributed (the partial kernel's range)
    int t0 = 0, t1 = 0;
    route_range(bh / Hkv, S, lens, cu, total, window, t0, t1);
    const int count = (t1 - t0) * G;
    inv_count = count > 0 ? 1.0f / (float)count : 0.f;
  }
  {
    const int d = threadIdx.x % D, j = threadIdx.x / D;
    float s = 0.f;
#pragma unroll 8
    for (int c = j; c < chunks; c += NJ) s += workspace[((size_t)bh * chunks + c) * D + d];
    part[j][d] = s;
  }
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) s += part[j][threadIdx.x];
    qbar[threadIdx.x] = s * inv_count;
  }
  __syncthreads();
  route_weights<D, kFinishThreads / 64>(qbar, pr, M, mode, tau, dots, pnorm2, threadIdx.x >> 6, threadIdx.x & 63,
                                        w_out + (size_t)bh * M);
}


// ---- query projection with the routing sums in its epilogue (Sec. 3.3: the routing query is a by-product of the
// projection that produces Q, so it need not be read back) ----
//
// E of 2^22 and more, where the lane offsets of the kernels that load straight into LDS would leave 32 bits:
// Q[t, n] = sum_e X[t, e] W[n, e]  (bf16 in, fp32 accumulate, bf16 out; W is the projection weight with one row per
// output feature, the layout of a linear layer).  One workgroup = 128 tokens x 128 output features (one head at
// D = 128), four waves of 64 x 64, v_mfma_f32_32x32x16_bf16; 64-wide slices of E go through two LDS stages, the
// next slice's global loads are in flight while the current one is multiplied.  ROUTE: every wave also sums the
// rounded outputs of its 64 tokens per feature and writes them as one partial sum of seka_route's first stage, so
// route_finish_kernel completes the routing without a pass over Q.
constexpr int kProjTile = 128, kProjK = 64, kProjLd = kProjK + 8;     // LDS row stride in elements (144 bytes: conflict-free 16-byte reads)

template <bool ROUTE>
__global__ __launch_bounds__(256) void project_route_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
                                                            uint16_t* __restrict__ Qout, int E, int N, int S, int G,
                                                            int Hkv, float* __restrict__ workspace) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * 2 * kProjTile * kProjLd];   // [stage][A | B][128][72]; reused for the output tile
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, hf = lane >> 5;
  const size_t row0 = (size_t)blockIdx.y * kProjTile;     // first token of the tile (B*S is a multiple of 128)
  const int col0 = blockIdx.x * kProjTile;                // first output feature
  // global -> registers: thread t takes 64 contiguous bytes of row t / 2 of both operand tiles
  const int lrow = tid >> 1, lhalf = tid & 1;
  const uint16_t* xa = X + (row0 + lrow) * (size_t)E + 32 * lhalf;
  const uint16_t* wb = W + ((size_t)col0 + lrow) * (size_t)E + 32 * lhalf;
  // Two register sets: a slice is requested two turns before it is multiplied (one turn in flight, written to
  // LDS at the end of the next), so a turn of 16 MFMAs per wave does not have to cover the whole memory latency.
  typedef unsigned int proj_u32x4 __attribute__((ext_vector_type(4)));
  struct Slice { proj_u32x4 a0, a1, a2, a3, b0, b1, b2, b3; };
  Slice r0, r1;
#define SEKA_PROJ_GLOAD(r, kt)                                                                \
  {                                                                                           \
    const int kt_ = (kt) < nk ? (kt) : nk - 1;            /* past the end: a slice nobody uses */ \
    const proj_u32x4* pa_ = reinterpret_cast<const proj_u32x4*>(xa + (size_t)kt_ * kProjK);   \
    const proj_u32x4* pb_ = reinterpret_cast<const proj_u32x4*>(wb + (size_t)kt_ * kProjK);   \
    r.a0 = pa_[0]; r.a1 = pa_[1]; r.a2 = pa_[2]; r.a3 = pa_[3];                               \
    r.b0 = pb_[0]; r.b1 = pb_[1]; r.b2 = pb_[2]; r.b3 = pb_[3];                               \
  }
#define SEKA_PROJ_LSTORE(r, stage)                                                            \
  {                                                                                           \
    proj_u32x4* A_ = reinterpret_cast<proj_u32x4*>(lds + (stage) * (2 * kProjTile * kProjLd) + lrow * kProjLd + 32 * lhalf); \
    proj_u32x4* B_ = reinterpret_cast<proj_u32x4*>(lds + (stage) * (2 * kProjTile * kProjLd) + kProjTile * kProjLd + lrow * kProjLd + 32 * lhalf); \
    A_[0] = r.a0; A_[1] = r.a1; A_[2] = r.a2; A_[3] = r.a3;                                   \
    B_[0] = r.b0; B_[1] = r.b1; B_[2] = r.b2; B_[3] = r.b3;                                   \
  }
  // Tokens are the MFMA's rows and features its columns, so that a lane owns one feature column and its 16
  // registers are 16 tokens: the routing sum over tokens is a sum over registers.
#define SEKA_PROJ_COMPUTE(stage)                                                              \
  {                                                                                           \
    const uint16_t* A_ = lds + (stage) * (2 * kProjTile * kProjLd);                           \
    const uint16_t* B_ = A_ + kProjTile * kProjLd;                                            \
    _Pragma("unroll") for (int ks = 0; ks < kProjK / 16; ++ks) {                              \
      bf16x8 a_[2], b_[2];                                                                    \
      _Pragma("unroll") for (int i = 0; i < 2; ++i)                                           \
        a_[i] = *reinterpret_cast<const bf16x8*>(A_ + (64 * wm + 32 * i + l32) * kProjLd + 16 * ks + 8 * hf); \
      _Pragma("unroll") for (int j = 0; j < 2; ++j)                                           \
        b_[j] = *reinterpret_cast<const bf16x8*>(B_ + (64 * wn + 32 * j + l32) * kProjLd + 16 * ks + 8 * hf); \
      _Pragma("unroll") for (int i = 0; i < 2; ++i)                                           \
        _Pragma("unroll") for (int j = 0; j < 2; ++j)                                         \
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_[i], b_[j], acc[i][j], 0, 0, 0); \
    }                                                                                         \
  }
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int nk = E / kProjK;
  SEKA_PROJ_GLOAD(r0, 0)
  SEKA_PROJ_LSTORE(r0, 0)
  __syncthreads();
  SEKA_PROJ_GLOAD(r0, 1)
  int kt = 0;
  for (; kt + 1 < nk; kt += 2) {
    // even turn: stage 0 holds slice kt, set 0 holds slice kt + 1
    SEKA_PROJ_GLOAD(r1, kt + 2)
    SEKA_PROJ_COMPUTE(0)
    SEKA_PROJ_LSTORE(r0, 1)
    __syncthreads();
    // odd turn: stage 1 holds slice kt + 1, set 1 holds slice kt + 2 (past the end: a copy of the last slice)
    SEKA_PROJ_GLOAD(r0, kt + 3)
    SEKA_PROJ_COMPUTE(1)
    SEKA_PROJ_LSTORE(r1, 0)
    __syncthreads();
  }
  if (kt < nk) SEKA_PROJ_COMPUTE(0)                        // an odd number of slices: the last one sits in stage 0
  __syncthreads();
#undef SEKA_PROJ_GLOAD
#undef SEKA_PROJ_LSTORE
#undef SEKA_PROJ_COMPUTE
  // ---- epilogue: round, sum for the routing, stage the tile in LDS, store 16 bytes per lane ----
  constexpr int OLD = kProjTile + 8;                      // output tile row stride in elements
  uint16_t* Ct = lds;                                     // [128][136] = 34816 B <= the operand stages
  float colsum[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const __bf16 v = (__bf16)acc[i][j][r];
        colsum[j] += (float)v;
        const int m = 64 * wm + 32 * i + 8 * (r >> 2) + 4 * hf + (r & 3);
        Ct[m * OLD + 64 * wn + 32 * j + l32] = __builtin_bit_cast(uint16_t, v);
      }
  if (ROUTE) {
    // this wave's 64 tokens lie in one prompt (S is a multiple of 128); feature column -> (head, d)
    const size_t tok = row0 + 64 * wm;
    const int b = (int)(tok / S), tchunk = (int)(tok % S) / 64;
    const int hq = col0 / 128, h = hq / G, g = hq % G;            // D = 128: one tile column block = one head
    const int chunks = (S / 64) * G;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float tot = colsum[j] + __shfl_xor(colsum[j], 32);    // the other 32 tokens of the wave
      if (hf == 0)
        workspace[(((size_t)b * Hkv + h) * chunks + (size_t)tchunk * G + g) * 128 + 64 * wn + 32 * j + l32] = tot;
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < (kProjTile * kProjTile / 8) / 256; ++it) {
    const int idx = tid + 256 * it, m = idx / (kProjTile / 8), c8 = idx % (kProjTile / 8);
    const uint4 v = *reinterpret_cast<const uint4*>(Ct + m * OLD + 8 * c8);
    *reinterpret_cast<uint4*>(Qout + (row0 + m) * (size_t)N + col0 + 8 * c8) = v;
  }
}

}  // namespace

size_t route_workspace_bytes(int B, int Hkv, int D, int t0, int t1) {
  return (size_t)B * Hkv * route_chunks(t1 - t0, B * Hkv) * D * sizeof(float);
}

hipError_t launch_route(const void* Q, int B, int S, int Hq, int Hkv, int D, int dtype, const float* proto, int M,
                        int t0, int t1, int mode, float tau, float* w_out, void* workspace, hipStream_t s,
                        const int* lens, const int* cu, int total, int window) {
  const bool ragged = lens != nullptr || cu != nullptr;
  if (ragged) { t0 = 0; t1 = window < S ? window : S; }      // the longest range a prompt can have
  const int chunks = route_chunks(t1 - t0, B * Hkv);
  const dim3 grid(chunks, B * Hkv);
  float* ws = static_cast<float*>(workspace);
  const float inv_count = 1.0f / ((float)(t1 - t0) * (float)(Hq / Hkv));
  // Up to 128 rows (the last-token rule: G of them) one workgroup per (prompt, KV head) does everything: a second kernel
  // would cost what the first does (8.2 us for the two at 64 tokens x 4 heads, 4.4 in one).
  const bool all = (long long)(t1 - t0) * (Hq / Hkv) <= kRouteAllRows;
#define SEKA_ROUTE_CASE(T, DD)                                                                                       \
  do {                                                                                                               \
    if (all) {                                                                                                       \
      hipLaunchKernelGGL((route_partial_kernel<T, DD, true>), dim3(1, B * Hkv), dim3(kRouteThreads), 0, s,           \
                         static_cast<const T*>(Q), S, Hq, Hkv, t0, t1, 1, lens, cu, total, window, ws, proto, M,     \
                         mode, tau, w_out);                                                                          \
    } else {                                                                                                         \
      hipLaunchKernelGGL((route_partial_kernel<T, DD, false>), grid, dim3(kRouteThreads), 0, s,                      \
                         static_cast<const T*>(Q), S, Hq, Hkv, t0, t1, chunks, lens, cu, total, window, ws, proto, M, \
                         mode, tau, w_out);                                                                          \
      hipLaunchKernelGGL((route_finish_kernel<DD>), dim3(B * Hkv), dim3(kFinishThreads), 0, s, ws, chunks, inv_count, \
                         proto, Hkv, M, mode, tau, lens, cu, total, S, window, Hq / Hkv, w_out);                     \
    }                                                                                                                \
  } while (0)
  if (dtype == SEKA_BF16) {
    if (D == 128) SEKA_ROUTE_CASE(uint16_t, 128); else SEKA_ROUTE_CASE(uint16_t, 64);
  } else {
    if (D == 128) SEKA_ROUTE_CASE(float, 128); else SEKA_ROUTE_CASE(float, 64);
  }
#undef SEKA_ROUTE_CASE
  return hipGetLastError();
}


size_t project_route_workspace_bytes(int B, int S, int Hq) {
  return (size_t)B * Hq * (S / 64) * 128 * sizeof(float);
}

// Which tiles a projection takes: the least estimate of 3 us + (slices of E) x (sum over rounds of 256 workgroups of a slice's
// time).  A slice costs more the more of the chip is busy (its power, HBM): measured, us at an eighth, half and all of the
// compute units, 256 x 256 0.95 / 1.1 / 1.6, 256 x 128 0.69 / 0.75 / 0.94, 128 x 128 0.38 / 0.41 / 0.53, 128 x 64
// 0.27 / 0.29 / 0.32.  us for E = 4096, N = 4096 in that order of tiles (128 x 128 register-staged before): 128 tokens
// 60 / 46 / 27 / 20 (44), 512 62 / 48 / 29 / 24 (46), 1024 64 / 51 / 37 / 48 (51), 2048 69 / 63 / 72 / 89, 32768 811 with the
// first; 1536 tokens E = 2880 48 / 40 / 46 / 51, 4096 x 1024 x 5120 82 / 67 / 44 / 57 (66).  Those are figures of 32 x 32 x 16
// products and three stages; with 16 x 16 x 32 ones and four stages for 128 x 64 all four are up to 10 % faster and the rule still takes a kind
// within 0.11 % of the best one (geometric mean over 260 shapes timed with each, at most 2.5 %; always 128 x 128 14 %).
inline int project_tile_of(long long tokens, int N, int E) {
  constexpr struct { int bm, bn; double alone, crowded; } kinds[4] = {{256, 256, 0.92, 0.66}, {256, 128, 0.68, 0.26}, {128, 128, 0.375, 0.155}, {128, 64, 0.27, 0.05}};
  int best = 0;
  double least = 0;
  for (int i = 0; i < 4; ++i) {
    const long long tiles = ((tokens + kinds[i].bm - 1) / kinds[i].bm) * ((N + kinds[i].bn - 1) / kinds[i].bn);
    const long long full = (tiles - 1) / 256;
    const double last = (double)(tiles - 256 * full) / 256;
    const double cost = 3 + E / kWideK * (full * (kinds[i].alone + kinds[i].crowded) + kinds[i].alone + kinds[i].crowded * last * last);
    if (i == 0 || cost < least) {
      least = cost;
      best = i;
    }
  }
  return best;
}

hipError_t launch_project_route(const void* X, const void* W, int E, void* Qout, int B, int S, int Hq, int Hkv,
                                const float* proto, int M, int mode, float tau, float* w_out, void* workspace,
                                hipStream_t s) {
  const int N = Hq * 128, G = Hq / Hkv;
  const long long tokens = (long long)B * S;
  float* ws = static_cast<float*>(workspace);
  const uint16_t *x = static_cast<const uint16_t*>(X), *wq = static_cast<const uint16_t*>(W);
  uint16_t* q = static_cast<uint16_t*>(Qout);
  auto launch = [&](auto kernel, int bm, int bn, int threads, size_t smem) {
    const long long tiles = ((tokens + bm - 1) / bm) * ((N + bn - 1) / bn);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(threads), smem, s, x, wq, q, E, tokens, N, S, G, Hkv, ws);
    return hipSuccess;
  };
#define SEKA_PROJ_TILE(BM, BN, WM, WN, NS)                                                                           \
  launch(w_out ? project_route_tile_kernel<BM, BN, WM, WN, NS, true> : project_route_tile_kernel<BM, BN, WM, WN, NS, false>, BM, BN, \
         64 * WM * WN, (size_t)NS * (BM + BN) * kWideK * 2)
  hipError_t e = hipSuccess;
  if (E >= (1 << 22)) {
    const dim3 grid(N / kProjTile, (unsigned)(tokens / kProjTile));
    if (w_out) hipLaunchKernelGGL((project_route_kernel<true>), grid, dim3(256), 0, s, x, wq, q, E, N, S, G, Hkv, ws);
    else hipLaunchKernelGGL((project_route_kernel<false>), grid, dim3(256), 0, s, x, wq, q, E, N, S, G, Hkv, ws);
  } else {
    switch (project_tile_of(tokens, N, E)) {
      case 0: e = launch(w_out ? project_route_wide_kernel<true> : project_route_wide_kernel<false>, kWideTile, kWideTile, 512, (size_t)8 * kWideHalf); break;
      case 1: e = SEKA_PROJ_TILE(256, 128, 4, 2, 3); break;
      case 2: e = SEKA_PROJ_TILE(128, 128, 2, 4, 3); break;
      default: e = SEKA_PROJ_TILE(128, 64, 2, 2, 4); break;
    }
  }
#undef SEKA_PROJ_TILE
  if (e != hipSuccess) return e;
  if (w_out != nullptr) {
    const float inv_count = 1.0f / ((float)S * (float)G);
    hipLaunchKernelGGL((route_finish_kernel<128>), dim3(B * Hkv), dim3(kFinishThreads), 0, s, ws, (S / 64) * G, inv_count,
                       proto, Hkv, M, mode, tau, static_cast<const int*>(nullptr), static_cast<const int*>(nullptr), 0, S, 0, G,
                       w_out);
  }
  return hipGetLastError();
}

}  // namespace seka
