// Eigenvalues and eigenvectors of the Gram matrices of the offline stage (fp64, one D x D matrix per KV head):
// Householder reduction to a tridiagonal T (one workgroup per head), then every eigenvalue on a wave of its own:
// multisection on sign counts, its vector from a twisted factorisation, and the reflectors applied back to it.
#pragma once
#include <type_traits>

#include "common.h"

namespace seka {

// What the kernels hand on, in doubles, per head (over the head's slot of Omega, which nothing reads any more).
template <int D>
struct EigWork {
  // kMinor: pairs (diagonal element, square of the off-diagonal element above it) of T, row by row
  static constexpr int kMinor = 0, kOff = 2 * D, kTau = 3 * D, kLambda = 4 * D, kUnit = 5 * D, kStatus = 5 * D + 1, kBad = 5 * D + 2;
  static_assert((kBad + D) * 2 <= D * D, "fits the slot");
};

// What counts as nothing of a sum of squares beside T's diagonal, of a matrix whose largest element is 1 to 4: 1e-20 of it is
// below its rounding by four orders.  (In what is left of a matrix of exactly low rank every further step is some 1e-16 of the
// one before, and 1 / h^2 leaves fp64 when n2 passes 1e-154.)
constexpr double kEigNothing = 1e-40;

// Off-diagonal elements below this share of what their rows and columns are: a matrix that is diagonal already.
constexpr double kEigApart = 2e-7;

__device__ __forceinline__ bool is_finite(double v) {               // by its bits
  return ((unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32) & 0x7ff00000u) != 0x7ff00000u;
}
__device__ __forceinline__ unsigned wave_max(unsigned v) {
  auto step = [&](unsigned u) __attribute__((always_inline)) { v = max(v, u); };
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true));
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true));
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true));   // mirrored in 8
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true));   // mirrored in 16
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (unsigned)__builtin_amdgcn_readfirstlane((int)max(b[0], b[1]));
}
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// b in the lanes where `mask` is all ones, a where it is 0: bit selects.  (From `lane & 8 ? b : a` the compiler makes the
// comparison anew for every element: 50 of them in a step of the reduction below.)
__device__ __forceinline__ double select_double(double a, double b, unsigned mask) {
  const unsigned long long ua = __builtin_bit_cast(unsigned long long, a), ub = __builtin_bit_cast(unsigned long long, b);
  const unsigned lo = (mask & (unsigned)ub) | (~mask & (unsigned)ua), hi = (mask & (unsigned)(ub >> 32)) | (~mask & (unsigned)(ua >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Sum over 16 consecutive lanes, the same bits in all of them.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_double<0xB1>(v);                       // lane ^ 1
  v += dpp_double<0x4E>(v);                       // lane ^ 2
  v += dpp_double<0x141>(v);                      // mirrored in 8
  return v + dpp_double<0x140>(v);                // mirrored in 16
}
struct DoublePair { double a, b; };
// {a, b} with the odd rows of 16 lanes of a and the even ones of b exchanged, or the upper half of a and the lower half of b
template <int LANES>
__device__ __forceinline__ DoublePair swap_double(double a, double b) {
  const unsigned long long ua = __builtin_bit_cast(unsigned long long, a), ub = __builtin_bit_cast(unsigned long long, b);
  auto join = [](unsigned lo, unsigned hi) __attribute__((always_inline)) {
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
  };
  if constexpr (LANES == 16) {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    return {join(lo[0], hi[0]), join(lo[1], hi[1])};
  } else {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    return {join(lo[0], hi[0]), join(lo[1], hi[1])};
  }
}
__device__ __forceinline__ double wave_sum(double v) {
  v = row_sum(v);
  const DoublePair s = swap_double<16>(v, v);
  v = s.a + s.b;
  const DoublePair t = swap_double<32>(v, v);
  return t.a + t.b;
}
// The sum of a over the wave in lanes 0 - 31, that of b in lanes 32 - 63.
__device__ __forceinline__ double half_sums(double a, double b) {
  const DoublePair s = swap_double<32>(a, b);
  const double v = s.a + s.b;
  const DoublePair t = swap_double<16>(v, v);
  return row_sum(t.a + t.b);
}
__device__ __forceinline__ double lane_double(double v, int l) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l), hi = (unsigned)__builtin_amdgcn_readlane((int)(u >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Hardware estimates (2^-24 and better) and one correction of third order.
__device__ __forceinline__ double fast_reciprocal(double v) {
  const double r = __builtin_amdgcn_rcp(v), e = __builtin_fma(-v, r, 1.0);
  return __builtin_fma(__builtin_fma(e, e, e), r, r);
}
__device__ __forceinline__ double fast_rsqrt(double v) {
  const double r = __builtin_amdgcn_rsq(v), e = __builtin_fma(-v * r, r, 1.0);
  return __builtin_fma(__builtin_fma(0.375 * e, e, 0.5 * e), r, r);
}

// T = Q^T B Q, B = 2^-e times the head's Gram matrix (e even, largest element in [1, 4): B's own, from 2^-298 to 2^263,
// would leave fp32 further on; powers of two, no bit changes).  grid (Hkv), 256 threads as 16 x 16: thread (ti, tj) keeps
// elements (ti + 16 i, tj' + 16 j), tj' = tj ^ ti, in registers; rows and columns that are done leave in chunks of 16 (`P`).
// Step k takes x = row k right of the diagonal, v = x - alpha e_{k+1}, H = I - v v^T / h:
//   every thread holds x at its columns; y = B x is summed over 16 lanes (all columns of a row), and y, row k + 1 as it
//   stands and x go to LDS; behind the step's one barrier every thread forms q = B v = y - alpha row_{k+1} and
//   w = q / h - (v.q / 2 h^2) v at its columns, takes v and w at its rows from lane 0 of its 16 (tj' = ti there),
//   B -= v w^T + w v^T, and the next x from row k + 1, which needs no second barrier.
// The lanes of every 16 hold the columns in an order of their own, but the sums pair them alike (all partners differ by an
// exclusive or), so every thread has the same bits of v, w and alpha.
// The reflectors replace the strictly upper triangle of the Gram matrix (row k: v of step k), the diagonal and the lower
// triangle stay as they are.
// Bound by a step's chain (sums over 16 lanes, LDS, barrier: 1000 cycles) and by issue, one wave per SIMD: 3100 cycles in
// the first steps at D = 128, of which 950 B's update, 950 the last; 107 us at D = 128, 40 at D = 64.  More waves repeat
// the vectors' share of the work and wait for the LDS port: 512 threads 133 us, 1024 183.
template <int D>
__global__ __launch_bounds__(256) void tridiag_kernel(double* gram, float* omega) {
  constexpr int NC = D / 16;
  constexpr int LD = NC + 2;                      // 16-byte reads by 16 lanes without conflicts
  typedef EigWork<D> W;
  __shared__ __attribute__((aligned(16))) double ybuf[2][16 * LD], cbuf[2][16 * LD], xbuf[2][16 * LD];      // index j at (j % 16) LD + j / 16
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, ti = tid >> 4, tj = (tid ^ ti) & 15;
  const int row_at = ti * LD, col_at = tj * LD;
  double* B = gram + (size_t)h * D * D;
  double* work = reinterpret_cast<double*>(omega + (size_t)h * D * D);
  double a[NC][NC], x[NC];                        // x at the thread's columns
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j) a[i][j] = B[(size_t)(ti + 16 * i) * D + tj + 16 * j];
#pragma unroll
  for (int j = 0; j < NC; ++j) x[j] = B[tj + 16 * j];
  double dk = B[0], x0 = B[1];                    // of row k: its diagonal element, and the one beside it
  unsigned top = 0;                               // high word of the largest diagonal element (they are sums of squares)
#pragma unroll
  for (int q = 0; q < D / 64; ++q)
    top = max(top, (unsigned)(__builtin_bit_cast(unsigned long long, B[(size_t)(lane + 64 * q) * (D + 1)]) >> 32) & 0x7fffffffu);
  top = wave_max(top);
  const bool finite = top < 0x7ff00000u;
  const int e = top && finite ? ((int)(top >> 20) - 1023) & ~1 : 0;
  if (tid == 0) {
    work[W::kUnit] = __builtin_bit_cast(double, (unsigned long long)(1023 + e / 2) << 52);
    work[W::kStatus] = finite ? 0.0 : 1.0;       // 2: diagonal, with eigenvalues too close for what follows
    work[W::kMinor + 1] = 0.0;
  }
  if (!finite) return;                            // the same in every wave
  const double down = __builtin_bit_cast(double, (unsigned long long)(1023 - e) << 52);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    x[i] *= down;
#pragma unroll
    for (int j = 0; j < NC; ++j) a[i][j] *= down;
  }
  dk *= down;
  x0 *= down;
  // A matrix that is diagonal with equal elements would come back from all of this with directions that cannot be told apart,
  // and have the iteration before it, which finds nothing to rotate there (D = 128, 8 heads: 318 -> 172 us; 0.2 us for the
  // others, which row 0 rules out).  Row 0 is in every wave, so all of them go the same way.
  bool some_off = false;
  double dc[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    dc[j] = B[(size_t)(tj + 16 * j) * (D + 1)] * down;
    some_off |= tj + 16 * j > 0 && x[j] * x[j] > kEigApart * kEigApart * dk * dc[j];
  }
  if (!__any(some_off)) {
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const double dr = B[(size_t)(ti + 16 * i) * (D + 1)] * down;
#pragma unroll
      for (int j = 0; j < NC; ++j) some_off |= ti + 16 * i != tj + 16 * j && a[i][j] * a[i][j] > kEigApart * kEigApart * dr * dc[j];
    }
    if (tid < 16) {
#pragma unroll
      for (int j = 0; j < NC; ++j) ybuf[0][tj + 16 * j] = dc[j];
    }
    some_off = __syncthreads_or(some_off);
    bool twins = false;                           // the limits are those of svd_kernel, a little tighter
    if (tid < D && !some_off) {
      const double me = ybuf[0][tid], limit = 0.9 * fmax(1e-13, 1e-7 * me);
#pragma unroll 8
      for (int i = 0; i < D; ++i) twins |= i != tid && me > 1e-9 && fabs(ybuf[0][i] - me) < limit;
    }
    if (__syncthreads_or(twins)) {
      if (tid == 0) work[W::kStatus] = 2.0;
      return;
    }
  }
  unsigned up8 = -(lane >> 3 & 1), up4 = -(lane >> 2 & 1), up2 = -(lane >> 1 & 1);
  asm("" : "+v"(up8), "+v"(up4), "+v"(up2));     // or they become comparisons again
  const int row = NC == 8 ? ((lane >> 3 & 1) << 2) + ((lane >> 2 & 1) << 1) + (lane >> 1 & 1) : ((lane >> 3 & 1) << 1) + (lane >> 2 & 1);
  int buf = 0;
  auto steps = [&](auto phase) __attribute__((always_inline)) {
    constexpr int P = decltype(phase)::value;     // rows and columns below 16 P are done
    const int k_end = 16 * P + 16 < D - 2 ? 16 * P + 16 : D - 2;
    for (int k = 16 * P; k < k_end; ++k) {
      if (16 * P + tj <= k) x[P] = 0.0;
      const int k1 = k + 1, at1 = (k1 & 15) * LD + (k1 >> 4), at2 = ((k1 + 1) & 15) * LD + ((k1 + 1) >> 4);
      double y[NC], n2 = 0.0;
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        y[i] = 0.0;
        if (i < P) continue;
#pragma unroll
        for (int j = P; j < NC; ++j) y[i] = __builtin_fma(a[i][j], x[j], y[i]);
      }
#pragma unroll
      for (int j = P; j < NC; ++j) n2 = __builtin_fma(x[j], x[j], n2);
      // sums over the 16 lanes: halves of the rows change sides, so that a lane ends with one row's total
      double total;
      if constexpr (NC == 8) {
        double t[4], u[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {             // rows i + 4 to lanes 8 - 15 (row_ror:8), rows i + 2 to odd fours, ...
          if (i + 4 < P) t[i] = 0.0;
          else if (i < P) t[i] = y[i + 4] + dpp_double<0x128>(y[i + 4]);
          else t[i] = select_double(y[i], y[i + 4], up8) + dpp_double<0x128>(select_double(y[i + 4], y[i], up8));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (P >= 4 && i + 6 < P) u[i] = 0.0;
          else u[i] = select_double(t[i], t[i + 2], up4) + dpp_double<0x141>(select_double(t[i + 2], t[i], up4));
        }
        total = select_double(u[0], u[1], up2) + dpp_double<0x4E>(select_double(u[1], u[0], up2));
      } else {
        static_assert(NC == 4, "head dimensions 64 and 128");
        double t[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) t[i] = select_double(y[i], y[i + 2], up8) + dpp_double<0x128>(select_double(y[i + 2], y[i], up8));
        total = select_double(t[0], t[1], up4) + dpp_double<0x141>(select_double(t[1], t[0], up4));
        total += dpp_double<0x4E>(total);
      }
      total += dpp_double<0xB1>(total);
      n2 = row_sum(n2);
      // v = x - alpha e_{k+1}, h = v.v / 2; nothing right of the diagonal: H = I
      const bool some = n2 > kEigNothing;
      const double alpha = some ? -copysign(n2 * fast_rsqrt(n2), x0) : 0.0, v1 = x0 - alpha;
      const double inv = some ? fast_reciprocal(__builtin_fma(-alpha, x0, n2)) : 0.0;      // 1 / h
      if ((lane & (16 / NC - 1)) == 0) ybuf[buf][row_at + row] = total;
      if (ti == (k1 & 15)) {
        const bool here = P + 1 >= NC || k1 >> 4 == P;
#pragma unroll
        for (int j = P; j < NC; ++j) cbuf[buf][col_at + j] = here ? a[P][j] : a[P + 1 < NC ? P + 1 : P][j];
      }
      if (ti == 0) {                              // only x at k + 2 is asked for
        xbuf[buf][col_at + P] = x[P];
        if (P + 1 < NC) xbuf[buf][col_at + P + 1] = x[P + 1 < NC ? P + 1 : P];
      }
      __syncthreads();
      const double c1 = cbuf[buf][at1], y1 = ybuf[buf][at1], c2 = cbuf[buf][at2], y2 = ybuf[buf][at2], x2 = xbuf[buf][at2];
      double c[NC], w[NC], vq = 0.0;
#pragma unroll
      for (int j = P; j < NC; ++j) {
        c[j] = cbuf[buf][col_at + j];
        w[j] = __builtin_fma(-alpha, c[j], ybuf[buf][col_at + j]);
      }
      // x becomes v: its element k + 1 lies in chunk P or at the start of the next
      if (16 * P + tj == k1) x[P] = v1;
      if constexpr (P + 1 < NC) if (16 * P + 16 + tj == k1) x[P + 1] = v1;
#pragma unroll
      for (int j = P; j < NC; ++j) vq = __builtin_fma(x[j], w[j], vq);
      vq = row_sum(vq);
      const double kk = 0.5 * vq * inv * inv;
#pragma unroll
      for (int j = P; j < NC; ++j) w[j] = __builtin_fma(-kk, x[j], w[j] * inv);
      if (16 * P + tj <= k) w[P] = 0.0;
      const double w1 = __builtin_fma(-kk, v1, __builtin_fma(-alpha, c1, y1) * inv);
      const double w2 = __builtin_fma(-kk, x2, __builtin_fma(-alpha, c2, y2) * inv);
      if (ti == (k & 15)) {                       // the reflector, and this row of T
#pragma unroll
        for (int j = P; j < NC; ++j)
          if (j > P || 16 * P + tj > k) B[(size_t)k * D + tj + 16 * j] = x[j];
        if (tj == 0) {
          work[W::kMinor + 2 * k] = dk;
          work[W::kMinor + 2 * k + 3] = fmax(alpha * alpha, kEigNothing);      // never 0: a zero minor is followed by one that is not
          work[W::kOff + k] = alpha;
          work[W::kTau + k] = inv;
        }
      }
#pragma unroll
      for (int i = P; i < NC; ++i) {
        const double vr = dpp_double<0x150>(x[i]), wr = dpp_double<0x150>(w[i]);      // row_newbcast:0
#pragma unroll
        for (int j = P; j < NC; ++j) a[i][j] = __builtin_fma(-wr, x[j], __builtin_fma(-vr, w[j], a[i][j]));
      }
      dk = __builtin_fma(-2.0 * v1, w1, c1);
      x0 = __builtin_fma(-w1, x2, __builtin_fma(-v1, w2, c2));
#pragma unroll
      for (int j = P; j < NC; ++j) x[j] = __builtin_fma(-w1, x[j], __builtin_fma(-v1, w[j], c[j]));
      buf ^= 1;
    }
  };
  steps(std::integral_constant<int, 0>{});
  steps(std::integral_constant<int, 1>{});
  steps(std::integral_constant<int, 2>{});
  steps(std::integral_constant<int, 3>{});
  if constexpr (NC == 8) {
    steps(std::integral_constant<int, 4>{});
    steps(std::integral_constant<int, 5>{});
    steps(std::integral_constant<int, 6>{});
    steps(std::integral_constant<int, 7>{});
  }
  if (tid == 255 - 15) {                          // ti = tj = 15: the last 2 x 2
    work[W::kMinor + 2 * (D - 2)] = dk;
    work[W::kMinor + 2 * (D - 2) + 3] = fmax(x[NC - 1] * x[NC - 1], kEigNothing);
    work[W::kOff + D - 2] = x[NC - 1];
    work[W::kOff + D - 1] = 0.0;
    work[W::kMinor + 2 * (D - 1)] = a[NC - 1][NC - 1];
  }
}

// Four eigenvalues of T per workgroup (indices 4 blockIdx.x + wave from below), and their vectors.  grid (D / 4, Hkv), 384
// threads: waves 0-3 have an eigenvalue each; meanwhile wave 4 factors T + delta = L Delta L^T (delta: 2e-14 of T's norm,
// which makes T, a Gram matrix up to rounding, definite) and wave 5 forms the products of neighbouring reflectors.
//  1. Multisection: the signs of det(T_i - x), i = 1 .. D, change as often as there are eigenvalues below x (the recurrence
//     of the leading minors, no division; rescaled every 8 steps); 64 lanes cut the interval in 65, nine times.  T comes by
//     scalar loads (from LDS the four waves wait for its one port: 41 cycles per row instead of 25).
//  2. The vectors: forward and backward factorisation of L Delta L^T - lambda, joined where the pivot is smallest (the twisted
//     factorisation of Parlett and Dhillon, Linear Algebra and its Applications 267, 1997, and 387, 2004), twice, with the
//     eigenvalue corrected in between.  Chains of D steps: wave 0 runs all eight of them in lanes 0 - 7 (a wave
//     per eigenvalue has four times the LDS instructions and takes twice as long).  On the factored form vectors of
//     eigenvalues that differ by a fraction r of themselves are orthogonal to about D 2^-53 / r, whatever lies between
//     them and the largest one (on T itself the tail of the spectrum would lose its directions).
//  3. u = H_0 ... H_{D-3} z, a wave per vector, D / 64 elements per lane, reflectors from L2, two at a time.
// Columns whose eigenvalue is too small for a direction (below the caller's limit) are written as zeros.
// kLambda: all D of them, ascending; kBad: 1 where the two factorisations did not end at the eigenvalue they started from.
constexpr int kEigThreads = 384;
struct EigPair { double x, y; };
typedef const __attribute__((address_space(4))) double* eig_const_ptr;      // uniform addresses: scalar loads
template <int D>
__global__ __launch_bounds__(kEigThreads) void eig_kernel(const double* __restrict__ gram, float* omega, float* __restrict__ U_out,
                                                          double direction_limit) {
  typedef EigWork<D> W;
  typedef EigPair Pair;
  constexpr int RPL = D / 64;
  __shared__ __attribute__((aligned(16))) Pair fact[2][D];         // Delta_i, l_i^2 Delta_i; the same backwards and swapped
  __shared__ __attribute__((aligned(16))) Pair pivots[4][2][D + 1];      // (eight lanes, eight banks) state before a step, reciprocal pivot
  __shared__ double off[2][D], tau[D];                             // -e_i forwards and backwards
  __shared__ double zbuf[4][2][D + 9], cross[D / 2];               // elements ahead of and behind r; v_k . v_{k-1}, k = D - 1 - 2 j
  __shared__ double lam_s[4], zz_s[4];
  __shared__ int r_s[4], bad_s[4];
  __shared__ __attribute__((aligned(16))) float out[D][4];
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* work = reinterpret_cast<double*>(omega + (size_t)h * D * D);
  const eig_const_ptr T = (eig_const_ptr)(work + W::kMinor);
  if (work[W::kStatus] != 0.0) return;                             // nothing here reads on
  double norm = 0.0, largest = 0.0;                                // Gershgorin bound of T, largest diagonal element
#pragma unroll
  for (int x = 0; x < RPL; ++x) {
    const int i = lane + 64 * x;
    const double d = work[W::kMinor + 2 * i], e = work[W::kOff + i], b = i ? work[W::kOff + i - 1] : 0.0;
    norm = fmax(norm, fabs(d) + fabs(e) + fabs(b));
    largest = fmax(largest, d);
    if (wave == 0) {
      off[0][i] = -e;
      off[1][i < D - 1 ? D - 2 - i : D - 1] = -e;                  // e_{D-1} = 0
      tau[i] = i < D - 2 ? work[W::kTau + i] : 0.0;
    }
  }
#pragma unroll
  for (int s = 1; s < 64; s *= 2) {
    norm = fmax(norm, __shfl_xor(norm, s));
    largest = fmax(largest, __shfl_xor(largest, s));
  }
  const double delta = 2e-14 * norm;
  const int idx = 4 * blockIdx.x + wave;
  const double* rows = gram + (size_t)h * D * D + lane;
  // reflectors k, k - 1, ..., k - 7, elements lane + 64 x for x >= X0 (those below are zero); a reflector starts behind its index
  auto fetch_rows = [&](int k, double (&to)[8][RPL], auto first) __attribute__((always_inline)) {
    constexpr int X0 = decltype(first)::value;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int x = X0; x < RPL; ++x) to[j][x] = rows[(size_t)(k - j) * D + 64 * x];
  };
  if (wave == 4) {
    double diag[RPL], sq[RPL];                                     // lane l: rows l, l + 64
#pragma unroll
    for (int x = 0; x < RPL; ++x) {
      diag[x] = work[W::kMinor + 2 * (lane + 64 * x)] + delta;
      sq[x] = work[W::kMinor + 2 * (lane + 64 * x) + 1];
    }
    double d = lane_double(diag[0], 0);
    __builtin_amdgcn_s_setprio(2);                                 // one long chain beside a wave that always has something to issue
#pragma unroll
    for (int x = 0; x < RPL; ++x)
      for (int i = 0; i < 64; ++i) {                               // row 64 x + i; the next one's elements
        const bool over = i == 63;
        const double dn = over && x + 1 < RPL ? lane_double(diag[x + 1 < RPL ? x + 1 : x], 0) : lane_double(diag[x], (i + 1) & 63);
        double le = over && x + 1 < RPL ? lane_double(sq[x + 1 < RPL ? x + 1 : x], 0) : lane_double(sq[x], (i + 1) & 63);
        le = over && x + 1 == RPL ? 0.0 : le * fast_reciprocal(fmax(d, 1e-30));
        if (lane == 0) {
          const int at = 64 * x + i;
          fact[0][at] = Pair{d, le};
          fact[1][at < D - 1 ? D - 2 - at : D - 1] = Pair{le, d};
        }
        d = dn - le;
      }
  } else if (wave == 5) {
    double v[2][8][RPL];
    constexpr auto all = std::integral_constant<int, 0>{};
    fetch_rows(D - 1, v[0], all);
    for (int k0 = D - 1; k0 >= 0; k0 -= 16) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int k = k0 - 8 * c;
        fetch_rows(max(k - 8, 7), v[c ^ 1], all);
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
          double s = 0.0;
#pragma unroll
          for (int x = 0; x < RPL; ++x) s = __builtin_fma(lane + 64 * x > k - j ? v[c][j][x] : 0.0, v[c][j + 1][x], s);
          s = wave_sum(s);
          if (lane == 0) cross[(D - 1 - k + j) / 2] = s;
        }
      }
    }
  } else {
    double lo = -1e-13 * norm, hi = norm * (1.0 + 1e-13);
    for (int pass = 0; pass < 9; ++pass) {
      const double step = (hi - lo) * (1.0 / 65.0), x = __builtin_fma(step, (double)(lane + 1), lo);
      double p0 = 0.0, p1 = 1.0;
      unsigned before = 0;
      int below = 0;
#pragma unroll 1
      for (int i0 = 0; i0 < D; i0 += 32) {
        unsigned signs = 0;
#pragma unroll
        for (int j = 0; j < 32; ++j) {
          const double p2 = __builtin_fma(T[2 * (i0 + j)] - x, p1, -(T[2 * (i0 + j) + 1] * p0));
          p0 = p1;
          p1 = p2;
          signs = __builtin_amdgcn_alignbit(signs, (unsigned)(__builtin_bit_cast(unsigned long long, p2) >> 32), 31);
          if ((j & 7) == 7) {
            const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
            p0 = __builtin_amdgcn_ldexp(p0, ex);
            p1 = __builtin_amdgcn_ldexp(p1, ex);
          }
        }
        below += __popc(signs ^ ((signs >> 1) | (before << 31)));
        before = signs & 1;
      }
      const unsigned long long past = __ballot(below > idx);       // the first of these is above the eigenvalue
      const int cut = past ? __ffsll((unsigned long long)past) - 1 : 64;
      if (cut < 64) hi = __builtin_fma(step, (double)(cut + 1), lo);
      if (cut > 0) lo = __builtin_fma(step, (double)cut, lo);
    }
    if (lane == 0) lam_s[wave] = work[W::kLambda + idx] = 0.5 * (lo + hi);
  }
  __syncthreads();
  if (wave == 0) {
    const int chain = (lane >> 1) & 3, dir = lane & 1;             // of lanes 0 - 7
    const int who = lane >> 4, l16 = lane & 15;                    // eigenvalue that the 16 lanes look after otherwise
    const double lam = lam_s[who];
    double mu = lam + delta;
    for (int turn = 0; turn < 2; ++turn) {
      const double mine = __shfl(mu, 16 * chain);
      if (lane < 8) {
        double s = dir ? fact[1][D - 1].y - mine : -mine;
        Pair f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = fact[dir][j];
        for (int t0 = 0; t0 < D; t0 += 8) {
          Pair next[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) next[j] = fact[dir][min(t0 + 8, D - 8) + j];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const double den = f[j].x + s;
            const double q = fast_reciprocal(copysign(fmax(fabs(den), 1e-250), den));
            pivots[chain][dir][t0 + j] = Pair{s, q};
            s = __builtin_fma(f[j].y * s, q, -mine);
            f[j] = next[j];
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
      // the smallest pivot: magnitudes as bits, the lowest 7 of them the index
      unsigned key = 0xffffffffu;
#pragma unroll
      for (int x = 0; x < D / 16; ++x) {
        const int i = l16 + 16 * x;
        const Pair fwd = pivots[who][0][i], bwd = pivots[who][1][i];
        const double g = fwd.x + pivots[who][1][D - 1 - i].x + mu;
        key = min(key, ((unsigned)(__builtin_bit_cast(unsigned long long, g) >> 32) & 0x7fffff80u) | (unsigned)i);
        pivots[who][0][i].y = fwd.y * off[0][i];
        pivots[who][1][i].y = bwd.y * off[1][i];
      }
#pragma unroll
      for (int m = 1; m < 16; m *= 2) key = min(key, (unsigned)__shfl_xor((int)key, m));
      const int r = (int)(key & 127u);
      const double pivot = pivots[who][0][r].x + pivots[who][1][D - 1 - r].x + mu;
      const int my_r = __shfl(r, 16 * chain);
      __builtin_amdgcn_wave_barrier();
      if (lane < 8) {                                              // outwards from element r, where z = 1
        const int base = dir ? D - 2 - my_r : my_r - 1;
        const Pair* rat = pivots[chain][dir];
        double* to = zbuf[chain][dir] + 8;
        double v = 1.0, f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = rat[max(base - j, 0)].y;
        for (int t0 = base; t0 >= 0; t0 -= 8) {
          double next[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) next[j] = rat[max(t0 - 8 - j, 0)].y;
#pragma unroll
          for (int j = 0; j < 8; ++j) {                            // counted from the direction's end; below 0: room nobody reads
            v *= f[j];
            to[t0 - j] = v;
            f[j] = next[j];
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
      double zz = 0.0;
#pragma unroll
      for (int x = 0; x < D / 16; ++x) {
        const int i = l16 + 16 * x;
        const double z = i == r ? 1.0 : i < r ? zbuf[who][0][8 + i] : zbuf[who][1][8 + D - 1 - i];
        zz = __builtin_fma(z, z, zz);
      }
      zz = row_sum(zz);
      if (turn == 0) {
        mu += pivot * fast_reciprocal(zz);
      } else if (l16 == 0) {
        zz_s[who] = zz;
        r_s[who] = r;
        bad_s[who] = !(is_finite(zz) && fabs(mu - lam - delta) <= delta && fabs(pivot) <= 1e-13 * norm * sqrt(zz));
      }
    }
  }
  __syncthreads();
  if (wave < 4) {
    double z[RPL];
    if (lam_s[wave] > direction_limit * largest) {                 // wave-uniform
      double v[2][8][RPL];
      // The last two rows have no reflector (tau = 0).  X0 = 1: rows 64 and up, whose reflectors are zero in elements 0 - 63.
      fetch_rows(D - 1, v[0], std::integral_constant<int, RPL - 1>{});
      const int r = r_s[wave];
#pragma unroll
      for (int x = 0; x < RPL; ++x) {
        const int i = lane + 64 * x;
        z[x] = i == r ? 1.0 : i < r ? zbuf[wave][0][8 + i] : zbuf[wave][1][8 + D - 1 - i];
      }
      auto reflect = [&](auto first) __attribute__((always_inline)) {
        constexpr int X0 = decltype(first)::value;
        for (int k0 = 64 * X0 + 63; k0 >= 64 * X0; k0 -= 16) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const int k = k0 - 8 * c;
            if (X0 > 0 && k == 64 * X0 + 7) fetch_rows(k - 8, v[c ^ 1], std::integral_constant<int, X0 == 0 ? 0 : X0 - 1>{});
            else fetch_rows(max(k - 8, 7), v[c ^ 1], first);
#pragma unroll
            for (int j = 0; j < 8; j += 2) {     // two at a time: their sums do not wait for each other
              double (&a)[RPL] = v[c][j], (&b)[RPL] = v[c][j + 1];
              a[X0] = lane > k - j - 64 * X0 ? a[X0] : 0.0;
              b[X0] = lane > k - j - 1 - 64 * X0 ? b[X0] : 0.0;
              double sa = a[X0] * z[X0], sb = b[X0] * z[X0];
#pragma unroll
              for (int x = X0 + 1; x < RPL; ++x) {
                sa = __builtin_fma(a[x], z[x], sa);
                sb = __builtin_fma(b[x], z[x], sb);
              }
              const double both = half_sums(sa, sb);
              sa = lane_double(both, 0) * tau[k - j];
              sb = __builtin_fma(-sa, cross[(D - 1 - k + j) / 2], lane_double(both, 32)) * tau[k - j - 1];
#pragma unroll
              for (int x = X0; x < RPL; ++x) z[x] = __builtin_fma(-sb, b[x], __builtin_fma(-sa, a[x], z[x]));
            }
          }
        }
      };
      if constexpr (RPL == 2) reflect(std::integral_constant<int, 1>{});
      reflect(std::integral_constant<int, 0>{});
      const double scale = 1.0 / sqrt(zz_s[wave]);
#pragma unroll
      for (int x = 0; x < RPL; ++x) z[x] *= scale;
    } else {
#pragma unroll
      for (int x = 0; x < RPL; ++x) z[x] = 0.0;
    }
    if (lane == 0) reinterpret_cast<int*>(work + W::kBad)[idx] = bad_s[wave];
#pragma unroll
    for (int x = 0; x < RPL; ++x) out[lane + 64 * x][3 - wave] = (float)z[x];
  }
  __syncthreads();
  if (tid < D)                                                     // columns in descending order
    *reinterpret_cast<f32x4*>(U_out + ((size_t)h * D + tid) * D + D - 4 - 4 * blockIdx.x) = *reinterpret_cast<const f32x4*>(out[tid]);
}

}  // namespace seka
