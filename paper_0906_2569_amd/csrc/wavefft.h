// Transforms of length N = A B in two in-register steps on one wave: lane
// (t, b) takes the A-point DFT of x[b + B j] (j < A) of transform t, the
// partial results change lanes through LDS words of the wave's own, and lane
// (t, k) takes the B-point DFT over b, which leaves X[k + A m] (m < B):
//
//   X[k + A m] = sum_b W_B^(s b m) W_N^(s b k) sum_j x[b + B j] W_A^(s j k).
//
// The forward direction runs the same steps backwards, so that lane (t, k)
// holds the same points before and after a pointwise product.  A wave works
// on RB transforms at a time, R1 (R2) tasks of the A (B) side per lane.  The
// exchange needs no workgroup barrier (one wave's LDS operations complete in
// order) and moves real parts, then imaginary parts, through the same words:
// half the LDS, so more waves fit a CU.
#pragma once
#include "fft_reg.h"

// Range-checked view of n complex values: a load at index -1 (any index past
// the end) gives zero, a store there is dropped, by the buffer unit's own
// bounds check, so gathers and scatters through index maps need no branches.
struct BufView {
  __amdgpu_buffer_rsrc_t r;
  typedef unsigned int word __attribute__((ext_vector_type(4)));
  __device__ __forceinline__ BufView(const c128* p, size_t n)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<c128*>(p), 0, (int)(unsigned)(n * sizeof(c128)), 0x00027000)) {}
  __device__ __forceinline__ c128 load(int i) const {
    return __builtin_bit_cast(c128, __builtin_amdgcn_raw_buffer_load_b128(r, i * 16, 0, 0));
  }
  __device__ __forceinline__ void store(int i, c128 x) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(word, x), r, i * 16, 0, 0);
  }
};

namespace wavefft {

// N = A B with both factors within a lane's registers, A >= B
constexpr int split_a(int n) {
  switch (n) {
    case 24: return 6;
    case 25: return 5;
    case 27: return 9;
    case 30: return 6;
    case 32: return 8;
    case 36: return 6;
    case 40: return 8;
    case 45: return 9;
    case 48: return 8;
    case 50: return 10;
    case 54: return 9;
    case 60: return 10;
    case 64: return 8;
    case 72: return 9;
    case 75: return 15;
    case 80: return 10;
    case 81: return 9;
    case 90: return 10;
    case 96: return 12;
    case 100: return 10;
    case 108: return 12;
    case 120: return 12;
    case 125: return 25;
    case 128: return 16;
    case 135: return 15;
    default: return 0;
  }
}

constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }

// transforms per wave: the count that leaves the fewest lanes idle, weighing
// the two steps by their points, with at most 12 points per lane in each
// step (or one task of more)
constexpr int batch_of(int A, int B) {
  int best = 1;
  double score = -1.0;
  for (int rb = 1; rb <= 16; ++rb) {
    const int r1 = cdiv(rb * B, 64), r2 = cdiv(rb * A, 64);
    if ((r1 > 1 && r1 * A > 12) || (r2 > 1 && r2 * B > 12)) continue;
    const double s = 2.0 * rb * A * B / (64.0 * (r1 * A + r2 * B));
    if (s > score + 0.02) {
      score = s;
      best = rb;
    }
  }
  return best;
}

template <int N_>
struct Axis {
  static constexpr int N = N_, A = split_a(N_), B = N_ / split_a(N_);
  static_assert(A * B == N, "no two-step split of this length");
  static constexpr int RB = batch_of(A, B);                      // transforms per wave
  static constexpr int R1 = cdiv(RB * B, 64), R2 = cdiv(RB * A, 64);   // tasks per lane
  static constexpr int BP = B | 1;                               // odd stride: lanes k hit distinct banks
  static constexpr int words = RB * A * BP;                      // exchange words of a wave
  static constexpr int band = (N - 1) / 4;                       // largest |index| the sphere reaches
  // input j of lane b is index b + B j; the sphere's indices stay within
  // `band` of 0 (grids have N >= 4 max|m| + 1), so the middle j are zero for every lane
  static constexpr bool used(int j) { return B * j <= band || B * j + B - 1 >= N - band; }
};

// N-point DFT in registers.  Coprime factors take the prime-factor form (no
// twiddles between the steps); powers of one prime the mixed-radix form.
template <int N>
constexpr int coprime_factor() {
  if (N % 3 == 0 && N % 9 != 0 && N > 3) return 3;
  if (N % 5 == 0 && N % 25 != 0 && N > 5) return 5;
  if (N % 9 == 0 && N > 9) return 9;
  return 0;
}
constexpr int inv_mod(int a, int m) {
  for (int i = 1; i < m; ++i)
    if ((a * i) % m == 1) return i;
  return m == 1 ? 0 : -1;
}

template <int N, int F = coprime_factor<N>()>
struct WDft {
  static __device__ __forceinline__ void run(c128* x, double s) {
    constexpr int N1 = F, N2 = N / F;
    constexpr int e1 = N2 * inv_mod(N2 % N1, N1), e2 = N1 * inv_mod(N1 % N2, N2);   // 1 mod N1 (N2), 0 mod the other
    c128 a[N];
#pragma unroll
    for (int n2 = 0; n2 < N2; ++n2) {
      c128 t[N1];
#pragma unroll
      for (int n1 = 0; n1 < N1; ++n1) t[n1] = x[(N2 * n1 + N1 * n2) % N];
      WDft<N1>::run(t, s);
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) a[n2 * N1 + k1] = t[k1];
    }
#pragma unroll
    for (int k1 = 0; k1 < N1; ++k1) {
      c128 t[N2];
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) t[n2] = a[n2 * N1 + k1];
      WDft<N2>::run(t, s);
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) x[(e1 * k1 + e2 * k2) % N] = t[k2];
    }
  }
};
template <int N>
struct WDft<N, 0> {
  static __device__ __forceinline__ void run(c128* x, double s) { regfft::RDft<N, double>::run(x, s); }
};
template <>
struct WDft<8, 0> {
  static __device__ __forceinline__ void run(c128* x, double s) { Dft<8, double>::run(x, s); }
};
// 16 = 2 x 8: the odd half's twiddles are the only products besides Dft<8>'s
template <>
struct WDft<16, 0> {
  static __device__ __forceinline__ void run(c128* x, double s) {
    c128 e[8], o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      e[i] = x[2 * i];
      o[i] = x[2 * i + 1];
    }
    Dft<8, double>::run(e, s);
    Dft<8, double>::run(o, s);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      c128 v = o[k];
      if (k == 4) v = mul_is(v, s);
      else if (k != 0) v = cmul(v, c128{croot::RootTab<16>::v.c[k], s * croot::RootTab<16>::v.s[k]});
      x[k] = e[k] + v;
      x[k + 8] = e[k] - v;
    }
  }
};

// orders the wave's LDS accesses (in program order in hardware) for the compiler
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// How twiddle_powers takes its factors: w and w^4 (kTwo) or w, w^2 and w^4
// (kThree) held in registers over the passes of a caller's loop, the compiler
// kept from computing all powers ahead of it (2 A registers, spilled); or the
// three read again in each pass (kAgain).
enum Twiddles { kTwo, kThree, kAgain };

// x[k] *= w^k, k < A, w = tw[b] (conjugated where `conj`): two or three powers
// from the table, the others as products of those, so that none is far from the
// table.  (In one chain of w^2, A / 2 deep, the rounding of V psi was up to
// twice that of the kernels that read every power: 75^3 2.2, 120^3 1.44, 50^3
// 1.34 times; now 0.7 to 1.04 times on 25^3 to 120^3.)
template <int A, Twiddles HOW>
__device__ __forceinline__ void twiddle_powers(c128 (&x)[A], const c128* __restrict__ tw, int b, bool conj) {
  auto get = [&](int i) {
    c128 w = tw[i];
    if (conj) w.y = -w.y;
    return w;
  };
  if constexpr (HOW == kAgain) asm volatile("" : "+v"(b));
  c128 w1 = get(b), w4 = get(4 * b), w2{0.0, 0.0};
  if constexpr (HOW != kTwo) w2 = get(2 * b);
  if constexpr (HOW != kAgain) asm volatile("" : "+v"(w1.x), "+v"(w1.y), "+v"(w4.x), "+v"(w4.y));
  if constexpr (HOW == kThree) asm volatile("" : "+v"(w2.x), "+v"(w2.y));
  if constexpr (HOW == kTwo) w2 = cmul(w1, w1);
  const c128 w3 = cmul(w1, w2);
  x[1] = cmul(x[1], w1);
  x[2] = cmul(x[2], w2);
  x[3] = cmul(x[3], w3);
  c128 h = w4;   // w^(4 q)
#pragma unroll
  for (int k = 4; k < A; ++k) {
    if (k > 4 && k % 4 == 0) h = cmul(h, w4);
    const c128 w = k % 4 == 0 ? h : cmul(h, k % 4 == 1 ? w1 : k % 4 == 2 ? w2 : w3);
    x[k] = cmul(x[k], w);
  }
}

// A side -> B side: lane (t, b) holds x[.][k], lane (t, k) receives y[.][b]
template <class X>
__device__ __forceinline__ void exchange_ab(const c128 (&x)[X::R1][X::A], c128 (&y)[X::R2][X::B], double* W, int lane) {
#pragma unroll
  for (int part = 0; part < 2; ++part) {
#pragma unroll
    for (int r = 0; r < X::R1; ++r) {
      const int id = lane + 64 * r, t = id / X::B, b = id % X::B;
      if (id < X::RB * X::B) {
#pragma unroll
        for (int k = 0; k < X::A; ++k) W[(t * X::A + k) * X::BP + b] = part ? x[r][k].y : x[r][k].x;
      }
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < X::R2; ++r) {
      const int id = lane + 64 * r;   // = t A + k
      if (id < X::RB * X::A) {
#pragma unroll
        for (int b = 0; b < X::B; ++b) (part ? y[r][b].y : y[r][b].x) = W[id * X::BP + b];
      }
    }
    wave_sync();
  }
}

// B side -> A side: lane (t, k) holds y[.][b], lane (t, b) receives x[.][k]
template <class X>
__device__ __forceinline__ void exchange_ba(const c128 (&y)[X::R2][X::B], c128 (&x)[X::R1][X::A], double* W, int lane) {
#pragma unroll
  for (int part = 0; part < 2; ++part) {
#pragma unroll
    for (int r = 0; r < X::R2; ++r) {
      const int id = lane + 64 * r;
      if (id < X::RB * X::A) {
#pragma unroll
        for (int b = 0; b < X::B; ++b) W[id * X::BP + b] = part ? y[r][b].y : y[r][b].x;
      }
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < X::R1; ++r) {
      const int id = lane + 64 * r, t = id / X::B, b = id % X::B;
      if (id < X::RB * X::B) {
#pragma unroll
        for (int k = 0; k < X::A; ++k) (part ? x[r][k].y : x[r][k].x) = W[(t * X::A + k) * X::BP + b];
      }
    }
    wave_sync();
  }
}

}  // namespace wavefft
