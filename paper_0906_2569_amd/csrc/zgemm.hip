// Complex GEMMs on the matrix cores (v_mfma_f64_16x16x4f64 for float64,
// v_mfma_f32_16x16x4f32 for float32), used for the projector term of H.psi
// (<beta|psi>, then sum_j beta_j (D <beta|psi>)_j) and for the Davidson
// subspace products (phi^H H phi, phi^H phi, Ritz rotations).
//
// Complex products use three real MFMAs per 16x16x4 block (Gauss's product,
// as in the 3M complex GEMMs): t1 += Re A Re B, t2 += Im A Im B,
// t3 += (Re A + Im A)(Re B + Im B), and at the end Re C = t1 - t2,
// Im C = t3 - t1 - t2.  That is 6 M N K real flops on the matrix cores
// instead of the 8 of the four-product form.  The error bound of the
// imaginary part grows from about K u (|Re A||Im B| + |Im A||Re B|) to about
// K u (|Re A| + |Im A|)(|Re B| + |Im B|) (u the unit roundoff of the
// precision), a small constant factor on the same order.  Im A is negated
// once, at the LDS store, when A enters conjugated.  The four-product form
// is kept (kGauss = false) for comparison.
//
// Two shapes:
//   cn : C[m, n] = sum_k conj(A[k, m]) B[k, n]; A and B are stored as
//        K-contiguous columns (the plane-wave index runs fastest).  K is the
//        long plane-wave dimension, so K is split over workgroups and the
//        partial tiles are summed in a fixed order by a second kernel
//        (deterministic, no atomics).
//   nn : C[m, n] = alpha sum_k A[m, k] B[k, n] + beta C[m, n]; A is M-contiguous
//        (a block of plane-wave vectors), B K-contiguous (small coefficients).
#include <algorithm>

#include "plan.h"
#include "profile.h"

namespace {

template <typename T>
struct Mma;
template <>
struct Mma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 run(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 run(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Operand / result placement of the 16x16x4 MFMAs (64 lanes): lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16].  Result element q (0..3) of lane l
// is D[4 (l / 16) + q][l % 16] for the float32 instruction and
// D[4 q + l / 16][l % 16] for the float64 one (checked on gfx950).
template <typename T>
__device__ __forceinline__ int mrow(int lane, int q);
template <>
__device__ __forceinline__ int mrow<float>(int lane, int q) { return 4 * (lane >> 4) + q; }
template <>
__device__ __forceinline__ int mrow<double>(int lane, int q) { return 4 * q + (lane >> 4); }
__device__ __forceinline__ int mcol(int lane) { return lane & 15; }

// Both kernels are bound by the matrix cores; what they lose is the time in
// which no wave of a SIMD has products ready (a K slice takes a fetch, an LDS
// store and two barriers).  So the loads of a full slice carry no bounds
// checks (a check per load split the fetch into branches: 512-atom cell in
// float32 22.5 -> 20.5 ms calbec, 21.0 -> 19.2 ms add-back), calbec keeps two
// slices in flight, and the add-back runs at three waves per SIMD (168
// registers; float64, 200 atoms: 2649 us at two waves, 2477 at three).
// Accumulators must stay in VGPRs: with AGPR accumulators the float64 MFMA
// issues at 48 instead of 77 TFLOP/s.
constexpr int BN = 64, BK = 16, NT = 256;
// Output tile rows per workgroup (BM) and waves per SIMD the kernels are
// built for.  The calbec-shaped product (k_gemm_cn) in float32 takes 128 rows
// at two waves per SIMD (each wave a 64 x 32 block of 4 x 2 MFMA tiles: twice
// the products per operand byte loaded and per LDS read of a 64 x 64 tile;
// 22.4 against 23.7 ms at the 512-atom cell) unless 64 balance the CUs better
// (launch_cn), at three; the add-back (k_gemm_nn) 64 rows; float64 calbec 64
// rows at two waves (three accumulator sets and two slices in flight).  BM of
// k_gemm_cn also fixes the K split, and with it the rounding.
template <typename T, bool CN>
struct GT {
  static constexpr int BM = (sizeof(T) == 4 && CN) ? 128 : 64;
  static constexpr int waves = 3;      // of k_gemm_nn
};

// Workgroups go to the 8 XCDs round-robin in linear launch order.  Each XCD is
// given one contiguous range of a work order in which tile y (YFAST) or tile x
// runs fastest, then the other, then z: the workgroups that read the same
// operand strips then run on one XCD at about the same time and share its L2.
template <bool YFAST>
__device__ __forceinline__ void xcd_block(int& bx, int& by, int& bz) {
  const int gx = gridDim.x, gy = gridDim.y;
  const int T = gx * gy * gridDim.z;
  const int L = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int x = L & 7, s = L >> 3, per = T >> 3, rem = T & 7;
  // XCD x holds slots s < per + (x < rem): a bijection onto [0, T)
  const int w = x < rem ? x * (per + 1) + s : rem * (per + 1) + (x - rem) * per + s;
  if (YFAST) {
    by = w % gy;
    bx = (w / gy) % gx;
  } else {
    bx = w % gx;
    by = (w / gx) % gy;
  }
  bz = w / (gx * gy);
}

// One K slice of the operands in LDS, row k holding the slice's M (N) entries;
// real and imaginary parts apart, or (IL) together as 16-byte entries (float64
// k_gemm_nn: 2442 against 2477 us for the 200-atom add-back; in float32, and in
// k_gemm_cn with its transposing writes, slower: 24.4 against 20.5 ms for the
// 512-atom calbec, 3267 against 2839 us for the float64 200-atom one).
template <typename T, int BM, int BC, bool IL>
struct Tile {
  T ar[BK][BM + 1], ai[BK][BM + 1], br[BK][BC + 1], bi[BK][BC + 1];
  __device__ __forceinline__ void put_a(int k, int m, cpx<T> v) { ar[k][m] = v.x; ai[k][m] = v.y; }
  __device__ __forceinline__ void put_b(int k, int n, cpx<T> v) { br[k][n] = v.x; bi[k][n] = v.y; }
  __device__ __forceinline__ cpx<T> get_a(int k, int m) const { return cpx<T>{ar[k][m], ai[k][m]}; }
  __device__ __forceinline__ cpx<T> get_b(int k, int n) const { return cpx<T>{br[k][n], bi[k][n]}; }
};
template <typename T, int BM, int BC>
struct Tile<T, BM, BC, true> {
  cpx<T> a[BK][BM + 1], b[BK][BC + 1];
  __device__ __forceinline__ void put_a(int k, int m, cpx<T> v) { a[k][m] = v; }
  __device__ __forceinline__ void put_b(int k, int n, cpx<T> v) { b[k][n] = v; }
  __device__ __forceinline__ cpx<T> get_a(int k, int m) const { return a[k][m]; }
  __device__ __forceinline__ cpx<T> get_b(int k, int n) const { return b[k][n]; }
};

// The 4 waves' share of a BM x BC output tile: WN waves along N (two, or one
// for a 16-column tile), 4 / WN along M, each with IM x JN MFMA tiles of 16 x 16.
template <int BM, int BC>
struct Part {
  static constexpr int WN = BC == 16 ? 1 : 2, WM = 4 / WN, IM = BM / (16 * WM), JN = BC / (16 * WN);
  static __device__ __forceinline__ int row0(int wave) { return (wave % WM) * IM * 16; }
  static __device__ __forceinline__ int col0(int wave) { return (wave / WM) * JN * 16; }
};

// Accumulators of one wave's block of IM x JN MFMA tiles: a = t1,
// b = t2, c = t3 of the three-product form (a = Re C, b = Im C in the
// four-product form).
constexpr bool kGauss = true;

template <typename T, int IM, int JN>
struct CAcc {
  typedef typename Mma<T>::v4 v4;
  static constexpr bool k3 = kGauss;
  v4 a[IM][JN], b[IM][JN], c[IM][JN];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) a[i][j] = b[i][j] = c[i][j] = v4{0, 0, 0, 0};
  }
  __device__ __forceinline__ cpx<T> get(int i, int j, int q) const {
    if constexpr (k3) {
      const T t1 = a[i][j][q], t2 = b[i][j][q];
      return cpx<T>{t1 - t2, (c[i][j][q] - t1) - t2};
    } else {
      return cpx<T>{a[i][j][q], b[i][j][q]};
    }
  }
};

// One BK slice of a BM x BC tile product held in LDS
template <typename T, int BM, int BC, bool IL>
__device__ __forceinline__ void tile_mma(const Tile<T, BM, BC, IL>& t, CAcc<T, Part<BM, BC>::IM, Part<BM, BC>::JN>& acc,
                                         int wave, int lane) {
  constexpr int IM = Part<BM, BC>::IM, JN = Part<BM, BC>::JN;
  const int rm = Part<BM, BC>::row0(wave), cn = Part<BM, BC>::col0(wave);
  const int r = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int k4 = 0; k4 < BK; k4 += 4) {
    const int kk = k4 + kq;
    T ar[IM], ai[IM], br[JN], bi[JN];
#pragma unroll
    for (int i = 0; i < IM; ++i) {
      const cpx<T> v = t.get_a(kk, rm + i * 16 + r);
      ar[i] = v.x;
      ai[i] = v.y;
    }
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      const cpx<T> v = t.get_b(kk, cn + j * 16 + r);
      br[j] = v.x;
      bi[j] = v.y;
    }
    if constexpr (CAcc<T, IM, JN>::k3) {
      T sa[IM], sb[JN];
#pragma unroll
      for (int i = 0; i < IM; ++i) sa[i] = ar[i] + ai[i];
#pragma unroll
      for (int j = 0; j < JN; ++j) sb[j] = br[j] + bi[j];
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          acc.a[i][j] = Mma<T>::run(ar[i], br[j], acc.a[i][j]);
          acc.b[i][j] = Mma<T>::run(ai[i], bi[j], acc.b[i][j]);
          acc.c[i][j] = Mma<T>::run(sa[i], sb[j], acc.c[i][j]);
        }
    } else {
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          acc.a[i][j] = Mma<T>::run(ar[i], br[j], acc.a[i][j]);
          acc.a[i][j] = Mma<T>::run(-ai[i], bi[j], acc.a[i][j]);
          acc.b[i][j] = Mma<T>::run(ar[i], bi[j], acc.b[i][j]);
          acc.b[i][j] = Mma<T>::run(ai[i], br[j], acc.b[i][j]);
        }
    }
  }
}

// partial[z][n][m] = sum_{k in chunk z} conj(A[m*lda + k]) B[n*ldb + k]
// gridDim.z = 2 nsplit for two products of one launch: z >= nsplit takes B1
// and writes the partials after those of the first product
template <typename T, typename TA, typename TB, int BM, int BC = BN>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && BM <= 64 ? 3 : 2)))
k_gemm_cn(int M, int N, int K, int kchunk, int nsplit, const cpx<TA>* __restrict__ A, int lda,
          const cpx<TB>* __restrict__ B0, const cpx<TB>* __restrict__ B1, int ldb, cpx<T>* __restrict__ P) {
  constexpr int IM = Part<BM, BC>::IM, JN = Part<BM, BC>::JN;
  __shared__ Tile<T, BM, BC, false> t;
  int bx, by, bz;
  xcd_block<false>(bx, by, bz);   // the output tiles of one K chunk share an XCD
  const int m0 = bx * BM, n0 = by * BC;
  const int zs = bz % nsplit;
  const cpx<TB>* __restrict__ B = bz >= nsplit ? B1 : B0;
  const int kbeg = zs * kchunk, kend = min(K, kbeg + kchunk);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  CAcc<T, IM, JN> acc;
  acc.zero();

  // Two K slices are in flight in registers while one is multiplied out of
  // LDS: under this kernel's load a fetch takes longer than one slice's
  // products.  Rows past M and columns past N read the last one (their
  // products are not stored), so the loads of a full slice need no checks.
  constexpr int PA = BM * BK / NT, PB = BC * BK / NT;
  const int kk = threadIdx.x % BK;
  const int r0 = threadIdx.x / BK;
  const cpx<TA>* pa[PA];
  const cpx<TB>* pb[PB];
#pragma unroll
  for (int it = 0; it < PA; ++it) pa[it] = A + (size_t)min(m0 + r0 + it * (NT / BK), M - 1) * lda + kbeg + kk;
#pragma unroll
  for (int it = 0; it < PB; ++it) pb[it] = B + (size_t)min(n0 + r0 + it * (NT / BK), N - 1) * ldb + kbeg + kk;
  const int klen = max(kend - kbeg, 0), nfull = klen / BK, rem = klen % BK, nslice = nfull + (rem ? 1 : 0);
  cpx<TA> ra[2][PA];
  cpx<TB> rb[2][PB];
  auto load = [&](cpx<TA>(&xa)[PA], cpx<TB>(&xb)[PB], int sl) {
    if (sl < nfull) {
#pragma unroll
      for (int it = 0; it < PA; ++it) { xa[it] = *pa[it]; pa[it] += BK; }
#pragma unroll
      for (int it = 0; it < PB; ++it) { xb[it] = *pb[it]; pb[it] += BK; }
    } else {   // the last, partial slice: zeros past its end
      const bool in = kk < rem;
      const int back = in ? 0 : rem - 1 - kk;
#pragma unroll
      for (int it = 0; it < PA; ++it) {
        const cpx<TA> v = pa[it][back];
        xa[it] = in ? v : cpx<TA>{TA(0), TA(0)};
      }
#pragma unroll
      for (int it = 0; it < PB; ++it) {
        const cpx<TB> v = pb[it][back];
        xb[it] = in ? v : cpx<TB>{TB(0), TB(0)};
      }
    }
  };
  auto slice = [&](cpx<TA>(&xa)[PA], cpx<TB>(&xb)[PB], int sl) {
#pragma unroll
    for (int it = 0; it < PA; ++it) {
      const int mi = r0 + it * (NT / BK);
      t.put_a(kk, mi, cpx<T>{(T)xa[it].x, -(T)xa[it].y});  // conj(A)
    }
#pragma unroll
    for (int it = 0; it < PB; ++it) {
      const int ni = r0 + it * (NT / BK);
      t.put_b(kk, ni, cpx<T>{(T)xb[it].x, (T)xb[it].y});
    }
    __syncthreads();
    if (sl + 2 < nslice) load(xa, xb, sl + 2);
    tile_mma(t, acc, wave, lane);
    __syncthreads();
  };
  if (nslice > 0) load(ra[0], rb[0], 0);
  if (nslice > 1) load(ra[1], rb[1], 1);
  for (int sl = 0; sl < nslice; sl += 2) {
    slice(ra[0], rb[0], sl);
    if (sl + 1 < nslice) slice(ra[1], rb[1], sl + 1);
  }
  cpx<T>* out = P + (size_t)bz * M * N;
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + Part<BM, BC>::row0(wave) + i * 16 + mrow<T>(lane, q);
        const int n = n0 + Part<BM, BC>::col0(wave) + j * 16 + mcol(lane);
        if (m < M && n < N) out[(size_t)n * M + m] = acc.get(i, j, q);
      }
}

// C[n*ldc + m] = alpha sum_k A[k*lda + m] B[n*ldb + k] + beta C[n*ldc + m]
// The z index of the grid selects the product: (A0, C0) or (A1, C1), same B (two products of
// one launch fill the device better than two launches).
// SPLIT: the z index is instead the K chunk [z kchunk, (z + 1) kchunk) of the one
// product (A0), whose partial tile goes to P[z][n][m] unscaled, for k_reduce.
template <typename T, typename TA, typename TB, bool SPLIT = false, int BM = GT<T, false>::BM, int BC = BN>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(GT<T, false>::waves)))
k_gemm_nn(int M, int N, int K, double alpha, const cpx<TA>* __restrict__ A0, const cpx<TA>* __restrict__ A1,
          int lda, const cpx<TB>* __restrict__ B, int ldb, double beta, c128* __restrict__ C0,
          c128* __restrict__ C1, int ldc, const int* __restrict__ guard, int kchunk = 0,
          cpx<T>* __restrict__ P = nullptr, const double* __restrict__ kin = nullptr,
          const c128* __restrict__ X = nullptr, int ldx = 0) {
  if (guard != nullptr && *guard != 0) return;
  int bx, by, bz;
  xcd_block<true>(bx, by, bz);    // the column tiles of one row strip of A share an XCD
  const cpx<TA>* __restrict__ A = (!SPLIT && bz) ? A1 : A0;
  c128* __restrict__ C = (!SPLIT && bz) ? C1 : C0;
  const int kbeg = SPLIT ? bz * kchunk : 0;
  const int kend = SPLIT ? min(K, kbeg + kchunk) : K;
  constexpr int IM = Part<BM, BC>::IM, JN = Part<BM, BC>::JN;
  __shared__ Tile<T, BM, BC, sizeof(T) == 8> t;
  const int m0 = bx * BM, n0 = by * BC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  CAcc<T, IM, JN> acc;
  acc.zero();

  // the next K slice is loaded while the current one is multiplied; rows past
  // M and columns past N read the last one (not stored)
  constexpr int PA = BM * BK / NT, PB = BC * BK / NT;
  const int mi = threadIdx.x % BM, ka = threadIdx.x / BM;   // A: this thread's row, first k
  const int kk = threadIdx.x % BK, nb = threadIdx.x / BK;   // B: its k, first column
  const cpx<TA>* pa = A + (size_t)(kbeg + ka) * lda + min(m0 + mi, M - 1);
  const cpx<TB>* pb[PB];
#pragma unroll
  for (int it = 0; it < PB; ++it) pb[it] = B + (size_t)min(n0 + nb + it * (NT / BK), N - 1) * ldb + kbeg + kk;
  const size_t astep = (size_t)(NT / BM) * lda, aslice = (size_t)BK * lda;
  const int klen = max(kend - kbeg, 0), nfull = klen / BK, rem = klen % BK, nslice = nfull + (rem ? 1 : 0);
  cpx<TA> ra[PA];
  cpx<TB> rb[PB];
  auto load = [&](int sl) {
    if (sl < nfull) {
#pragma unroll
      for (int it = 0; it < PA; ++it) ra[it] = pa[it * astep];
      pa += aslice;
#pragma unroll
      for (int it = 0; it < PB; ++it) { rb[it] = *pb[it]; pb[it] += BK; }
    } else {   // the last, partial slice: zeros past its end
#pragma unroll
      for (int it = 0; it < PA; ++it) {
        const int k = ka + it * (NT / BM);
        const cpx<TA> v = *(pa + ((long)min(k, rem - 1) - ka) * lda);
        ra[it] = k < rem ? v : cpx<TA>{TA(0), TA(0)};
      }
#pragma unroll
      for (int it = 0; it < PB; ++it) {
        const cpx<TB> v = pb[it][min(kk, rem - 1) - kk];
        rb[it] = kk < rem ? v : cpx<TB>{TB(0), TB(0)};
      }
    }
  };
  if (nslice > 0) load(0);
  for (int sl = 0; sl < nslice; ++sl) {
#pragma unroll
    for (int it = 0; it < PA; ++it) {
      const int k = ka + it * (NT / BM);
      t.put_a(k, mi, cpx<T>{(T)ra[it].x, (T)ra[it].y});
    }
#pragma unroll
    for (int it = 0; it < PB; ++it) {
      t.put_b(kk, nb + it * (NT / BK), cpx<T>{(T)rb[it].x, (T)rb[it].y});
    }
    __syncthreads();
    if (sl + 1 < nslice) load(sl + 1);
    tile_mma(t, acc, wave, lane);
    __syncthreads();
  }
  if constexpr (SPLIT) {
    cpx<T>* out = P + (size_t)bz * M * N;
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = m0 + Part<BM, BC>::row0(wave) + i * 16 + mrow<T>(lane, q);
          const int n = n0 + Part<BM, BC>::col0(wave) + j * 16 + mcol(lane);
          if (m < M && n < N) out[(size_t)n * M + m] = acc.get(i, j, q);
        }
    return;
  }
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + Part<BM, BC>::row0(wave) + i * 16 + mrow<T>(lane, q);
        const int n = n0 + Part<BM, BC>::col0(wave) + j * 16 + mcol(lane);
        if (m < M && n < N) {
          c128* c = C + (size_t)n * ldc + m;
          const cpx<T> v = acc.get(i, j, q);
          double re = alpha * (double)v.x, im = alpha * (double)v.y;
          if (beta != 0.0) {
            const c128 old = *c;
            re += beta * old.x;
            im += beta * old.y;
          }
          if (kin != nullptr) {   // + diag(kin) X (kinetic term of H.psi)
            const c128 x = X[(size_t)n * ldx + m];
            re += kin[m] * x.x;
            im += kin[m] * x.y;
          }
          *c = c128{re, im};
        }
      }
}

// In k_reduce the split-K partials of one output element are summed by RZ
// thread groups:
// group y adds the partials z in [y nsplit / RZ, (y + 1) nsplit / RZ) in
// increasing z, then the RZ group sums are added in increasing y.  The order
// is fixed, so results are reproducible, and the groups keep RZ times more
// loads in flight than one thread per element would.
constexpr int RZ = 4;

// sum_z P[z * stride + off] for z0 <= z < z1 in increasing z; the loads of
// eight partials are issued before they are added
template <typename T>
__device__ __forceinline__ cpx<T> sum_partials(const cpx<T>* __restrict__ P, int z0, int z1, size_t stride,
                                               size_t off) {
  T re = 0, im = 0;
  int z = z0;
  for (; z + 8 <= z1; z += 8) {
    cpx<T> v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = P[(size_t)(z + u) * stride + off];
#pragma unroll
    for (int u = 0; u < 8; ++u) { re += v[u].x; im += v[u].y; }
  }
  for (; z < z1; ++z) {
    const cpx<T> v = P[(size_t)z * stride + off];
    re += v.x;
    im += v.y;
  }
  return cpx<T>{re, im};
}

template <typename T>
__device__ __forceinline__ cpx<T> add_groups(const cpx<T> (*s)[64], int x) {
  cpx<T> v = s[0][x];
#pragma unroll
  for (int y = 1; y < RZ; ++y) v = cpx<T>{v.x + s[y][x].x, v.y + s[y][x].y};
  return v;
}

// C[n*ldc + m] = alpha sum_z P[z][n][m] + beta Cin[n*ldcin + m]; block (64, RZ).
// Cin = C (in place) unless another matrix is given.  gridDim.y = 2 sums two
// products in one launch: blockIdx.y = 1 takes the partials after the first
// product's (nsplit M N of them) into C1.
template <typename T>
__global__ void __launch_bounds__(64 * RZ) k_reduce(int M, int N, int nsplit, const cpx<T>* __restrict__ P0,
                                                    c128* __restrict__ C0, c128* __restrict__ C1, int ldc,
                                                    double alpha, double beta, const c128* __restrict__ Cin = nullptr,
                                                    int ldcin = 0) {
  __shared__ cpx<T> s[RZ][64];
  const cpx<T>* __restrict__ P = P0 + (size_t)blockIdx.y * nsplit * M * N;
  c128* __restrict__ C = blockIdx.y ? C1 : C0;
  const size_t total = (size_t)M * N;
  const int x = threadIdx.x, y = threadIdx.y;
  const int z0 = y * nsplit / RZ, z1 = (y + 1) * nsplit / RZ;
  // the loop bound depends on the block only, so every thread reaches the barriers
  for (size_t base = (size_t)blockIdx.x * 64; base < total; base += (size_t)gridDim.x * 64) {
    const size_t idx = base + x;
    if (idx < total) s[y][x] = sum_partials(P, z0, z1, total, idx);
    __syncthreads();
    if (y == 0 && idx < total) {
      const cpx<T> sum = add_groups<T>(s, x);
      const int m = (int)(idx % M), n = (int)(idx / M);
      c128* c = C + (size_t)n * ldc + m;
      double r = alpha * (double)sum.x, i = alpha * (double)sum.y;
      if (beta != 0.0) {
        const c128 cin = Cin ? Cin[(size_t)n * ldcin + m] : *c;
        r += beta * cin.x;
        i += beta * cin.y;
      }
      *c = c128{r, i};
    }
    __syncthreads();
  }
}

// One workgroup per band n: becp[j] = sum_z P[z][n][j] into LDS, then
// out[n][j] = sum_{t < dlen_j} drow[j][t] becp[dstart_j + t].  It runs beside
// the transform passes, so its workgroups stay small (256 threads) to find
// room on CUs those passes occupy.
template <typename T>
__global__ void k_reduce_dapply(int M, int N, int nsplit, const cpx<T>* __restrict__ P,
                                const int* __restrict__ dstart, const int* __restrict__ dlen,
                                const cpx<T>* __restrict__ drow, int nhmax,
                                cpx<T>* __restrict__ out) {
  extern __shared__ __align__(16) char smem_raw[];
  cpx<T>* red = reinterpret_cast<cpx<T>*>(smem_raw);
  const int n = blockIdx.x;
  const size_t total = (size_t)M * N;
  for (int j = threadIdx.x; j < M; j += blockDim.x)
    red[j] = sum_partials(P, 0, nsplit, total, (size_t)n * M + j);
  __syncthreads();
  for (int j = threadIdx.x; j < M; j += blockDim.x) {
    const int j0 = dstart[j], nh = dlen[j];
    cpx<T> acc{T(0), T(0)};
    for (int t = 0; t < nh; ++t) acc = acc + cmul(drow[(size_t)j * nhmax + t], red[j0 + t]);
    out[(size_t)n * M + j] = acc;
  }
}

struct Split {
  int nsplit, kchunk;
};

// Output tile of a product with z planes of workgroups (K chunks or
// products).  A CU multiplies one 64 x 64 tile's K slice in the time of four
// 32 x 32 or 64 x 16 ones, and a product with fewer 64 x 64 tiles than CUs
// leaves the others idle (or multiplies padding, below 64 columns): the small
// tile is taken where the fullest CU's share is less even at a third more
// time per product (its operands are read twice as often).  The order of the
// sums over K does not depend on the tile: the results are the same.
// Measured, 64 x 64 -> small: 8 atoms, one band, H psi 32.5 -> 24.6 us; phi^H H phi
// of 64 and 16 columns, K = 949, 20.2 -> 8 us; 64 atoms, 128 bands, float32
// add-back 78.6 -> 60.2 us (379 tiles on 256 CUs).
enum TileForm { kTile64, kTile32, kTile16 };
TileForm tile_form(int M, int N, long z) {
  constexpr long cus = 256;
  const long wide = 4 * ceil_div((long)ceil_div(M, 64) * ceil_div(N, 64) * z, cus);
  const long t32 = ceil_div((long)ceil_div(M, 32) * ceil_div(N, 32) * z, cus);
  const long t16 = ceil_div((long)ceil_div(M, 64) * ceil_div(N, 16) * z, cus);
  if (4 * std::min(t32, t16) > 3 * wide) return kTile64;
  return t16 < t32 || N <= 16 ? kTile16 : kTile32;
}

// Launch of k_gemm_cn with ns K chunks in all (two products: twice the
// splits).  The chunks, hence the rounding, are the caller's; the tile height
// is free.  float32 takes 128 rows unless 64 fill the 256 CUs so much better
// that they win in spite of their lower intensity (6% at the 512-atom cell):
// the fullest CU's rows decide.  (200-atom calbec, 539 workgroups of 128 rows
// or 1001 of 64: 2.26 against 1.62 ms.)
template <typename T, typename TA, typename TB>
void launch_cn(int M, int N, int K, int kchunk, int nsplit, int ns, const cpx<TA>* A, int lda, const cpx<TB>* B0,
               const cpx<TB>* B1, int ldb, cpx<T>* P, hipStream_t s) {
  constexpr int cus = 256;
  const int gy = ceil_div(N, BN);
  auto go = [&](auto kernel, int bm, int bc) {
    kernel<<<dim3(ceil_div(M, bm), ceil_div(N, bc), ns), NT, 0, s>>>(M, N, K, kchunk, nsplit, A, lda, B0, B1, ldb, P);
  };
  const TileForm f = tile_form(M, N, ns);
  if (f == kTile32) return go(k_gemm_cn<T, TA, TB, 32, 32>, 32, 32);
  if (f == kTile16) return go(k_gemm_cn<T, TA, TB, 64, 16>, 64, 16);
  if constexpr (GT<T, true>::BM == 128) {
    const long wide = ceil_div((long)ceil_div(M, 128) * gy * ns, cus), half = ceil_div((long)ceil_div(M, 64) * gy * ns, cus);
    if (100 * 128 * wide <= 106 * 64 * half) return go(k_gemm_cn<T, TA, TB, 128>, 128, BN);
  }
  go(k_gemm_cn<T, TA, TB, 64>, 64, BN);
}

// Launch of k_gemm_nn (SPLIT: z K chunks of one product; else z products)
template <typename T, typename TA, typename TB, bool SPLIT = false>
void launch_nn(int z, int M, int N, int K, double alpha, const cpx<TA>* A0, const cpx<TA>* A1, int lda,
               const cpx<TB>* B, int ldb, double beta, c128* C0, c128* C1, int ldc, const int* guard, hipStream_t s,
               int kchunk = 0, cpx<T>* P = nullptr, const double* kin = nullptr, const c128* X = nullptr, int ldx = 0) {
  constexpr int BM = GT<T, false>::BM;
  auto go = [&](auto kernel, int bm, int bc) {
    kernel<<<dim3(ceil_div(M, bm), ceil_div(N, bc), z), NT, 0, s>>>(M, N, K, alpha, A0, A1, lda, B, ldb, beta, C0, C1,
                                                                    ldc, guard, kchunk, P, kin, X, ldx);
  };
  const TileForm f = tile_form(M, N, z);
  if (f == kTile32) return go(k_gemm_nn<T, TA, TB, SPLIT, 32, 32>, 32, 32);
  if (f == kTile16) return go(k_gemm_nn<T, TA, TB, SPLIT, 64, 16>, 64, 16);
  go(k_gemm_nn<T, TA, TB, SPLIT>, BM, BN);
}

Split choose_split(int M, int N, int K, int BM) {
  const int tiles = ceil_div(M, BM) * ceil_div(N, BN);
  const int target = 512;
  int nsplit = std::max(1, ceil_div(target, tiles));
  // A long K splits into at least one chunk per XCD even when the tiles alone
  // fill the device: the work order then gives each XCD its own K range, and
  // every operand element is read from memory once instead of by every tile
  // row or column (calbec of the 512-atom cell read its operands 9 times)
  if (nsplit < 8 && K >= 8 * 256 * BK) nsplit = 8;
  nsplit = std::min(nsplit, std::max(1, ceil_div(K, 4 * BK)));
  int kchunk = ceil_div(ceil_div(K, nsplit), BK) * BK;
  kchunk = std::max(kchunk, BK);
  nsplit = std::max(1, ceil_div(K, kchunk));
  return Split{nsplit, kchunk};
}

}  // namespace

size_t pw::splitk_part_bytes(int M, int N, int K, int elem_bytes) {
  // Upper bound over every M' <= M, N' <= N: nsplit <= 512/tiles + 1, so
  // nsplit M' N' <= 512 BM BN + M N; a long K adds the 8-chunk minimum.
  // Complex64 partials come from the 128-row tiles, complex128 ones from the
  // 64-row tiles; a complex128-sized bound covers the complex64 partials of
  // the same product (512 x 128 x 64 x 8 B = 512 x 64 x 64 x 16 B).
  const size_t mn = (size_t)std::max(M, 1) * std::max(N, 1);
  const size_t bm = elem_bytes <= 8 ? (size_t)GT<float, true>::BM : (size_t)GT<double, true>::BM;
  size_t e = (size_t)512 * bm * BN + mn;
  if (K >= 8 * 256 * BK) e = std::max(e, 8 * mn);
  return e * elem_bytes + 256;
}

template <typename T, typename TA, typename TB>
pw_status pw::zgemm_cn(int M, int N, int K, const cpx<TA>* A, int lda, const cpx<TB>* B, int ldb,
                       c128* C, int ldc, void* part, size_t part_bytes, hipStream_t s, double alpha,
                       double beta, const c128* Cin, int ldcin) {
  if (M <= 0 || N <= 0) return PW_OK;
  const Split sp = choose_split(M, N, K, GT<T, true>::BM);
  const size_t need = (size_t)sp.nsplit * M * N * sizeof(cpx<T>);
  PW_CHECK(need <= part_bytes, PW_ENOMEM, "split-K workspace too small");
  cpx<T>* P = static_cast<cpx<T>*>(part);
  if (K <= 0) {
    // a sum over no partials is zero: C = beta C
    k_reduce<T><<<std::min(4096, ceil_div((size_t)M * N, 64)), dim3(64, RZ), 0, s>>>(M, N, 0, P, C, C, ldc,
                                                                                   alpha, beta, Cin, ldcin);
    PW_HIP(hipGetLastError());
    return PW_OK;
  }
  {
    pw::ProfScope ps(pw::PK_GEMM_CN, s, 8.0 * M * N * K);
    launch_cn<T>(M, N, K, sp.kchunk, sp.nsplit, sp.nsplit, A, lda, B, B, ldb, P, s);
  }
  {
    pw::ProfScope ps(pw::PK_GEMM_RED, s, (double)sp.nsplit * M * N * sizeof(cpx<T>) + 16.0 * M * N);
    k_reduce<T><<<std::min(4096, ceil_div((size_t)M * N, 64)), dim3(64, RZ), 0, s>>>(M, N, sp.nsplit, P, C, C,
                                                                                   ldc, alpha, beta, Cin, ldcin);
  }
  PW_HIP(hipGetLastError());
  return PW_OK;
}

pw_status pw::zgemm_cn_pair(int M, int N, int K, const c128* A, int lda, const c128* B0, const c128* B1,
                            int ldb, c128* C0, c128* C1, int ldc, void* part, size_t part_bytes, hipStream_t s) {
  if (M <= 0 || N <= 0) return PW_OK;
  Split sp = choose_split(M, N, K, GT<double, true>::BM);
  // half the splits per product: the two products together fill the device
  const int ns = std::max(1, sp.nsplit / 2);
  const int kchunk = std::max(BK, ceil_div(ceil_div(K, ns), BK) * BK);
  const int nsplit = std::max(1, ceil_div(K, kchunk));
  const size_t need = 2 * (size_t)nsplit * M * N * sizeof(c128);
  if (K <= 0 || need > part_bytes) {
    PW_TRY((zgemm_cn<double, double, double>(M, N, K, A, lda, B0, ldb, C0, ldc, part, part_bytes, s)));
    return zgemm_cn<double, double, double>(M, N, K, A, lda, B1, ldb, C1, ldc, part, part_bytes, s);
  }
  c128* P = static_cast<c128*>(part);
  {
    pw::ProfScope ps(pw::PK_GEMM_CN, s, 16.0 * M * N * K);
    launch_cn<double>(M, N, K, kchunk, nsplit, 2 * nsplit, A, lda, B0, B1, ldb, P, s);
  }
  {
    pw::ProfScope ps(pw::PK_GEMM_RED, s, 2.0 * ((double)nsplit * M * N * sizeof(c128) + 16.0 * M * N));
    const int g = std::min(4096, ceil_div((size_t)M * N, 64));
    k_reduce<double><<<dim3(g, 2), dim3(64, RZ), 0, s>>>(M, N, nsplit, P, C0, C1, ldc, 1.0, 0.0);
  }
  PW_HIP(hipGetLastError());
  return PW_OK;
}

template <typename T>
pw_status pw::calbec_d(pw_plan p, int nb, const c128* psi, int ldpsi, cpx<T>* out, hipStream_t s,
                       const cpx<T>* rows) {
  const int M = p->nbeta, N = nb, K = p->npw;
  const Split sp = choose_split(M, N, K, GT<T, true>::BM);
  const size_t need = (size_t)sp.nsplit * M * N * sizeof(cpx<T>);
  PW_CHECK(need <= p->part_bytes, PW_ENOMEM, "split-K workspace too small");
  cpx<T>* P = static_cast<cpx<T>*>(p->part);
  const cpx<T>* beta = sizeof(T) == 8 ? (const cpx<T>*)p->beta64 : (const cpx<T>*)p->beta32;
  const cpx<T>* drow = rows ? rows : (sizeof(T) == 8 ? (const cpx<T>*)p->drow64 : (const cpx<T>*)p->drow32);
  {
    pw::ProfScope ps(pw::PK_CALBEC, s, 8.0 * M * N * K);
    launch_cn<T>(M, N, K, sp.kchunk, sp.nsplit, sp.nsplit, beta, p->ldb, psi, psi, ldpsi, P, s);
  }
  {
    pw::ProfScope ps(pw::PK_CALBEC_RED, s, (double)sp.nsplit * M * N * sizeof(cpx<T>) + (double)M * N * sizeof(cpx<T>));
    k_reduce_dapply<T><<<N, 256, sizeof(cpx<T>) * M, s>>>(M, N, sp.nsplit, P, p->dstart, p->dlen,
                                                        drow, p->nhmax, out);
  }
  PW_HIP(hipGetLastError());
  return PW_OK;
}

template <typename T, typename TA, typename TB>
pw_status pw::zgemm_nn(int M, int N, int K, double alpha, const cpx<TA>* A, int lda,
                       const cpx<TB>* B, int ldb, double beta, c128* C, int ldc, hipStream_t s,
                       const int* guard, const double* kin, const c128* X, int ldx) {
  if (M <= 0 || N <= 0) return PW_OK;
  pw::ProfScope ps(pw::PK_GEMM_NN, s, 8.0 * M * N * K);
  launch_nn<T>(1, M, N, K, alpha, A, A, lda, B, ldb, beta, C, C, ldc, guard, s, 0, (cpx<T>*)nullptr, kin, X, ldx);
  PW_HIP(hipGetLastError());
  return PW_OK;
}

pw_status pw::zgemm_nn_sk(int M, int N, int K, double alpha, const c128* A, int lda, const c128* B, int ldb,
                          double beta, c128* C, int ldc, void* part, size_t part_bytes, hipStream_t s) {
  if (M <= 0 || N <= 0) return PW_OK;
  const int tiles = ceil_div(M, GT<double, false>::BM) * ceil_div(N, BN);
  // chunks of at least two K slices, up to about 512 workgroups in all
  const int ns = std::min(ceil_div(512, tiles), ceil_div(K, 2 * BK));
  const int kchunk = std::max(BK, ceil_div(ceil_div(K, std::max(ns, 1)), BK) * BK);
  const int nsplit = ceil_div(K, kchunk);
  const size_t need = (size_t)nsplit * M * N * sizeof(c128);
  if (tiles >= 128 || nsplit < 2 || need > part_bytes)
    return zgemm_nn<double, double, double>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s);
  c128* P = static_cast<c128*>(part);
  {
    pw::ProfScope ps(pw::PK_GEMM_NN, s, 8.0 * M * N * K);
    launch_nn<double, double, double, true>(nsplit, M, N, K, 1.0, A, A, lda, B, ldb, 0.0, nullptr, nullptr, ldc,
                                            nullptr, s, kchunk, P);
  }
  {
    pw::ProfScope ps(pw::PK_GEMM_RED, s, (double)nsplit * M * N * sizeof(c128) + 16.0 * M * N);
    k_reduce<double><<<std::min(4096, ceil_div((size_t)M * N, 64)), dim3(64, RZ), 0, s>>>(M, N, nsplit, P, C, C,
                                                                                         ldc, alpha, beta);
  }
  PW_HIP(hipGetLastError());
  return PW_OK;
}

template <typename T>
pw_status pw::zgemm_nn_pair(int M, int N, int K, const c128* A0, const c128* A1, int lda, const c128* B,
                            int ldb, c128* C0, c128* C1, int ldc, hipStream_t s, const int* guard) {
  if (M <= 0 || N <= 0) return PW_OK;
  pw::ProfScope ps(pw::PK_GEMM_NN, s, 16.0 * M * N * K);
  launch_nn<T>(2, M, N, K, 1.0, A0, A1, lda, B, ldb, 0.0, C0, C1, ldc, guard, s);
  PW_HIP(hipGetLastError());
  return PW_OK;
}

template pw_status pw::zgemm_nn_pair<double>(int, int, int, const c128*, const c128*, int, const c128*, int, c128*,
                                             c128*, int, hipStream_t, const int*);
template pw_status pw::zgemm_nn_pair<float>(int, int, int, const c128*, const c128*, int, const c128*, int, c128*,
                                            c128*, int, hipStream_t, const int*);
template pw_status pw::zgemm_cn<double, double, double>(int, int, int, const c128*, int, const c128*,
                                                        int, c128*, int, void*, size_t, hipStream_t,
                                                        double, double, const c128*, int);
template pw_status pw::zgemm_cn<float, double, double>(int, int, int, const c128*, int, const c128*,
                                                       int, c128*, int, void*, size_t, hipStream_t,
                                                       double, double, const c128*, int);
template pw_status pw::calbec_d<double>(pw_plan, int, const c128*, int, c128*, hipStream_t, const c128*);
template pw_status pw::calbec_d<float>(pw_plan, int, const c128*, int, c64*, hipStream_t, const c64*);
template pw_status pw::zgemm_nn<double, double, double>(int, int, int, double, const c128*, int,
                                                        const c128*, int, double, c128*, int,
                                                        hipStream_t, const int*, const double*, const c128*,
                                                        int);
template pw_status pw::zgemm_nn<float, float, float>(int, int, int, double, const c64*, int,
                                                     const c64*, int, double, c128*, int,
                                                     hipStream_t, const int*, const double*, const c128*,
                                                     int);
template pw_status pw::zgemm_nn<float, double, double>(int, int, int, double, const c128*, int,
                                                       const c128*, int, double, c128*, int,
                                                        hipStream_t, const int*, const double*, const c128*,
                                                        int);
