// Real GEMMs on the matrix cores (v_mfma_f64_16x16x4f64 / v_mfma_f32_16x16x4f32,
// one MFMA per 16x16x4 block) for the Gamma-point real-wavefunction path.
//
// At Gamma a real function f(r) has f(-G) = conj(f(G)), so only the half
// sphere is stored.  Viewing a half-sphere column of complex values as a
// real column of twice the length (re, im interleaved), the full-sphere inner
// product of two such functions is
//     <a|b> = sum_{G in full} conj(a(G)) b(G) = 2 sum_k a_k b_k - a(0) b(0),
// k over the interleaved reals and G = 0 at half-sphere index 0 (a(0), b(0)
// real).  So the projector and subspace products become real products with
// K = 2 npw_half and a rank-one correction, and combinations with real
// coefficients (Ritz rotations, the projector add-back) real products with
// M = 2 npw_half: a quarter of the complex products' flops.
//
//   tn : C[m, n] = alpha (2 sum_k A[m*lda + k] B[n*ldb + k] - w0 A[m*lda] B[n*ldb]) + beta C
//        (split K, partials summed in a fixed order: deterministic)
//   nn : C[n*ldc + m] = alpha sum_k A[k*lda + m] B[n*ldb + k] + beta C[n*ldc + m]
#include <algorithm>
#include <climits>

#include "plan.h"
#include "profile.h"

namespace {

template <typename T>
struct RMma;
template <>
struct RMma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 run(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct RMma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 run(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// result element q of lane l: row as below, column l % 16 (same placement as
// the complex kernels)
template <typename T>
__device__ __forceinline__ int rrow(int lane, int q);
template <>
__device__ __forceinline__ int rrow<float>(int lane, int q) { return 4 * (lane >> 4) + q; }
template <>
__device__ __forceinline__ int rrow<double>(int lane, int q) { return 4 * q + (lane >> 4); }

constexpr int BM = 64, BN = 64, BK = 32, NT = 256;

// One K slice in LDS, row k holding its M (N) entries.  Reads take 16
// neighbouring entries of four rows, writes one entry of 32 rows (tn, and B of
// nn).  float64: rows k and k + 1 lie half the banks apart, and within a row
// entry c sits at c ^ s(k), s spreading the rows that share a bank offset over
// 16 entries.  float32: rows of odd stride; the same spreading took 20 KB
// in place of 17 a workgroup and held up the transforms beside it (mixed Gamma
// products of 140 atoms, 7 bands 178 against 169 us, 4 bands 163 against 160;
// 200 atoms, 6 bands 230 against 221).
template <typename T>
struct RTile {
  static constexpr bool spread = sizeof(T) == 8;
  static constexpr int pad = spread ? 16 : 1;
  T a[BK][BM + pad], b[BK][BN + pad];
  static __device__ __forceinline__ int at(int k, int c) { return spread ? c ^ ((k >> 1) & 15) : c; }
};

// workgroups of one output tile range share an XCD (round-robin launch order)
__device__ __forceinline__ void xcd_map(int& bx, int& by, int& bz, bool yfast) {
  const int gx = gridDim.x, gy = gridDim.y;
  const int T = gx * gy * gridDim.z;
  const int L = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int x = L & 7, s = L >> 3, per = T >> 3, rem = T & 7;
  const int w = x < rem ? x * (per + 1) + s : rem * (per + 1) + (x - rem) * per + s;
  if (yfast) {
    by = w % gy;
    bx = (w / gy) % gx;
  } else {
    bx = w % gx;
    by = (w / gx) % gy;
  }
  bz = w / (gx * gy);
}

template <typename T>
__device__ __forceinline__ void rtile_mma(const RTile<T>& t, typename RMma<T>::v4 (&c)[2][2], int wm, int wn,
                                          int lane) {
  const int r = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int k4 = 0; k4 < BK; k4 += 4) {
    const int kk = k4 + kq, rs = RTile<T>::at(kk, r);   // at() stays within aligned groups of 16
    T a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = t.a[kk][wm * 32 + i * 16 + rs];
      b[i] = t.b[kk][wn * 32 + i * 16 + rs];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) c[i][j] = RMma<T>::run(a[i], b[j], c[i][j]);
  }
}

// P[z][n][m] = sum_{k in chunk z} A[m*lda + k] B[n*ldb + k].  Off holds the
// offset of a row within its tile, up to 63 strides (dgemm_tn picks it).
template <typename T, typename TA, typename TB, typename Off>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3)))
k_dgemm_tn(int M, int N, int K, int kchunk, const TA* __restrict__ A, long lda, const TB* __restrict__ B, long ldb,
           T* __restrict__ P) {
  __shared__ RTile<T> t;
  typedef typename RMma<T>::v4 v4;
  int bx, by, bz;
  xcd_map(bx, by, bz, false);
  const int m0 = bx * BM, n0 = by * BN;
  const int kbeg = bz * kchunk, kend = min(K, kbeg + kchunk);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  v4 c[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) c[i][j] = v4{0, 0, 0, 0};
  // the next K slice is loaded while the current one is multiplied; rows past
  // M and columns past N read the last one (not stored), so full slices need no
  // checks
  constexpr int PER = BM * BK / NT, RP = NT / BK;
  const int kk = threadIdx.x % BK, r0 = threadIdx.x / BK;
  const TA* a0 = A + (size_t)m0 * lda + kbeg;
  const TB* b0 = B + (size_t)n0 * ldb + kbeg;
  Off oa[PER], ob[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    oa[it] = (Off)min(r0 + it * RP, M - 1 - m0) * (Off)lda + kk;
    ob[it] = (Off)min(r0 + it * RP, N - 1 - n0) * (Off)ldb + kk;
  }
  const int klen = max(kend - kbeg, 0), nfull = klen / BK, rem = klen % BK, nslice = nfull + (rem ? 1 : 0);
  TA ra[PER];
  TB rb[PER];
  auto load = [&](int sl) {
    if (sl < nfull) {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        ra[it] = a0[oa[it]];
        rb[it] = b0[ob[it]];
      }
      a0 += BK;
      b0 += BK;
    } else {   // the last, partial slice: zeros past its end
      const bool in = kk < rem;
      const int back = in ? 0 : kk - (rem - 1);
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const TA va = a0[oa[it] - back];
        const TB vb = b0[ob[it] - back];
        ra[it] = in ? va : TA(0);
        rb[it] = in ? vb : TB(0);
      }
    }
  };
  if (nslice > 0) load(0);
  for (int sl = 0; sl < nslice; ++sl) {
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      t.a[kk][RTile<T>::at(kk, r0 + it * RP)] = (T)ra[it];
      t.b[kk][RTile<T>::at(kk, r0 + it * RP)] = (T)rb[it];
    }
    __syncthreads();
    if (sl + 1 < nslice) load(sl + 1);
    rtile_mma<T>(t, c, wm, wn, lane);
    __syncthreads();
  }
  T* out = P + (size_t)bz * M * N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + wm * 32 + i * 16 + rrow<T>(lane, q);
        const int n = n0 + wn * 32 + j * 16 + (lane & 15);
        if (m < M && n < N) out[(size_t)n * M + m] = c[i][j][q];
      }
}

// C[n*ldc + m] = alpha (2 sum_z P[z][n][m] - w0 A[m*lda] B[n*ldb]) + beta C, in
// increasing z; C real (cplx = 0) or the real part of a complex matrix whose
// imaginary part is set to 0 (cplx = 1)
template <typename T, typename TA, typename TB>
__global__ void k_dreduce(int M, int N, int nsplit, const T* __restrict__ P, const TA* __restrict__ A, long lda,
                          const TB* __restrict__ B, long ldb, double w0, double alpha, double beta,
                          double* __restrict__ C, int ldc, int cplx) {
  const size_t total = (size_t)M * N;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < total;
       idx += (size_t)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int z = 0; z < nsplit; ++z) s += (double)P[(size_t)z * total + idx];
    const int m = (int)(idx % M), n = (int)(idx / M);
    double v = 2.0 * s - w0 * (double)A[(size_t)m * lda] * (double)B[(size_t)n * ldb];
    v *= alpha;
    if (cplx) {
      double* c = C + 2 * ((size_t)n * ldc + m);
      if (beta != 0.0) v += beta * c[0];
      c[0] = v;
      c[1] = 0.0;
    } else {
      double* c = C + (size_t)n * ldc + m;
      if (beta != 0.0) v += beta * *c;
      *c = v;
    }
  }
}

// C[n*ldc + m] = alpha sum_k A[k*lda + m] B[n*ldb + k] + beta C[n*ldc + m]  (C double)
template <typename T, typename TA, typename TB>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3)))
k_dgemm_nn(int M, int N, int K, double alpha, const TA* __restrict__ A, long lda, const TB* __restrict__ B,
           long ldb, double beta, double* __restrict__ C, long ldc, const int* __restrict__ guard) {
  if (guard != nullptr && *guard != 0) return;
  __shared__ RTile<T> t;
  typedef typename RMma<T>::v4 v4;
  int bx, by, bz;
  xcd_map(bx, by, bz, true);
  const int m0 = bx * BM, n0 = by * BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  v4 c[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) c[i][j] = v4{0, 0, 0, 0};
  constexpr int PER = BM * BK / NT, AP = NT / BM, RP = NT / BK;
  const int mi = threadIdx.x % BM, ka = threadIdx.x / BM;   // A: this thread's row, first k
  const int kk = threadIdx.x % BK, r0 = threadIdx.x / BK;   // B: its k, first column
  const TA* pa = A + (size_t)ka * lda + min(m0 + mi, M - 1);
  const TB* pb[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) pb[it] = B + (size_t)min(n0 + r0 + it * RP, N - 1) * ldb + kk;
  const size_t astep = (size_t)AP * lda, aslice = (size_t)BK * lda;
  const int nfull = max(K, 0) / BK, rem = max(K, 0) % BK, nslice = nfull + (rem ? 1 : 0);
  TA ra[PER];
  TB rb[PER];
  auto load = [&](int sl) {
    if (sl < nfull) {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        ra[it] = pa[it * astep];
        rb[it] = *pb[it];
        pb[it] += BK;
      }
      pa += aslice;
    } else {   // the last, partial slice: zeros past its end
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const int k = ka + it * AP;
        const TA va = *(pa + ((long)min(k, rem - 1) - ka) * lda);
        const TB vb = pb[it][min(kk, rem - 1) - kk];
        ra[it] = k < rem ? va : TA(0);
        rb[it] = kk < rem ? vb : TB(0);
      }
    }
  };
  if (nslice > 0) load(0);
  for (int sl = 0; sl < nslice; ++sl) {
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int k = ka + it * AP;
      t.a[k][RTile<T>::at(k, mi)] = (T)ra[it];
      t.b[kk][RTile<T>::at(kk, r0 + it * RP)] = (T)rb[it];
    }
    __syncthreads();
    if (sl + 1 < nslice) load(sl + 1);
    rtile_mma<T>(t, c, wm, wn, lane);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + wm * 32 + i * 16 + rrow<T>(lane, q);
        const int n = n0 + wn * 32 + j * 16 + (lane & 15);
        if (m < M && n < N) {
          double* p = C + (size_t)n * ldc + m;
          double v = alpha * (double)c[i][j][q];
          if (beta != 0.0) v += beta * *p;
          *p = v;
        }
      }
}

int dsplit(int M, int N, int K, int& kchunk) {
  const int tiles = ceil_div(M, BM) * ceil_div(N, BN);
  int ns = std::max(1, ceil_div(512, tiles));
  if (ns < 8 && K >= 8 * 256 * BK) ns = 8;   // one K range per XCD (see the complex products)
  ns = std::min(ns, std::max(1, ceil_div(K, 4 * BK)));
  kchunk = std::max(BK, ceil_div(ceil_div(K, ns), BK) * BK);
  return std::max(1, ceil_div(K, kchunk));
}

}  // namespace

size_t pw::dgemm_part_bytes(int M, int N) {
  const size_t mn = (size_t)std::max(M, 1) * std::max(N, 1);
  return std::max((size_t)512 * BM * BN + mn, 8 * mn) * sizeof(double) + 256;
}

template <typename T, typename TA, typename TB>
pw_status pw::dgemm_tn(int M, int N, int K, const TA* A, long lda, const TB* B, long ldb, double w0, double alpha,
                       double beta, double* C, int ldc, bool cplx_out, void* part, size_t part_bytes,
                       hipStream_t s, int prof) {
  if (M <= 0 || N <= 0) return PW_OK;
  int kchunk = 0;
  const int ns = dsplit(M, N, K, kchunk);
  PW_CHECK((size_t)ns * M * N * sizeof(T) <= part_bytes, PW_ENOMEM, "split-K workspace too small");
  T* P = static_cast<T*>(part);
  {
    pw::ProfScope ps(prof >= 0 ? prof : pw::PK_GEMM_CN, s, 2.0 * M * N * (double)K);
    auto go = [&](auto kernel) {
      kernel<<<dim3(ceil_div(M, BM), ceil_div(N, BN), ns), NT, 0, s>>>(M, N, K, kchunk, A, lda, B, ldb, P);
    };
    // 32-bit row offsets (16 registers fewer) while a tile's rows stay within
    // them.  A block of bands may have any stride its caller gave it.
    if ((BM - 1) * std::max(lda, ldb) + BK <= (long)UINT_MAX) go(k_dgemm_tn<T, TA, TB, unsigned>);
    else go(k_dgemm_tn<T, TA, TB, size_t>);
  }
  const int g = std::min(4096, ceil_div((size_t)M * N, 256));
  k_dreduce<T, TA, TB><<<g, 256, 0, s>>>(M, N, ns, P, A, lda, B, ldb, w0, alpha, beta, C, ldc, cplx_out ? 1 : 0);
  PW_HIP(hipGetLastError());
  return PW_OK;
}

template <typename T, typename TA, typename TB>
pw_status pw::dgemm_nn(int M, int N, int K, double alpha, const TA* A, long lda, const TB* B, long ldb, double beta,
                       double* C, long ldc, hipStream_t s, const int* guard, int prof) {
  if (M <= 0 || N <= 0) return PW_OK;
  pw::ProfScope ps(prof >= 0 ? prof : pw::PK_GEMM_NN, s, 2.0 * M * N * (double)K);
  k_dgemm_nn<T, TA, TB><<<dim3(ceil_div(M, BM), ceil_div(N, BN), 1), NT, 0, s>>>(M, N, K, alpha, A, lda, B, ldb,
                                                                                beta, C, ldc, guard);
  PW_HIP(hipGetLastError());
  return PW_OK;
}

template pw_status pw::dgemm_tn<double, double, double>(int, int, int, const double*, long, const double*, long,
                                                        double, double, double, double*, int, bool, void*, size_t,
                                                        hipStream_t, int);
template pw_status pw::dgemm_tn<float, float, double>(int, int, int, const float*, long, const double*, long, double,
                                                      double, double, double*, int, bool, void*, size_t, hipStream_t,
                                                      int);
template pw_status pw::dgemm_nn<double, double, double>(int, int, int, double, const double*, long, const double*,
                                                        long, double, double*, long, hipStream_t, const int*, int);
template pw_status pw::dgemm_nn<float, float, float>(int, int, int, double, const float*, long, const float*, long,
                                                     double, double*, long, hipStream_t, const int*, int);
// float32 arithmetic on float64 operands (subspace products of the float32 stage)
template pw_status pw::dgemm_tn<float, double, double>(int, int, int, const double*, long, const double*, long,
                                                       double, double, double, double*, int, bool, void*, size_t,
                                                       hipStream_t, int);
template pw_status pw::dgemm_nn<float, double, double>(int, int, int, double, const double*, long, const double*,
                                                       long, double, double*, long, hipStream_t, const int*, int);
