// z passes of H.psi on two-step transforms (n3 = A B, see wavefft.h) for the
// lengths the quad and 16-lane forms do not cover: a workgroup holds 16
// sticks, thread (b, s) takes the A-point step of stick s, thread (k, s) the
// B-point step, and the two meet in LDS [position][stick] (the sticks of a
// position are contiguous: no bank conflicts, and stick rows of 256 bytes in
// HBM).  The passes move the sphere's scattered 16-byte entries and are bound
// by memory; the two steps keep every thread's points in registers, where the
// radix loop of the generic kernels went through LDS once per radix (both
// passes of 2.4e7 points: n3 = 120 144 -> 70 us, 90 105 -> 48, 50 66 -> 47).
// 125 = 25 x 5 stays on the generic kernels (174 us against 204).
#include "wavefft.h"
#include "zpass.h"

namespace {

constexpr int ZS = 16;   // sticks per workgroup

template <int N>
constexpr int zthreads() { return ZS * (wavefft::Axis<N>::A > wavefft::Axis<N>::B ? wavefft::Axis<N>::A : wavefft::Axis<N>::B); }

// inverse transform of the columns x[] that `load(s, z)` gives, into out
template <int N, class Load>
__device__ __forceinline__ void zinv_tile(const SphereMap& m, int s0, c128* __restrict__ out,
                                          const c128* __restrict__ tw, c128* L, Load load) {
  using X = wavefft::Axis<N>;
  const int sl = threadIdx.x % ZS, u = threadIdx.x / ZS, s = s0 + sl;
  if (u < X::B) {
    c128 x[X::A];
#pragma unroll
    for (int j = 0; j < X::A; ++j) x[j] = (X::used(j) && s < m.nst) ? load(s, u + X::B * j) : c128{0.0, 0.0};
    wavefft::WDft<X::A>::run(x, 1.0);
    wavefft::twiddle_powers<X::A, wavefft::kAgain>(x, tw, u, false);
#pragma unroll
    for (int k = 0; k < X::A; ++k) L[(k * X::B + u) * ZS + sl] = x[k];
  }
  __syncthreads();
  if (u < X::A && s < m.nst) {
    c128 y[X::B];
#pragma unroll
    for (int b = 0; b < X::B; ++b) y[b] = L[(u * X::B + b) * ZS + sl];
    wavefft::WDft<X::B>::run(y, 1.0);
#pragma unroll
    for (int q = 0; q < X::B; ++q) out[(size_t)(u + X::A * q) * m.ldst + s] = y[q];
  }
}

// forward transform of the columns of `in`; store(s, z, v) takes the positions the sphere can reach
template <int N, class Store>
__device__ __forceinline__ void zfwd_tile(const SphereMap& m, int s0, const c128* in, const c128* __restrict__ tw,
                                          c128* L, Store store) {
  using X = wavefft::Axis<N>;
  const int sl = threadIdx.x % ZS, u = threadIdx.x / ZS, s = s0 + sl;
  if (u < X::A) {
    c128 y[X::B];
#pragma unroll
    for (int q = 0; q < X::B; ++q) y[q] = s < m.nst ? in[(size_t)(u + X::A * q) * m.ldst + s] : c128{0.0, 0.0};
    wavefft::WDft<X::B>::run(y, -1.0);
#pragma unroll
    for (int b = 0; b < X::B; ++b) L[(u * X::B + b) * ZS + sl] = y[b];
  }
  __syncthreads();
  if (u < X::B && s < m.nst) {
    c128 x[X::A];
#pragma unroll
    for (int k = 0; k < X::A; ++k) x[k] = L[(k * X::B + u) * ZS + sl];
    wavefft::twiddle_powers<X::A, wavefft::kAgain>(x, tw, u, true);
    wavefft::WDft<X::A>::run(x, -1.0);
#pragma unroll
    for (int j = 0; j < X::A; ++j)
      if (X::used(j)) store(s, u + X::B * j, x[j]);
  }
}

template <int N>
__global__ void __launch_bounds__(zthreads<N>())
k_zinv_wave(SphereMap m, const c128* __restrict__ psi, int ldpsi, c128* __restrict__ sticks,
            const c128* __restrict__ tw, int gz, int nb) {
  __shared__ c128 L[N * ZS];
  int chunk, band;
  if (!pw::z_tile(gz, nb, chunk, band)) return;
  const c128* pb = psi + (size_t)band * ldpsi;
  zinv_tile<N>(m, chunk * ZS, sticks + (size_t)band * N * m.ldst, tw, L, [&](int s, int z) {
    const int g = m.zidx[(size_t)z * m.nst + s];
    return g >= 0 ? pb[g] : c128{0.0, 0.0};
  });
}

template <int N>
__global__ void __launch_bounds__(zthreads<N>())
k_zfwd_wave(SphereMap m, const c128* __restrict__ sticks, const c128* __restrict__ psi, int ldpsi,
            c128* __restrict__ hpsi, int ldhpsi, const c128* __restrict__ tw, double inv_n, int accumulate, int gz,
            int nb) {
  __shared__ c128 L[N * ZS];
  int chunk, band;
  if (!pw::z_tile(gz, nb, chunk, band)) return;
  const c128* pb = psi + (size_t)band * ldpsi;
  c128* hb = hpsi + (size_t)band * ldhpsi;
  zfwd_tile<N>(m, chunk * ZS, sticks + (size_t)band * N * m.ldst, tw, L, [&](int s, int z, c128 v) {
    const int g = m.zidx[(size_t)z * m.nst + s];
    if (g < 0) return;
    c128 r = c128{v.x * inv_n, v.y * inv_n};
    if (!(accumulate & 2)) {   // kinetic term (not yet in hpsi)
      const c128 p = pb[g];
      const double t = m.kin[g];
      r = c128{r.x + t * p.x, r.y + t * p.y};
    }
    if (accumulate & 1) {   // the projector and kinetic terms are already in hpsi
      const c128 o = hb[g];
      r = c128{r.x + o.x, r.y + o.y};
    }
    hb[g] = r;
  });
}

template <int N>
__global__ void __launch_bounds__(zthreads<N>())
k_zinv_wave_g(SphereMap m, const c128* __restrict__ psi, int ldpsi, c128* __restrict__ sticks,
              const c128* __restrict__ tw, int gz, int npair, int nbands) {
  __shared__ c128 L[N * ZS];
  int chunk, pair;
  if (!pw::z_tile(gz, npair, chunk, pair)) return;
  const c128* pa = psi + (size_t)(2 * pair) * ldpsi;
  const c128* pb = 2 * pair + 1 < nbands ? pa + ldpsi : nullptr;
  zinv_tile<N>(m, chunk * ZS, sticks + (size_t)pair * N * m.ldst, tw, L, [&](int s, int z) {
    const int enc = m.zidx[(size_t)z * m.nst + s];
    return enc >= 0 ? pw::gamma_pack(pa, pb, enc) : c128{0.0, 0.0};
  });
}

// in place: only the positions the gather reads are written back
template <int N>
__global__ void __launch_bounds__(zthreads<N>())
k_zfwd_wave_g(SphereMap m, c128* __restrict__ sticks, const c128* __restrict__ tw, int gz, int npair) {
  __shared__ c128 L[N * ZS];
  int chunk, pair;
  if (!pw::z_tile(gz, npair, chunk, pair)) return;
  c128* io = sticks + (size_t)pair * N * m.ldst;
  zfwd_tile<N>(m, chunk * ZS, io, tw, L, [&](int s, int z, c128 v) { io[(size_t)z * m.ldst + s] = v; });
}

template <int N>
pw::ZFns<double> entry() {
  pw::ZFns<double> f;
  f.inv = k_zinv_wave<N>;
  f.fwd = k_zfwd_wave<N>;
  f.inv_g = k_zinv_wave_g<N>;
  f.fwd_g = k_zfwd_wave_g<N>;
  f.sticks = ZS;
  f.threads = zthreads<N>();
  return f;
}

}  // namespace

pw::ZFns<double> pw::zwave_f64(int n3) {
  switch (n3) {
    case 24: return entry<24>();
    case 25: return entry<25>();
    case 27: return entry<27>();
    case 30: return entry<30>();
    case 45: return entry<45>();
    case 50: return entry<50>();
    case 54: return entry<54>();
    case 75: return entry<75>();
    case 81: return entry<81>();
    case 90: return entry<90>();
    case 100: return entry<100>();
    case 108: return entry<108>();
    case 120: return entry<120>();
    case 135: return entry<135>();
    default: return {};
  }
}
