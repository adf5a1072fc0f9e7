// Plane pass of H.psi on wave-local two-step transforms (wavefft.h): one
// workgroup per (PP consecutive z planes, band).
//
//   inverse y of the x columns   sticks (HBM) -> Y (LDS)
//   rows: inverse x, V(r), forward x            Y -> Y
//   forward y of the x columns   Y -> sticks (HBM)
//
// Y[PP][nxr][YS] holds the planes' x columns (odd stride YS: column and row
// accesses both spread over the banks); each wave exchanges within its own
// transforms through W, so the pass has two workgroup barriers in all.
//
// The pass is bound by its float64 vector instructions (about 24 per point
// and transform; 75% of the issue rate at 64^2, 55% at 72^2, where 12 waves a
// CU hide the LDS round trips).  Against the generic LDS kernel, which takes
// one LDS round trip and one workgroup barrier per radix, per pass over about
// 2.4e7 points: 50^2 391 -> 120 us, 90^2 814 -> 129, 108^2 734 -> 126,
// 120^2 795 -> 109; against the quad kernel 64^2 108 -> 69, 72^2 129 -> 107.
#pragma once
#include "plane_wave.h"
#include "wavefft.h"

namespace pw {

// Registers: up to 10 points a lane the kernel runs at three waves per SIMD
// (168 registers) and loads V(r) after the exchange; beyond, at two (256),
// with V(r) loaded ahead of it (60^2: 109 us against 115 at two waves and 283
// at four; 120^2: 109 us against 137 at three; spills cost more than the
// waves gain).  25 points do not fit either way (125^2 spills; the radix loop
// of the generic kernel is slower still, 900 against 570 us).
constexpr int plane_wave_points(int n1, int n2) {
  return wavefft::split_a(n1) > wavefft::split_a(n2) ? wavefft::split_a(n1) : wavefft::split_a(n2);
}
constexpr int plane_wave_threads(int n1, int n2) { return plane_wave_points(n1, n2) <= 10 ? 768 : 512; }

template <typename T, int N1, int N2>
__global__ void __launch_bounds__(plane_wave_threads(N1, N2))
k_plane_wave(SphereMap m, cpx<T>* __restrict__ sticks, const T* __restrict__ vr, const cpx<T>* __restrict__ tw1,
             const cpx<T>* __restrict__ tw2, int pp) {
  using X = wavefft::Axis<N1>;
  using Yx = wavefft::Axis<N2>;
  constexpr bool kVAhead = plane_wave_points(N1, N2) > 10 && plane_wave_points(N1, N2) < 25;
  constexpr int YS = N2 | 1;
  constexpr int WW = X::words > Yx::words ? X::words : Yx::words;
  extern __shared__ __align__(16) char smem_raw[];
  const int nxr = m.nxr, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  // each plane: its x columns, a column of zeros (read where the sphere has
  // no column) and one that takes what is written there
  const int zero = nxr * YS, plane = zero + 2 * YS;
  cpx<T>* Y = reinterpret_cast<cpx<T>*>(smem_raw);   // [pp][nxr + 2][YS]
  T* W = reinterpret_cast<T*>(Y + pp * plane) + wave * WW;
  const int z0 = blockIdx.y * pp, band = blockIdx.x;   // band fastest: workgroups in flight share V(r) planes
  const int np = min(pp, m.n3 - z0), ncol = np * nxr, nrow = np * N2;
  const BufView<T> st(sticks + ((size_t)band * m.n3 + z0) * m.ldst, (size_t)np * m.ldst);
  for (int i = threadIdx.x; i < np * YS; i += blockDim.x) Y[(i / YS) * plane + zero + i % YS] = cpx<T>{T(0), T(0)};

  // stick of (column c = pz nxr + x, y = b + B j), or -1
  auto stick_of = [&](int c, bool on, int b, int (&s)[Yx::A]) {
    const int pz = c / nxr;
    const int* cs = m.cy_st + (c - pz * nxr) * N2 + b;
#pragma unroll
    for (int j = 0; j < Yx::A; ++j)
      if (Yx::used(j)) {
        const int k = cs[Yx::B * j];
        s[j] = on && k >= 0 ? k + pz * m.ldst : -1;
      }
  };

  // inverse y
  for (int c0 = wave * Yx::RB; c0 < ncol; c0 += nw * Yx::RB) {
    cpx<T> x[Yx::R1][Yx::A], y[Yx::R2][Yx::B];
#pragma unroll
    for (int r = 0; r < Yx::R1; ++r) {
      const int id = lane + 64 * r, t = id / Yx::B, b = id % Yx::B, c = c0 + t;
      int s[Yx::A];
      stick_of(min(c, ncol - 1), id < Yx::RB * Yx::B && c < ncol, b, s);
#pragma unroll
      for (int j = 0; j < Yx::A; ++j) x[r][j] = Yx::used(j) ? st.load(s[j]) : cpx<T>{T(0), T(0)};
      wavefft::WDft<Yx::A, T>::run(x[r], T(1));
      wavefft::twiddle_powers<Yx::A, T>(x[r], tw2[b]);
    }
    wavefft::exchange_ab<Yx, T>(x, y, W, lane);
#pragma unroll
    for (int r = 0; r < Yx::R2; ++r) {
      const int id = lane + 64 * r, t = id / Yx::A, k = id % Yx::A, c = c0 + t;
      wavefft::WDft<Yx::B, T>::run(y[r], T(1));
      if (id < Yx::RB * Yx::A && c < ncol) {
        const int pz = c / nxr;
        cpx<T>* yc = Y + pz * plane + (c - pz * nxr) * YS + k;
#pragma unroll
        for (int q = 0; q < Yx::B; ++q) yc[Yx::A * q] = y[r][q];
      }
    }
  }
  __syncthreads();

  // rows (row pz N2 + r): inverse x, V(r), forward x
  int off[X::R1][X::A];   // offset in its plane of the x column at grid index b + B j
#pragma unroll
  for (int r = 0; r < X::R1; ++r)
#pragma unroll
    for (int j = 0; j < X::A; ++j)
      if (X::used(j)) {
        const int hx = m.i1_hx[(lane + 64 * r) % X::B + X::B * j];
        off[r][j] = hx >= 0 ? hx * YS : zero;
      }
  for (int q0 = wave * X::RB; q0 < nrow; q0 += nw * X::RB) {
    cpx<T> x[X::R1][X::A], y[X::R2][X::B];
    T v[X::R2][X::B];   // V(r), loaded ahead of its use
    auto load_v = [&]() {
#pragma unroll
      for (int r = 0; r < X::R2; ++r) {
        const int id = lane + 64 * r, row = min(q0 + id / X::A, nrow - 1);
        const T* vp = vr + ((size_t)z0 * N2 + row) * N1 + id % X::A;
#pragma unroll
        for (int q = 0; q < X::B; ++q) v[r][q] = vp[X::A * q];
      }
    };
    if constexpr (kVAhead) load_v();
#pragma unroll
    for (int r = 0; r < X::R1; ++r) {
      const int id = lane + 64 * r, b = id % X::B, row = min(q0 + id / X::B, nrow - 1);
      const int pz = row / N2;
      const cpx<T>* yp = Y + pz * plane + (row - pz * N2);
#pragma unroll
      for (int j = 0; j < X::A; ++j) x[r][j] = X::used(j) ? yp[off[r][j]] : cpx<T>{T(0), T(0)};
      wavefft::WDft<X::A, T>::run(x[r], T(1));
      wavefft::twiddle_powers<X::A, T>(x[r], tw1[b]);
    }
    wavefft::exchange_ab<X, T>(x, y, W, lane);
    if constexpr (!kVAhead) load_v();
#pragma unroll
    for (int r = 0; r < X::R2; ++r) {
      wavefft::WDft<X::B, T>::run(y[r], T(1));
#pragma unroll
      for (int q = 0; q < X::B; ++q) y[r][q] = y[r][q] * v[r][q];
      wavefft::WDft<X::B, T>::run(y[r], T(-1));
    }
    wavefft::exchange_ba<X, T>(y, x, W, lane);
#pragma unroll
    for (int r = 0; r < X::R1; ++r) {
      const int id = lane + 64 * r, b = id % X::B, row = q0 + id / X::B;
      cpx<T> w = tw1[b];
      w.y = -w.y;
      wavefft::twiddle_powers<X::A, T>(x[r], w);
      wavefft::WDft<X::A, T>::run(x[r], T(-1));
      if (id < X::RB * X::B && row < nrow) {
        const int pz = row / N2;
        cpx<T>* yp = Y + pz * plane + (row - pz * N2);
#pragma unroll
        for (int j = 0; j < X::A; ++j)
          if (X::used(j)) yp[off[r][j] == zero ? zero + YS : off[r][j]] = x[r][j];
      }
    }
  }
  __syncthreads();

  // forward y: only the stick positions are written
  for (int c0 = wave * Yx::RB; c0 < ncol; c0 += nw * Yx::RB) {
    cpx<T> x[Yx::R1][Yx::A], y[Yx::R2][Yx::B];
#pragma unroll
    for (int r = 0; r < Yx::R2; ++r) {
      const int id = lane + 64 * r, k = id % Yx::A, c = min(c0 + id / Yx::A, ncol - 1), pz = c / nxr;
      const cpx<T>* yc = Y + pz * plane + (c - pz * nxr) * YS + k;
#pragma unroll
      for (int q = 0; q < Yx::B; ++q) y[r][q] = yc[Yx::A * q];
      wavefft::WDft<Yx::B, T>::run(y[r], T(-1));
    }
    wavefft::exchange_ba<Yx, T>(y, x, W, lane);
#pragma unroll
    for (int r = 0; r < Yx::R1; ++r) {
      const int id = lane + 64 * r, b = id % Yx::B, c = c0 + id / Yx::B;
      cpx<T> w = tw2[b];
      w.y = -w.y;
      wavefft::twiddle_powers<Yx::A, T>(x[r], w);
      wavefft::WDft<Yx::A, T>::run(x[r], T(-1));
      int s[Yx::A];
      stick_of(min(c, ncol - 1), id < Yx::RB * Yx::B && c < ncol, b, s);
#pragma unroll
      for (int j = 0; j < Yx::A; ++j)
        if (Yx::used(j)) st.store(s[j], x[r][j]);
    }
  }
}

template <typename T, int N1, int N2>
PlaneWave<T> plane_wave_entry() {
  using X = wavefft::Axis<N1>;
  using Yx = wavefft::Axis<N2>;
  PlaneWave<T> e;
  e.fn = k_plane_wave<T, N1, N2>;
  e.ys = N2 | 1;
  e.wave_words = X::words > Yx::words ? X::words : Yx::words;
  e.rows = X::RB;
  e.cols = Yx::RB;
  e.max_waves = plane_wave_threads(N1, N2) / 64;
  return e;
}

}  // namespace pw
