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

// Twiddle factors of an axis.  Held is faster (120^2 Gamma block 7.20 against
// 7.33 ms) except in steps whose kernels have no registers left: of 10 points
// at three waves per SIMD (50^2 block 112 us held, 100 read again) and of 25
// (125^2 778 and 704 us).  Three held cost up to 9% in the same way (81^2 199
// and 218 us), and are taken on the lengths where two round more than the table
// kernels (V psi on 25^3 1.15 against 1.04 times them, 64^3 1.05 and 1.00, 27^3
// 1.05 and 0.98).
template <class X>
constexpr wavefft::Twiddles twiddles_of() {
  if (X::A == 10 || X::A >= 25) return wavefft::kAgain;
  return X::N == 25 || X::N == 27 || X::N == 64 ? wavefft::kThree : wavefft::kTwo;
}

// The planes of one workgroup in LDS: each plane's x columns [nxr][ys], a column of
// zeros (read where the sphere has no column) and one that takes what is
// written there.
struct PlaneLds {
  int nxr, ys, zero, plane;
  __device__ __forceinline__ PlaneLds(int nxr_, int ys_) : nxr(nxr_), ys(ys_), zero(nxr_ * ys_), plane((nxr_ + 2) * ys_) {}
};

__device__ __forceinline__ void clear_zero_columns(c128* Y, const PlaneLds& L, int np) {
  for (int i = threadIdx.x; i < np * L.ys; i += blockDim.x)
    Y[(i / L.ys) * L.plane + L.zero + i % L.ys] = c128{0.0, 0.0};
}

// sticks of (column c = pz nxr + x, y = b + B j), or -1
template <class Yx>
__device__ __forceinline__ void sticks_of(const SphereMap& m, int c, bool on, int b, int (&s)[Yx::A]) {
  const int pz = c / m.nxr;
  const int* cs = m.cy_st + (c - pz * m.nxr) * Yx::N + b;
#pragma unroll
  for (int j = 0; j < Yx::A; ++j)
    if (Yx::used(j)) {
      const int k = cs[Yx::B * j];
      s[j] = on && k >= 0 ? k + pz * m.ldst : -1;
    }
}

// inverse y transforms of all ncol columns: sticks -> Y
template <class Yx>
__device__ __forceinline__ void inverse_y(const SphereMap& m, const BufView& st, c128* Y, double* W, const PlaneLds& L,
                                          int ncol, const c128* __restrict__ tw2, int lane, int wave, int nw) {
  for (int c0 = wave * Yx::RB; c0 < ncol; c0 += nw * Yx::RB) {
    c128 x[Yx::R1][Yx::A], y[Yx::R2][Yx::B];
#pragma unroll
    for (int r = 0; r < Yx::R1; ++r) {
      const int id = lane + 64 * r, t = id / Yx::B, b = id % Yx::B, c = c0 + t;
      int s[Yx::A];
      sticks_of<Yx>(m, min(c, ncol - 1), id < Yx::RB * Yx::B && c < ncol, b, s);
#pragma unroll
      for (int j = 0; j < Yx::A; ++j) x[r][j] = Yx::used(j) ? st.load(s[j]) : c128{0.0, 0.0};
      wavefft::WDft<Yx::A>::run(x[r], 1.0);
      wavefft::twiddle_powers<Yx::A, twiddles_of<Yx>()>(x[r], tw2, b, false);
    }
    wavefft::exchange_ab<Yx>(x, y, W, lane);
#pragma unroll
    for (int r = 0; r < Yx::R2; ++r) {
      const int id = lane + 64 * r, t = id / Yx::A, k = id % Yx::A, c = c0 + t;
      wavefft::WDft<Yx::B>::run(y[r], 1.0);
      if (id < Yx::RB * Yx::A && c < ncol) {
        const int pz = c / L.nxr;
        c128* yc = Y + pz * L.plane + (c - pz * L.nxr) * L.ys + k;
#pragma unroll
        for (int q = 0; q < Yx::B; ++q) yc[Yx::A * q] = y[r][q];
      }
    }
  }
}

// offset in its plane of the x column at grid index b + B j of this lane
template <class X>
__device__ __forceinline__ void column_offsets(const SphereMap& m, const PlaneLds& L, int lane, int (&off)[X::R1][X::A]) {
#pragma unroll
  for (int r = 0; r < X::R1; ++r)
#pragma unroll
    for (int j = 0; j < X::A; ++j)
      if (X::used(j)) {
        const int hx = m.i1_hx[(lane + 64 * r) % X::B + X::B * j];
        off[r][j] = hx >= 0 ? hx * L.ys : L.zero;
      }
}

// A step of the inverse x transforms of rows q0 .. q0 + RB - 1 (row pz n2 + r), up to the exchange
template <class X, int N2>
__device__ __forceinline__ void inverse_x_first(const c128* Y, const PlaneLds& L, int q0, int nrow,
                                                const int (&off)[X::R1][X::A], const c128* __restrict__ tw1, int lane,
                                                c128 (&x)[X::R1][X::A]) {
#pragma unroll
  for (int r = 0; r < X::R1; ++r) {
    const int id = lane + 64 * r, b = id % X::B, row = min(q0 + id / X::B, nrow - 1);
    const int pz = row / N2;
    const c128* yp = Y + pz * L.plane + (row - pz * N2);
#pragma unroll
    for (int j = 0; j < X::A; ++j) x[r][j] = X::used(j) ? yp[off[r][j]] : c128{0.0, 0.0};
    wavefft::WDft<X::A>::run(x[r], 1.0);
    wavefft::twiddle_powers<X::A, twiddles_of<X>()>(x[r], tw1, b, false);
  }
}

template <int N1, int N2>
__global__ void __launch_bounds__(plane_wave_threads(N1, N2))
k_plane_wave(SphereMap m, c128* __restrict__ sticks, const double* __restrict__ vr, const c128* __restrict__ tw1,
             const c128* __restrict__ tw2, int pp) {
  using X = wavefft::Axis<N1>;
  using Yx = wavefft::Axis<N2>;
  constexpr bool kVAhead = plane_wave_points(N1, N2) > 10 && plane_wave_points(N1, N2) < 25;
  constexpr int WW = X::words > Yx::words ? X::words : Yx::words;
  extern __shared__ __align__(16) char smem_raw[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const PlaneLds L(m.nxr, N2 | 1);
  c128* Y = reinterpret_cast<c128*>(smem_raw);   // [pp][nxr + 2][ys]
  double* W = reinterpret_cast<double*>(Y + pp * L.plane) + wave * WW;
  const int z0 = blockIdx.y * pp, band = blockIdx.x;   // band fastest: workgroups in flight share V(r) planes
  const int np = min(pp, m.n3 - z0), ncol = np * m.nxr, nrow = np * N2;
  const BufView st(sticks + ((size_t)band * m.n3 + z0) * m.ldst, (size_t)np * m.ldst);
  clear_zero_columns(Y, L, np);
  inverse_y<Yx>(m, st, Y, W, L, ncol, tw2, lane, wave, nw);
  __syncthreads();

  // rows: inverse x, V(r), forward x
  int off[X::R1][X::A];
  column_offsets<X>(m, L, lane, off);
  for (int q0 = wave * X::RB; q0 < nrow; q0 += nw * X::RB) {
    c128 x[X::R1][X::A], y[X::R2][X::B];
    double v[X::R2][X::B];   // V(r)
    auto load_v = [&]() {
#pragma unroll
      for (int r = 0; r < X::R2; ++r) {
        const int id = lane + 64 * r, row = min(q0 + id / X::A, nrow - 1);
        const double* vp = vr + ((size_t)z0 * N2 + row) * N1 + id % X::A;
#pragma unroll
        for (int q = 0; q < X::B; ++q) v[r][q] = vp[X::A * q];
      }
    };
    if constexpr (kVAhead) load_v();
    inverse_x_first<X, N2>(Y, L, q0, nrow, off, tw1, lane, x);
    wavefft::exchange_ab<X>(x, y, W, lane);
    if constexpr (!kVAhead) load_v();
#pragma unroll
    for (int r = 0; r < X::R2; ++r) {
      wavefft::WDft<X::B>::run(y[r], 1.0);
#pragma unroll
      for (int q = 0; q < X::B; ++q) y[r][q] = y[r][q] * v[r][q];
      wavefft::WDft<X::B>::run(y[r], -1.0);
    }
    wavefft::exchange_ba<X>(y, x, W, lane);
#pragma unroll
    for (int r = 0; r < X::R1; ++r) {
      const int id = lane + 64 * r, b = id % X::B, row = q0 + id / X::B;
      wavefft::twiddle_powers<X::A, twiddles_of<X>()>(x[r], tw1, b, true);
      wavefft::WDft<X::A>::run(x[r], -1.0);
      if (id < X::RB * X::B && row < nrow) {
        const int pz = row / N2;
        c128* yp = Y + pz * L.plane + (row - pz * N2);
#pragma unroll
        for (int j = 0; j < X::A; ++j)
          if (X::used(j)) yp[off[r][j] == L.zero ? L.zero + L.ys : off[r][j]] = x[r][j];
      }
    }
  }
  __syncthreads();

  // forward y: only the stick positions are written
  for (int c0 = wave * Yx::RB; c0 < ncol; c0 += nw * Yx::RB) {
    c128 x[Yx::R1][Yx::A], y[Yx::R2][Yx::B];
#pragma unroll
    for (int r = 0; r < Yx::R2; ++r) {
      const int id = lane + 64 * r, k = id % Yx::A, c = min(c0 + id / Yx::A, ncol - 1), pz = c / L.nxr;
      const c128* yc = Y + pz * L.plane + (c - pz * L.nxr) * L.ys + k;
#pragma unroll
      for (int q = 0; q < Yx::B; ++q) y[r][q] = yc[Yx::A * q];
      wavefft::WDft<Yx::B>::run(y[r], -1.0);
    }
    wavefft::exchange_ba<Yx>(y, x, W, lane);
#pragma unroll
    for (int r = 0; r < Yx::R1; ++r) {
      const int id = lane + 64 * r, b = id % Yx::B, c = c0 + id / Yx::B;
      wavefft::twiddle_powers<Yx::A, twiddles_of<Yx>()>(x[r], tw2, b, true);
      wavefft::WDft<Yx::A>::run(x[r], -1.0);
      int s[Yx::A];
      sticks_of<Yx>(m, min(c, ncol - 1), id < Yx::RB * Yx::B && c < ncol, b, s);
#pragma unroll
      for (int j = 0; j < Yx::A; ++j)
        if (Yx::used(j)) st.store(s[j], x[r][j]);
    }
  }
}

// the density kernel's accumulators take the third wave's registers beyond 8 points a lane
constexpr int density_threads(int n1, int n2) { return plane_wave_points(n1, n2) <= 8 ? 768 : 512; }

// Rounds of rows per wave of the density kernel and its waves: all row
// batches of a plane at once, accumulators in registers (at most 24 float64
// a lane, 40 from 100 rows on), with as many waves on a CU as LDS and registers
// allow.
struct DensityShape {
  int rounds, waves;
};
template <int N1, int N2>
constexpr DensityShape density_shape() {
  using X = wavefft::Axis<N1>;
  using Yx = wavefft::Axis<N2>;
  constexpr int WW = X::words > Yx::words ? X::words : Yx::words;
  const int batches = wavefft::cdiv(N2, X::RB), maxw = density_threads(N1, N2) / 64;
  DensityShape best{0, 0};
  double score = -1.0;
  for (int rr = 1; rr <= 8 && (rr == 1 || rr * X::R2 * X::B <= (N2 >= 100 ? 40 : 24)); ++rr) {
    const int nw = wavefft::cdiv(batches, rr);
    const int lds = 16 * (2 * X::band + 3) * (N2 | 1) + 8 * nw * WW;
    if (nw > maxw || lds > 160 * 1024) continue;
    const int fit = 160 * 1024 / lds, wgs = fit < maxw / nw ? fit : maxw / nw;
    const double s = (double)(wgs < 1 ? 1 : wgs) * nw * batches / (nw * rr);
    if (s > score * 1.02) {
      score = s;
      best = DensityShape{rr, nw};
    }
  }
  return best;
}

// part[group][z][y][x] = sum over the group's transforms t of w_t |psi_t(r)|^2,
// or at Gamma (transform t holds psi_2t(r) + i psi_2t+1(r), both real)
// w_2t Re^2 + w_2t+1 Im^2: one workgroup per (z plane, group), its transforms
// in order, the sums in registers -- the plane never goes to memory.
template <int N1, int N2, int RR>
__global__ void __launch_bounds__(density_threads(N1, N2))
k_density_wave(SphereMap m, const c128* __restrict__ sticks, int nt, int per, int nbands, int gamma,
               const double* __restrict__ w, const c128* __restrict__ tw1, const c128* __restrict__ tw2,
               double* __restrict__ part) {
  using X = wavefft::Axis<N1>;
  using Yx = wavefft::Axis<N2>;
  constexpr int WW = X::words > Yx::words ? X::words : Yx::words;
  extern __shared__ __align__(16) char smem_raw[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const PlaneLds L(m.nxr, N2 | 1);
  c128* Y = reinterpret_cast<c128*>(smem_raw);
  double* W = reinterpret_cast<double*>(Y + L.plane) + wave * WW;
  const int z = blockIdx.x, t0 = blockIdx.y * per, t1 = min(nt, t0 + per);
  clear_zero_columns(Y, L, 1);
  int off[X::R1][X::A];
  column_offsets<X>(m, L, lane, off);
  double acc[RR][X::R2][X::B];
#pragma unroll
  for (int i = 0; i < RR; ++i)
#pragma unroll
    for (int r = 0; r < X::R2; ++r)
#pragma unroll
      for (int q = 0; q < X::B; ++q) acc[i][r][q] = 0.0;
  for (int t = t0; t < t1; ++t) {
    const BufView st(sticks + ((size_t)t * m.n3 + z) * m.ldst, (size_t)m.ldst);
    const double wa = gamma ? w[2 * t] : w[t];
    const double wi = gamma ? (2 * t + 1 < nbands ? w[2 * t + 1] : 0.0) : wa;
    __syncthreads();   // the rows of the transform before have been read
    inverse_y<Yx>(m, st, Y, W, L, m.nxr, tw2, lane, wave, nw);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      const int q0 = (wave + i * nw) * X::RB;
      if (q0 >= N2) break;   // uniform in the wave
      c128 x[X::R1][X::A], y[X::R2][X::B];
      inverse_x_first<X, N2>(Y, L, q0, N2, off, tw1, lane, x);
      wavefft::exchange_ab<X>(x, y, W, lane);
#pragma unroll
      for (int r = 0; r < X::R2; ++r) {
        wavefft::WDft<X::B>::run(y[r], 1.0);
#pragma unroll
        for (int q = 0; q < X::B; ++q) acc[i][r][q] += wa * (y[r][q].x * y[r][q].x) + wi * (y[r][q].y * y[r][q].y);
      }
    }
  }
  double* out = part + ((size_t)blockIdx.y * m.n3 + z) * N2 * N1;
#pragma unroll
  for (int i = 0; i < RR; ++i)
#pragma unroll
    for (int r = 0; r < X::R2; ++r) {
      const int id = lane + 64 * r, row = (wave + i * nw) * X::RB + id / X::A, k = id % X::A;
      if (id < X::RB * X::A && row < N2) {
#pragma unroll
        for (int q = 0; q < X::B; ++q) out[(size_t)row * N1 + k + X::A * q] = acc[i][r][q];
      }
    }
}

template <int N1, int N2, bool HPSI = true>
PlaneWave plane_wave_entry() {
  using X = wavefft::Axis<N1>;
  using Yx = wavefft::Axis<N2>;
  PlaneWave e;
  if constexpr (HPSI) e.fn = k_plane_wave<N1, N2>;
  e.ys = N2 | 1;
  e.wave_words = X::words > Yx::words ? X::words : Yx::words;
  e.rows = X::RB;
  e.cols = Yx::RB;
  e.max_waves = plane_wave_threads(N1, N2) / 64;
  constexpr DensityShape ds = density_shape<N1, N2>();
  if constexpr (ds.waves > 0) {
    e.density = k_density_wave<N1, N2, ds.rounds>;
    e.density_waves = ds.waves;
  }
  return e;
}

}  // namespace pw
