// Device helpers shared by the z passes of H.psi (hpsi.hip, zwave.hip).
#pragma once
#include "plan.h"

namespace pw {

template <typename T>
__device__ __forceinline__ cpx<T> to_t(c128 v) { return cpx<T>{(T)v.x, (T)v.y}; }

// Workgroup -> (stick chunk, band) of the z passes.  Workgroups go to the 8
// XCDs round-robin by linear id, so all chunks of one band get ids of one
// residue mod 8: each band's scattered sphere reads then meet one L2.  The
// grid has gz * roundup(nb, 8) workgroups; those past the last band exit.
constexpr int kXcds = 8;
__device__ __forceinline__ bool z_tile(int gz, int nb, int& chunk, int& band) {
  const int id = blockIdx.x;
  const int slot = id / kXcds;
  band = (slot / gz) * kXcds + id % kXcds;
  chunk = slot % gz;
  return band < nb;
}

__device__ __forceinline__ c128 gamma_pack(const c128* __restrict__ pa, const c128* __restrict__ pb, int enc) {
  const int g = enc >> 1;
  c128 a = pa[g];
  c128 b = pb ? pb[g] : c128{0.0, 0.0};
  if (g == 0) { a.y = 0.0; b.y = 0.0; }   // psi(0) is real
  return (enc & 1) ? c128{a.x + b.y, b.x - a.y} : c128{a.x - b.y, a.y + b.x};
}

// z passes of one length: sphere -> sticks and back, complex and Gamma forms
// (arguments as the kernels of hpsi.hip), `sticks` sticks per workgroup of
// `threads` threads.
template <typename T>
struct ZFns {
  void (*inv)(SphereMap, const c128*, int, cpx<T>*, const cpx<T>*, int, int) = nullptr;
  void (*fwd)(SphereMap, const cpx<T>*, const c128*, int, c128*, int, const cpx<T>*, double, int, int, int) = nullptr;
  void (*inv_g)(SphereMap, const c128*, int, cpx<T>*, const cpx<T>*, int, int, int) = nullptr;
  void (*fwd_g)(SphereMap, cpx<T>*, const cpx<T>*, int, int) = nullptr;
  int sticks = 0, threads = 0;
};

// z passes on two-step transforms (zwave.hip); inv == nullptr where none covers n3
ZFns<double> zwave_f64(int n3);

}  // namespace pw
