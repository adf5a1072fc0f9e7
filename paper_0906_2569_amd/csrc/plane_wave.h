// Plane pass kernels on wave-local two-step transforms (plane_wave_impl.h):
// lookup by grid size.
#pragma once
#include "plan.h"

namespace pw {

struct PlaneWave {
  void (*fn)(SphereMap, c128*, const double*, const c128*, const c128*, int) = nullptr;
  // density of transforms [0, nt): groups of `per` transforms along grid.y (k_density_wave)
  void (*density)(SphereMap, const c128*, int, int, int, int, const double*, const c128*, const c128*,
                  double*) = nullptr;
  int density_waves = 0;
  int ys = 0;           // LDS stride of an x column
  int wave_words = 0;   // exchange words (float64) of a wave
  int rows = 0, cols = 0;   // rows / x columns a wave transforms at a time
  int max_waves = 0;        // per workgroup
  size_t lds(int nxr, int pp, int nwaves) const {
    return sizeof(c128) * (size_t)pp * (nxr + 2) * ys + sizeof(double) * (size_t)nwaves * wave_words;
  }
};

// z planes per workgroup and waves of a launch
struct PlaneWaveShape {
  int pp = 0, nwaves = 0;
};

// fn (density) == nullptr where no plane pass (density) kernel covers n1 x n2
PlaneWave plane_wave_f64(int n1, int n2);
PlaneWave plane_wave_f64_pairs(int n1, int n2);   // n1 != n2

}  // namespace pw
