// Plane pass on wave-local two-step transforms: square planes.
#include "plane_wave_impl.h"

pw::PlaneWave pw::plane_wave_f64(int n1, int n2) {
  if (n1 != n2) return plane_wave_f64_pairs(n1, n2);
  switch (n1) {
#define PW_SQUARE(n) \
  case n: return plane_wave_entry<n, n>()
// the density's kernel alone: the register (60) and lane-group (80, 96, 128)
// kernels are the faster plane pass of H psi there, also when measured
#define PW_DENSITY(n) \
  case n: return plane_wave_entry<n, n, false>()
    PW_SQUARE(24);
    PW_SQUARE(25);
    PW_SQUARE(27);
    PW_SQUARE(30);
    PW_SQUARE(32);
    PW_SQUARE(36);
    PW_SQUARE(40);
    PW_SQUARE(45);
    PW_SQUARE(48);
    PW_SQUARE(50);
    PW_SQUARE(54);
    PW_DENSITY(60);
    PW_SQUARE(64);
    PW_SQUARE(72);
    PW_SQUARE(75);
    PW_DENSITY(80);
    PW_SQUARE(81);
    PW_SQUARE(90);
    PW_DENSITY(96);
    PW_SQUARE(100);
    PW_SQUARE(108);
    PW_SQUARE(120);
    PW_SQUARE(125);
    PW_DENSITY(128);
    PW_SQUARE(135);
#undef PW_SQUARE
#undef PW_DENSITY
    default: return {};
  }
}
