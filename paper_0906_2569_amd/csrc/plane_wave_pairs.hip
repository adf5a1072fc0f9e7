// Plane pass on wave-local two-step transforms: planes whose sides are
// neighbours among the grids of near-cubic cells (the smallest smooth
// n >= 4 h + 1 for h and h + 1, as a shifted k-point gives them), up to 125.
// Other unequal planes stay on the generic LDS kernel, three to seven times
// the time per point.
#include "plane_wave_impl.h"

pw::PlaneWave pw::plane_wave_f64_pairs(int n1, int n2) {
#define PW_PAIR(a, b)                                              \
  if (n1 == a && n2 == b) return plane_wave_entry<a, b>(); \
  if (n1 == b && n2 == a) return plane_wave_entry<b, a>();
  PW_PAIR(24, 25)
  PW_PAIR(25, 30)
  PW_PAIR(30, 36)
  PW_PAIR(36, 40)
  PW_PAIR(40, 45)
  PW_PAIR(45, 50)
  PW_PAIR(50, 54)
  PW_PAIR(54, 60)
  PW_PAIR(60, 64)
  PW_PAIR(64, 72)
  PW_PAIR(72, 75)
  PW_PAIR(75, 80)
  PW_PAIR(80, 81)
  PW_PAIR(81, 90)
  PW_PAIR(90, 96)
  PW_PAIR(96, 100)
  PW_PAIR(100, 108)
  PW_PAIR(108, 120)
  PW_PAIR(120, 125)
#undef PW_PAIR
  return {};
}
