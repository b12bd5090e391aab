// Host harness for tpmc_sah.hpp: for each line "level x0 y0 z0 x1 y1 z1" (two box
// centres, as hexadecimal floats) bins the pair as the build's wave stage does and
// prints its plane (-1: halved) and how many of the two triangles lie left of it.
#include <cstdio>

#include "tpmc_sah.hpp"

int main() {
  unsigned level;
  float c[2][3];
  while (std::scanf("%u %a %a %a %a %a %a", &level, &c[0][0], &c[0][1], &c[0][2], &c[1][0], &c[1][1], &c[1][2]) == 7) {
    bool use[3];
    uint32_t bins[2] = {0u, 0u};
    for (int k = 0; k < 3; ++k) {
      const int a = tpmc::f2o(c[0][k]), b = tpmc::f2o(c[1][k]);
      float cmin, scale;
      use[k] = tpmc::bin_axis(a < b ? a : b, a < b ? b : a, level, cmin, scale);
      for (int t = 0; use[k] && t < 2; ++t) bins[t] |= (uint32_t)tpmc::sah_bin(c[t][k], cmin, scale) << (8 * k);
    }
    const uint32_t t = tpmc::pair_plane(bins[0], bins[1]);
    if (t == tpmc::kNoPlane) {
      std::printf("-1 1\n");
      continue;
    }
    const uint32_t shift = 8u * (t / tpmc::kSahBins), plane = t % tpmc::kSahBins;
    std::printf("%u %d\n", t, (int)(((bins[0] >> shift) & 255u) < plane) + (int)(((bins[1] >> shift) & 255u) < plane));
  }
  return 0;
}
