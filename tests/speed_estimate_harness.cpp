// Host harness for the seeding estimate's normal speed (speed_estimate32 in
// tpmc_math.hpp): builds the table of starts as the library does (long double
// bisection), then for each line "s k" prints whether the estimate keeps the draw k
// at s and how far its speed is from the root of F(x | s) = u chi(s), u = (k + 1/2) 2^-32.
#include <cmath>
#include <cstdio>
#include <vector>

#include "tpmc_internal.h"
#include "tpmc_math.hpp"

static const long double kRootPi = 1.7724538509055160272981674833411451828L;

// Root for u = p / (p + q).
static long double root(long double s, long double p, long double q) {
  const long double es2 = expl(-s * s), es = erfcl(-s);
  const long double target = (es2 + kRootPi * s * es) * (p / (p + q));
  long double lo = 0.0L, hi = (s > 0.0L ? s : 0.0L) + 7.0L;
  for (int it = 0; it < 70; ++it) {
    const long double m = 0.5L * (lo + hi), d = m - s;
    const long double F = es2 - expl(-d * d) + kRootPi * s * (es - erfcl(d));
    (F < target ? lo : hi) = m;
  }
  return 0.5L * (lo + hi);
}

int main() {
  using namespace tpmc;
  std::vector<float> tab((size_t)kVnNS * kVnNT, -1.0f);  // filled where it is read
  auto at = [&](int i, int j) {
    float& v = tab[(size_t)i * kVnNT + j];
    if (v < 0.0f) v = (float)root(kVnS0 + i * (double)kVnDS, 1.0L, expl(-(kVnT0 + j * (long double)kVnDT)));
    return v;
  };
  float s;
  unsigned long long k;
  while (std::scanf("%a %llu", &s, &k) == 2) {
    const float u = ((float)k + 0.5f) * 0x1p-32f, um = ((float)(0xFFFFFFFFull - k) + 0.5f) * 0x1p-32f;
    const float fs = (s - kVnS0) / kVnDS;
    const float t = (logf(u) - logf(um) - kVnT0) / kVnDT;
    const float ft = fminf(fmaxf(t, 0.0f), (float)(kVnNT - 1));
    const int i = (int)fs < kVnNS - 2 ? (int)fs : kVnNS - 2, j = (int)ft < kVnNT - 2 ? (int)ft : kVnNT - 2;
    const float a = fs - (float)i, b = ft - (float)j;
    const float x0 = fmaf(b, at(i, j + 1) - at(i, j), at(i, j)), x1 = fmaf(b, at(i + 1, j + 1) - at(i + 1, j), at(i + 1, j));
    float x = fmaf(a, x1 - x0, x0);
    const bool keep = speed_estimate32(s, u, x);
    std::printf("%d %Lg\n", keep ? 1 : 0, fabsl((long double)x - root(s, 2.0L * k + 1.0L, 0x1p33L - (2.0L * k + 1.0L))));
  }
  return 0;
}
