// Host harness for tpmc_units.hpp: for each line "e0 all sub_log2 grid share_log2 cap_log2"
// walks every part's starting and counted units as the kernel's waves take them
// (start_div / start_rem workgroups of four waves per part) and prints "ok", or
// what is wrong: the units of the parts, in order, have to cover [e0, e0 + all)
// exactly once, in whole batches (but for the last), none above 64 2^cap_log2.
#include <cstdio>

#include "tpmc_units.hpp"

static const char* check(unsigned long long e0, unsigned long long all, unsigned sub, unsigned grid, unsigned share,
                         unsigned cap) {
  const unsigned parts = 1u << sub, div = grid / parts, rem = grid % parts;
  uint64_t at = e0;
  for (unsigned i = 0; i < parts; ++i) {
    const uint64_t ns = (uint64_t)(div + (i < rem ? 1u : 0u)) * 4u;
    const tpmc::UnitPlan p = tpmc::unit_plan_of(e0, all, sub, i, ns, share, cap);
    if (p.lo != at) return "part does not begin where the one before ended";
    uint64_t pos = 0;
    for (uint64_t w = 0; w < ns && (w << p.s_log2) < p.n; ++w) {
      const uint64_t e = (w + 1) << p.s_log2;
      pos = e < p.n ? e : p.n;
      if ((1ull << p.s_log2) > (64ull << cap)) return "starting unit above the cap";
    }
    uint64_t b, e;
    for (uint64_t t = 0; tpmc::counted_unit(p, t, b, e); ++t) {
      if (b != pos || e <= b) return "counted unit does not follow the one before";
      if (e - b > (64ull << cap)) return "counted unit above the cap";
      if (b % 64 || (e % 64 && e != p.n)) return "unit is not whole batches";
      pos = e;
      if (t > 100000000ull) return "too many units";
    }
    for (uint64_t t = 0; t < 3; ++t)  // beyond the end every index stays beyond it
      if (pos == p.n && p.ns_end + 64 * t > p.n && tpmc::counted_unit(p, p.n + t, b, e)) return "unit beyond the part";
    if (pos != p.n) return "part not covered";
    at += p.n;
  }
  return at == e0 + all ? "ok" : "entry not covered";
}

int main() {
  unsigned long long e0, all;
  unsigned sub, grid, share, cap;
  while (std::scanf("%llu %llu %u %u %u %u", &e0, &all, &sub, &grid, &share, &cap) == 6)
    std::printf("%s\n", check(e0, all, sub, grid, share, cap));
  return 0;
}
