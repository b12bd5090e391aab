// Host harness for the start of a launch (tpmc_units.hpp): for each line "groups
// parts n share_log2 cap_log2 start_cap_log2" prints "ok", or what is wrong: every part
// has a workgroup that starts on it, the workgroups of a part are numbered 0, 1, ... up
// to the number that the cut into units counts, own parts have one, and the units of a
// part of n particles, its starting units bounded, cover it exactly once.
#include <cstdio>
#include <vector>

#include "tpmc_units.hpp"

static const char* check(uint32_t groups, uint32_t parts) {
  const tpmc::StartPlan s = tpmc::start_plan_of(groups, parts);
  std::vector<uint32_t> of(parts, 0u);
  if (s.shared > parts || parts - s.shared >= groups || (parts > s.shared) != (s.div != 0u)) return "shared parts";
  for (uint32_t i = 0; i < groups; ++i) {
    for (uint32_t p = i * s.own; p < (i + 1) * s.own; ++p) {
      if (p >= s.shared || of[p] != 0u) return "own part that is another's";
      ++of[p];
    }
    if (s.div == 0u) continue;
    uint32_t p, rank;
    tpmc::start_shared(s, i, p, rank);
    if (p < s.shared || p >= parts || rank != of[p]) return "ranks of a shared part do not count up";
    ++of[p];
  }
  for (uint32_t p = 0; p < parts; ++p)
    if (of[p] == 0u || of[p] != tpmc::start_groups(s, p)) return "part without its workgroups";
  return "ok";
}

static const char* check_units(uint64_t n, uint64_t ns, uint32_t share, uint32_t cap, uint32_t start_cap) {
  const tpmc::UnitPlan p = tpmc::unit_plan_of(0, n, 0, 0, ns, share, cap, start_cap);
  if ((1ull << p.s_log2) > (64ull << start_cap) || (1ull << p.s_log2) > (64ull << cap)) return "starting unit above its cap";
  uint64_t pos = p.ns_end < n ? p.ns_end : n, b, e;
  for (uint64_t t = 0; tpmc::counted_unit(p, t, b, e); ++t) {
    if (b != pos || e <= b || e - b > (64ull << cap) || b % 64 || (e % 64 && e != n)) return "counted unit out of order";
    pos = e;
  }
  return pos == n ? "ok" : "part not covered";
}

int main() {
  uint32_t groups, parts, share, cap, start_cap;
  unsigned long long n;
  while (std::scanf("%u %u %llu %u %u %u", &groups, &parts, &n, &share, &cap, &start_cap) == 6) {
    const char* s = check(groups, parts);
    if (s[0] == 'o') s = check_units(n, tpmc::start_groups(tpmc::start_plan_of(groups, parts), parts / 2) * 4u, share, cap, start_cap);
    std::printf("%s\n", s);
  }
  return 0;
}
