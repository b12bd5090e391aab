// tpmc_units.hpp -- how the persistent kernel cuts a work entry's particles into
// the units its waves take.  Integer arithmetic on the entry lists alone, so
// every wave computes the same cut.
#ifndef TPMC_UNITS_HPP
#define TPMC_UNITS_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tpmc {

__host__ __device__ inline uint32_t log2_floor(uint64_t v) { return 63u - (uint32_t)__builtin_clzll(v | 1ull); }

// How the workgroups of a launch start: every part has workgroups of its own, so
// that no part is left to be found by waves that look for one.  Each workgroup has
// `own` consecutive parts, which it works off in turn; the parts from `shared` on,
// fewer than there are workgroups, are started on by several each: div of them, one
// more for the first rem.  With the parts beyond one per workgroup left to whoever
// came first, all waves of a launch went for the same part, thousands of atomics on
// its counter (20000 queries of 256 particles on a plate 430 ms, 0.8 now; 1500 of 1000
// 8.5 ms, 0.2).  With the parts dealt out whole, some workgroups had one more than
// others (1100 queries of 50000 on a cylinder 8.4 ms, 6.8 now).
struct StartPlan {
  uint32_t own, shared, div, rem;  // own 0, div 0: no workgroup has a part
};

__host__ __device__ inline StartPlan start_plan_of(uint32_t groups, uint32_t parts) {
  const uint32_t own = parts / groups, left = parts % groups;
  return StartPlan{own, own * groups, left ? groups / left : 0u, left ? groups % left : 0u};
}

// Workgroups that start on a part.
__host__ __device__ inline uint32_t start_groups(const StartPlan& s, uint32_t part) {
  return part < s.shared ? 1u : s.div + (part - s.shared < s.rem ? 1u : 0u);
}

// The shared part that workgroup i starts on (div > 0), and its number among the
// part's workgroups; its own are [i * own, (i + 1) * own).
__host__ __device__ inline void start_shared(const StartPlan& s, uint32_t i, uint32_t& part, uint32_t& rank) {
  const uint32_t more = s.rem * (s.div + 1u);
  if (i < more) {
    part = s.shared + i / (s.div + 1u);
    rank = i % (s.div + 1u);
  } else {
    part = s.shared + s.rem + (i - more) / s.div;
    rank = (i - more) % s.div;
  }
}

// One part's particles [lo, lo + n), in units of whole 64-particle batches:
//  * ns starting units of s particles, the w-th for the w-th wave that starts
//    on the part: no atomic, and at most half of an equal share each (the
//    whole part where it has at most 64 particles per starting wave).
//  * The rest by the part's counter: units of u0 first, then, over the last
//    2^lw u0 particles, 2^lw units (about one per wave that the part has work
//    for) of each size u0 / 2, u0 / 4, ..., 2^kUnitMinLog2, so that the waves
//    end within a small unit of each other.
// Fixed units of a quarter tile (4096 particles) left most of the chip idle:
// 1e5 particles ran on 25 waves (1.67 ms on a 1280-triangle sphere; 0.13 ms
// now), and 1e7 on 2442 of the 4096 resident ones (satellite 2.03 -> 1.48 ms).
// The smallest counted unit, 128 particles: 512 gave the plate sweep 4 % and
// took 2-3 % from the cylinder and attitude sweeps; 64 was slower on both.
constexpr uint32_t kUnitMinLog2 = 7;

struct UnitPlan {
  uint64_t lo, n;    // the part's particles
  uint64_t ns_end;   // particles of the starting units (may exceed n)
  uint64_t n0;       // counted units of the full size
  uint32_t s_log2;   // starting units hold 2^s_log2 particles
  uint32_t u_log2;   // full counted units 2^u_log2
  uint32_t lw;
  uint32_t top;      // halvings of u0 down to the smallest unit
};

// Part i of 2^sub_log2 of the entry [e0, e0 + all); ns starting waves; share
// 2^share_log2 particles per wave of the launch; no unit above 64 2^cap_log2, no
// starting unit above 64 2^start_cap_log2.
__host__ __device__ inline UnitPlan unit_plan_of(uint64_t e0, uint64_t all, uint32_t sub_log2, uint32_t i, uint64_t ns,
                                                 uint32_t share_log2, uint32_t cap_log2, uint32_t start_cap_log2 = 32u) {
  UnitPlan p;
  const uint64_t step = (((all + (1ull << sub_log2) - 1ull) >> sub_log2) + 63ull) & ~63ull;
  const uint64_t b = i * step < all ? i * step : all, e = (i + 1ull) * step < all ? (i + 1ull) * step : all;
  p.lo = e0 + b;
  p.n = e - b;
  // the largest s = 64 2^k with 2 ns s <= n
  uint32_t k = 0;
  if (ns != 0ull && ns * 128ull <= p.n) {
    k = log2_floor(p.n) - log2_floor(ns * 128ull);
    if ((ns * 128ull) << k > p.n) --k;
    if (k > cap_log2) k = cap_log2;
    if (k > start_cap_log2) k = start_cap_log2;
  }
  p.s_log2 = 6u + k;
  p.ns_end = ns << p.s_log2;
  const uint64_t rest = p.n > p.ns_end ? p.n - p.ns_end : 0ull;
  p.lw = log2_floor(p.n >> share_log2);
  const uint32_t d = log2_floor(rest >> (p.lw + 1u));
  p.u_log2 = d < 6u ? 6u : (d > 6u + cap_log2 ? 6u + cap_log2 : d);
  p.top = p.u_log2 > kUnitMinLog2 ? p.u_log2 - kUnitMinLog2 : 0u;
  const uint64_t tail = ((1ull << p.u_log2) - ((1ull << p.u_log2) >> p.top)) << p.lw;  // units below u0, 2^lw each
  p.n0 = rest > tail ? (rest - tail) >> p.u_log2 : 0ull;
  return p;
}

// Counted unit t of a part: [b, e) relative to p.lo; false when t lies beyond the part.
__host__ __device__ inline bool counted_unit(const UnitPlan& p, uint64_t t, uint64_t& b, uint64_t& e) {
  uint64_t at, size;
  if (t < p.n0) {
    size = 1ull << p.u_log2;
    at = t << p.u_log2;
  } else {
    t -= p.n0;
    const uint64_t l = (t >> p.lw) + 1ull;
    const uint32_t lev = l < p.top ? (uint32_t)l : p.top;  // size u0 >> lev
    size = (1ull << p.u_log2) >> lev;
    // levels 1 .. lev - 1 hold 2^lw (u0 - (u0 >> (lev - 1))) particles
    const uint64_t before = lev > 0u ? ((1ull << p.u_log2) - ((1ull << p.u_log2) >> (lev - 1u))) << p.lw : 0ull;
    at = (p.n0 << p.u_log2) + before + ((t - (lev > 0u ? (uint64_t)(lev - 1u) << p.lw : 0ull)) << (p.u_log2 - lev));
  }
  b = p.ns_end + at;
  e = b + size < p.n ? b + size : p.n;
  return b < p.n;
}

}  // namespace tpmc

#endif  // TPMC_UNITS_HPP
