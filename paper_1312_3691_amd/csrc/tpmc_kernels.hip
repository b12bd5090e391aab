// tpmc_kernels.hip -- the per-query hot path on gfx950:
//   seed_kernel     a2-a4  Philox streams, FP64 boundary seeding -> FP32 SoA
//   trace_kernel    a6-a9  BVH traversal, watertight hit, re-emission, tallies, bounce loop
//   batch_kernel    a11    persistent (query, tile) work queue; seeding fused on chip
//   reduce/finalize a10    exact integer reduction, force / moment / C_D in FP64
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <utility>

#include "tpmc_device.hpp"
#include "tpmc_launch.h"

#ifndef TPMC_PHASE_PROBE
#define TPMC_PHASE_PROBE 0
#endif

namespace tpmc {

#if TPMC_PHASE_PROBE
__device__ unsigned long long g_probe[kProbeSlots];  // ProbeSlot sums of the batched launches
#endif

namespace {

// ---------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------
__global__ void zero_i64_kernel(long long* __restrict__ p, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Several ranges in one launch (the work of a launch costs less than the launch).
__global__ void clear_kernel(ClearRanges r) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
#pragma unroll
  for (int k = 0; k < kClearRanges; ++k)
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < r.n[k]; i += stride) r.p[k][i] = 0;
}

struct ArgQueries {
  QueryDev q[kArgQueries];
};
static_assert(sizeof(ArgQueries) + sizeof(ClearRanges) + 64 <= 4096, "kernel arguments");

__global__ void clear_upload_kernel(ClearRanges r, ArgQueries h, QueryDev* __restrict__ qs, uint32_t n) {
  if (blockIdx.x == 0) {
    const uint64_t* src = reinterpret_cast<const uint64_t*>(&h);
    uint64_t* dst = reinterpret_cast<uint64_t*>(qs);
    for (uint32_t w = threadIdx.x; w < n * (uint32_t)(sizeof(QueryDev) / 8); w += blockDim.x) dst[w] = src[w];
  }
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
#pragma unroll
  for (int k = 0; k < kClearRanges; ++k)
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < r.n[k]; i += stride) r.p[k][i] = 0;
}

__global__ void zero_u32_kernel(uint32_t* __restrict__ p, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

int grid_for(uint64_t n, int cap) {
  const uint64_t g = (n + kBlock - 1) / kBlock;
  return (int)(g < (uint64_t)cap ? (g > 0 ? g : 1) : cap);
}

// ---------------------------------------------------------------------------
// a2-a4: seeding
// ---------------------------------------------------------------------------
// Tables of the latitude and normal-speed laws (latitude_start, latitude_fine,
// normal_speed_table); part of the code object, filled once per device.
__device__ float g_lat_start[kLatNS * kLatNT];
__device__ float g_lat_fine[kLatFNS * kLatFNT];  // the seeding estimate's latitude table
__device__ __align__(16) float g_vn_start[2 * (kVnNS - 1) * kVnNT];
// sin and cos of 2 pi j / 256, j = 0..255 (sincos_2pi_draw)
__device__ double g_sc_tab[512];
// exp(-y_j^2) and erfc(y_j) at y_j = j / 256 (exp_erfc_grid)
__device__ double g_ee_tab[2 * kExpErfcN];

__global__ void ee_table_kernel(double* __restrict__ tab) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= kExpErfcN) return;
  const double y = (double)j * 0x1p-8;  // y and y^2 are exact
  tab[2 * j] = exp(-(y * y));
  tab[2 * j + 1] = erfc(y);
}

__global__ void sc_table_kernel(double* __restrict__ tab) {
  const int j = threadIdx.x;
  if (j >= 256) return;
  double s, c;
  sincospi((double)j / 128.0, &s, &c);
  tab[2 * j] = s;
  tab[2 * j + 1] = c;
}

__global__ void lat_table_kernel(float* __restrict__ tab, const double* __restrict__ ee) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kLatNS * kLatNT) return;
  QueryDev q{};
  q.S = (double)kLatS0 * exp((double)(i / kLatNT) * (double)kLatDL);
  q.erfS = erf(q.S);
  q.erfcS = erfc(q.S);
  q.expmS2 = exp(-q.S * q.S);
  q.lat_k = kSqrtPi / (4.0 * q.S);
  const double t = (double)kLatT0 + (double)(i % kLatNT) * (double)kLatDT;
  const double u = 1.0 / (1.0 + exp(-t));
  double Z, G, dG, d2G, e, ta;
  latitude_G(q, ee, 1.0, Z, dG, d2G, e, ta);
  const double target = u * Z;
  double lo = -1.0, hi = 1.0;
  for (int it = 0; it < 60; ++it) {
    const double m = 0.5 * (lo + hi);
    latitude_G(q, ee, m, G, dG, d2G, e, ta);
    if (G < target) lo = m;
    else hi = m;
  }
  tab[i] = (float)(0.5 * (lo + hi));
}

// The seeding estimate's fine latitude table: the same root by the same
// FP64 bisection, at the fine table's nodes.
__global__ void lat_fine_kernel(float* __restrict__ tab, const double* __restrict__ ee) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kLatFNS * kLatFNT) return;
  QueryDev q{};
  q.S = exp(kLatFL0 + (double)(i / kLatFNT) * kLatFDL);
  q.erfS = erf(q.S);
  q.erfcS = erfc(q.S);
  q.expmS2 = exp(-q.S * q.S);
  q.lat_k = kSqrtPi / (4.0 * q.S);
  const double t = (double)kLatFT0 + (double)(i % kLatFNT) * (double)kLatFDT;
  const double u = 1.0 / (1.0 + exp(-t));
  double Z, G, dG, d2G, e, ta;
  latitude_G(q, ee, 1.0, Z, dG, d2G, e, ta);
  const double target = u * Z;
  double lo = -1.0, hi = 1.0;
  for (int it = 0; it < 60; ++it) {
    const double m = 0.5 * (lo + hi);
    latitude_G(q, ee, m, G, dG, d2G, e, ta);
    if (G < target) lo = m;
    else hi = m;
  }
  tab[i] = (float)(0.5 * (lo + hi));
}

__global__ void vn_table_kernel(float* __restrict__ tab, const double* __restrict__ ee) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kVnNS * kVnNT) return;
  const int row = i / kVnNT, col = i % kVnNT;
  const double s = (double)kVnS0 + (double)row * (double)kVnDS;
  const double t = (double)kVnT0 + (double)col * (double)kVnDT;
  const double u = 1.0 / (1.0 + exp(-t));
  const NormalSpeedConsts k = normal_speed_consts(ee, s);
  const double target = u * k.chi;
  double lo = 0.0, hi = (s > 0.0 ? s : 0.0) + 8.0;
  for (int it = 0; it < 80; ++it) {
    const double m = 0.5 * (lo + hi);
    double F, dF, d2F;
    normal_speed_F(ee, k, m, F, dF, d2F);
    if (F < target) lo = m;
    else hi = m;
  }
  const float x = (float)(0.5 * (lo + hi));
  if (row < kVnNS - 1) tab[2 * i] = x;             // first of its cells' pairs
  if (row > 0) tab[2 * (i - kVnNT) + 1] = x;       // second of the row below's
}

// Each query's own row of the fine latitude table (QueryDev::lat_own), query blockIdx.y.
__global__ __launch_bounds__(kBlock) void lat_own_kernel(const QueryDev* __restrict__ qs, float* __restrict__ rows) {
  const QueryDev& q = qs[blockIdx.y];
  const int j = blockIdx.x * kBlock + threadIdx.x;
  if (q.lat_own && j < kLatFNT) rows[(uint64_t)blockIdx.y * kLatOwnStride + j] = latitude_row(q, g_lat_fine, j);
}

struct Planes {
  float* p[6];
};

// Query blockIdx.y.
__global__ __launch_bounds__(kBlock) void seed_kernel(const QueryDev* __restrict__ qs, Planes planes) {
  const QueryDev& q = qs[blockIdx.y];
  float* __restrict__ const x0 = planes.p[0] + q.p_offset;
  float* __restrict__ const x1 = planes.p[1] + q.p_offset;
  float* __restrict__ const x2 = planes.p[2] + q.p_offset;
  float* __restrict__ const w0 = planes.p[3] + q.p_offset;
  float* __restrict__ const w1 = planes.p[4] + q.p_offset;
  float* __restrict__ const w2 = planes.p[5] + q.p_offset;
  const uint64_t n = q.N, stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
    double x[3], w[3];
    seed_particle(q, g_lat_start, g_lat_fine, nullptr, g_vn_start, g_sc_tab, g_ee_tab, i, x, w);
    x0[i] = (float)x[0];
    x1[i] = (float)x[1];
    x2[i] = (float)x[2];
    w0[i] = (float)w[0];
    w1[i] = (float)w[1];
    w2[i] = (float)w[2];
  }
}

// ---------------------------------------------------------------------------
// Loads through the global address space.  The mesh pointers reach the
// kernels inside the query record, so the compiler cannot prove that they
// address global memory and would emit flat loads, which also count against
// the LDS counter and so delay every LDS access behind them.
// ---------------------------------------------------------------------------
template <class T>
using gptr = const T __attribute__((address_space(1)))*;
typedef float vf4 __attribute__((ext_vector_type(4)));  // native vectors: HIP's float4 cannot
typedef int vi4 __attribute__((ext_vector_type(4)));    // be copied from an address-space reference

__device__ __forceinline__ TriRec load_tri(const TriRec* p, int k) {
  const gptr<vf4> g = (gptr<vf4>)(p + k);
  const vf4 a = g[0], b = g[1], c = g[2];
  return TriRec{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w};
}

// orig[] word of a triangle: original index in bits 0..29, supporting-plane
// flags in bits 30 (nothing above the plane) and 31 (nothing below).
__device__ __forceinline__ uint32_t load_orig_word(const uint32_t* p, int k) { return ((gptr<uint32_t>)p)[k]; }
__device__ __forceinline__ uint32_t load_orig(const uint32_t* p, int k) { return load_orig_word(p, k) & kOrigIdMask; }

// Mask of the lanes where p holds.  The builtin takes the comparison's lane
// mask as it is; __ballot(int) first turns it into 0/1 values and compares
// them again.
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// A pointer every lane holds the same value of, moved to scalar registers.
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T*>(lo | (hi << 32));
}

// One lane's particle in flight.
struct Lane {
  float ox = 0.0f, oy = 0.0f, oz = 0.0f, wx = 0.0f, wy = 0.0f, wz = 0.0f;
  float D;        // momentum given along U so far (this particle)
  float E;        // energy given to the body so far, sum of |w|^2 - |w'|^2
  int prev;       // Morton position of the triangle just left
  uint32_t hits;
  uint64_t pid;   // particle index within its query
  bool live;
};

// ---------------------------------------------------------------------------
// a6: closest hit, one BVH node per step.  Nearest-child-first traversal of
// the binary BVH with the far child on a per-lane stack in LDS
// (stack[slot][lane], conflict free); leaves are tested as soon as their box
// is hit.  The traversal state lives in registers between steps, so a lane
// whose segment has ended can be given its next segment while the other
// lanes of the wave are still traversing.  The closest hit does not depend
// on the visiting order: every triangle whose t is at most the final t_best
// lies in boxes that are never culled (conservative far bound), and equal t
// keeps the lower original index.  The ray's derived constants (Ray) are
// recomputed from the lane's origin and direction after every service pass,
// so they are not held in registers across the seeding code.
// ---------------------------------------------------------------------------
constexpr int kDone = -0x7FFFFFFF - 1;  // Seg::cur once the traversal has ended

struct Seg {
  int cur;     // next node to visit, or kDone
  int sp;      // stack depth
  int best;    // closest triangle so far (Morton position), -1 if none
  int p0, p1;  // leaves whose boxes were hit, waiting for a leaf phase (-1: none)
  float t_best, b0, b1, b2;
};

__device__ __forceinline__ void seg_begin(Seg& s) {
  s.cur = 0;
  s.sp = 0;
  s.best = -1;
  s.p0 = s.p1 = -1;
  s.t_best = __builtin_inff();
}

// Lane states: traversing (next node known, no leaf waiting), waiting for a
// leaf phase, or finished (segment ready for its service pass).
__device__ __forceinline__ bool seg_traversing(const Seg& s) { return s.cur != kDone && s.p0 < 0; }
__device__ __forceinline__ bool seg_finished(const Seg& s) { return s.cur == kDone && s.p0 < 0; }

// Candidate leaf k: two-sided test, the triangle just left excluded.
template <bool COUNT>
__device__ __forceinline__ void test_leaf(const TriRec* tris, const uint32_t* orig, const Ray& r, int k, int prev,
                                          Seg& s, uint32_t& n_tests) {
  if (COUNT && k != prev) ++n_tests;
  float t, u0, u1, u2;
  if (intersect_tri(r, load_tri(tris, k), s.t_best, t, u0, u1, u2) && k != prev) {
    // t <= t_best here; an exact tie keeps the lower original index
    const bool take = t < s.t_best || (s.best >= 0 && load_orig(orig, k) < load_orig(orig, s.best));
    if (take) {
      s.best = k;
      s.t_best = t;
      s.b0 = u0;
      s.b1 = u1;
      s.b2 = u2;
    }
  }
}

// One traversal step of a traversing lane.  Hit leaves are not tested here
// but recorded in p0 / p1 (a node has two children), and the lane then waits
// for a leaf phase: the costly triangle test runs for many lanes at once
// instead of for the few lanes that happen to reach a leaf in a given step.
// Each node is entered at most once per ray, so a segment takes at most nt - 1
// steps and nt leaf tests.  Trees of depth <= 4 (a 4-slot stack: meshes of a
// few triangles, where nearly every step ends at leaves) test them in place.
template <int STACK, bool COUNT>
__device__ __forceinline__ void trav_step(const Node* nodes, const TriRec* tris, const uint32_t* orig, const Ray& r,
                                          int prev, Seg& s, int (*stk)[kBlock], uint32_t& n_nodes,
                                          uint32_t& n_tests) {
  const int lane = threadIdx.x;
  // 32-bit byte offset from the (scalar) base: one shift, no 64-bit address math
  const gptr<char> base = (gptr<char>)nodes;
  const uint32_t off = (uint32_t)s.cur * (uint32_t)sizeof(Node);
  const gptr<vf4> np = (gptr<vf4>)(base + off);
  const vf4 A = np[0], B = np[1], C = np[2];
  const vi4 L = ((gptr<vi4>)(base + off))[3];
  if (COUNT) ++n_nodes;
  float tn0, tn1;
  bool h0 = slab(r, A.x, A.y, A.z, A.w, B.x, B.y, s.t_best, tn0);
  bool h1 = slab(r, B.z, B.w, C.x, C.y, C.z, C.w, s.t_best, tn1);
  const bool leaf0 = h0 && L.x < 0, leaf1 = h1 && L.y < 0;
  if (STACK <= 4) {
    if (leaf0) test_leaf<COUNT>(tris, orig, r, ~L.x, prev, s, n_tests);
    if (leaf1) test_leaf<COUNT>(tris, orig, r, ~L.y, prev, s, n_tests);
  } else {
    if (leaf0) s.p0 = ~L.x;
    if (leaf1) {
      if (leaf0) s.p1 = ~L.y;
      else s.p0 = ~L.y;
    }
  }
  h0 = h0 && !leaf0;
  h1 = h1 && !leaf1;
  if (h0 && h1 && s.sp < STACK) {
    const bool first0 = tn0 <= tn1;
    stk[s.sp][lane] = first0 ? L.y : L.x;
    ++s.sp;
    s.cur = first0 ? L.x : L.y;
  } else if (h0) {
    s.cur = L.x;
  } else if (h1) {
    s.cur = L.y;
  } else {
    s.cur = s.sp == 0 ? kDone : stk[--s.sp][lane];
  }
}

// Leaf phase (convergent): every waiting lane tests its first pending leaf;
// a second one moves up and waits for the next phase.
template <bool COUNT>
__device__ __forceinline__ void leaf_phase(const TriRec* tris, const uint32_t* orig, const Ray& r, int prev, Seg& s,
                                           uint32_t& n_tests) {
  if (s.p0 >= 0) {
    test_leaf<COUNT>(tris, orig, r, s.p0, prev, s, n_tests);
    s.p0 = s.p1;
    s.p1 = -1;
  }
}

// Whether a ray from (o, w) passes the slab test of either box of the root
// node with no distance bound, i.e. whether its first traversal step can find
// anything.  Same reciprocals and test as the traversal.
__device__ __forceinline__ bool ray_enters_root(const Node* nodes, const float o[3], const float w[3]) {
  Ray r;
  r.ox = o[0]; r.oy = o[1]; r.oz = o[2];
  r.idx = __builtin_amdgcn_rcpf(w[0]);
  r.idy = __builtin_amdgcn_rcpf(w[1]);
  r.idz = __builtin_amdgcn_rcpf(w[2]);
  const gptr<vf4> np = (gptr<vf4>)nodes;
  const vf4 A = np[0], B = np[1], C = np[2];
  float tn;
  const float inf = __builtin_inff();
  return slab(r, A.x, A.y, A.z, A.w, B.x, B.y, inf, tn) || slab(r, B.z, B.w, C.x, C.y, C.z, C.w, inf, tn);
}

// Momentum and moment of one hit, ready for the tallies.
struct Hit {
  bool valid;
  uint32_t id;    // original triangle index
  float dx, dy, dz, lx, ly, lz;
};

// Exact integer accumulators: per lane the quantised per-particle sums, per
// wave (scalar registers, from ballots at convergent points) the event
// counts.  Rays and segments are not kept: a particle retires by missing,
// escaping or reaching the hit cap, and every segment ends in a hit, an
// escape or a miss, so rays = missed + escaped + capped and segments = hits +
// missed + escaped (an escape through a supporting plane is one untraced
// segment after the hit).
struct Acc {
  long long sD, sD2, sE, sE2, tot[7];
  uint32_t nodes, tests;  // traversal work (counting kernels only)
  // wave-uniform
  uint64_t hits, missed, escaped, capped;
  uint64_t tr_capped;  // re-emissions whose temperature the kernel's bound limited
  uint64_t guard;      // segments ended by the traversal step bound
};

__device__ __forceinline__ void acc_zero(Acc& A) {
  A.sD = A.sD2 = A.sE = A.sE2 = 0;
#pragma unroll
  for (int c = 0; c < 7; ++c) A.tot[c] = 0;
  A.hits = A.missed = A.escaped = A.capped = 0;
  A.tr_capped = A.guard = 0;
  A.nodes = A.tests = 0;
}

__device__ __forceinline__ uint64_t lanes(bool p) { return (uint64_t)__popcll(__builtin_amdgcn_ballot_w64(p)); }

// The lane number as a value of its own: comparisons with it are not moved out of
// the loops around (a mask of two scalar registers each, held throughout).
__device__ __forceinline__ uint32_t local_lane() {
  uint32_t l = threadIdx.x & 63u;
  __asm__ volatile("" : "+v"(l));
  return l;
}

// Set bits of a wave mask below the calling lane (v_mbcnt; no per-lane mask kept live).
__device__ __forceinline__ uint32_t below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Phase probe of batch_kernel, in libraries built with TPMC_PHASE_PROBE=1
// (elsewhere PROBE(...) expands to nothing): each wave reads the shader clock
// around its phases and sums cycles, passes and active lanes, all
// wave-uniform, into one VGPR whose lane k holds ProbeSlot k (32 bits: a wave
// of one launch stays far below 2^32 cycles and passes); lanes kPrTs, kPrTc
// and kPrTp hold the clock at the wave's start, at the current tile claim and
// at the current phase's start.  Lanes are written with v_writelane and read
// with v_readlane (no lane masks, no long-lived scalar registers), so the
// instrumented kernel needs at most a register or two more than the ordinary
// one; the instances that run four waves per SIMD are held to that occupancy
// (amdgpu_waves_per_eu, at the cost of a few spilled dwords), so that the
// probe measures the kernel at its own occupancy.  At exit lane k adds its
// slot to g_probe.
#if TPMC_PHASE_PROBE
#define PROBE(...) __VA_ARGS__
constexpr int kPrTp = 29, kPrTs = 30, kPrTc = 31;
static_assert(kProbeSlots <= kPrTp, "probe lanes");
__device__ __forceinline__ uint32_t probe_now() { return (uint32_t)__builtin_amdgcn_s_memtime(); }
__device__ __forceinline__ uint32_t probe_get(uint32_t v, int k) { return __builtin_amdgcn_readlane(v, k); }
template <int K>
__device__ __forceinline__ void probe_set(uint32_t& v, uint32_t x) {
  // the trailing wait states keep a v_readlane of the written VGPR right after it exact
  asm("v_writelane_b32 %0, %1, %2\n\ts_nop 1" : "+v"(v) : "s"(x), "i"(K));
}
template <int K>
__device__ __forceinline__ void probe_add(uint32_t& v, uint32_t x) { probe_set<K>(v, probe_get(v, K) + x); }
template <int K>
__device__ __forceinline__ void probe_since(uint32_t& v, int t) { probe_add<K>(v, probe_now() - probe_get(v, t)); }
#else
#define PROBE(...)
#endif

// Outcome of a finished segment.  kOutHitLeft: a hit whose outgoing segment
// cannot hit anything (the mesh lies on the other side of the triangle's
// plane), so that segment is counted and the particle escapes untraced.
// (names distinct from the scalar-slot indices kMissed, kEscaped, kCapped)
enum Outcome : int { kOutGoOn = 0, kOutMissed = 1, kOutEscaped = 2, kOutCapped = 3, kOutHitLeft = 4 };

// a7-a9 for a lane whose traversal has ended: re-emission and bookkeeping of
// the hit, or the particle's exit.  The particle retires unless kOutGoOn.
__device__ __forceinline__ int finish_segment(const TriRec* tris, const uint32_t* orig, const QueryDev& q, Lane& L,
                                              const Seg& s, Hit& h, int32_t& first_id, bool& tr_limited) {
  const int k = s.best;
  first_id = -2;  // not the first segment's outcome
  if (k < 0) {
    if (L.hits == 0) {
      first_id = -1;
      return kOutMissed;
    }
    return kOutEscaped;
  }
  const TriRec tr = load_tri(tris, k);
  const uint32_t ow = load_orig_word(orig, k);
  const uint32_t id = ow & kOrigIdMask;
  const float px = s.b0 * tr.v0x + s.b1 * tr.v1x + s.b2 * tr.v2x;
  const float py = s.b0 * tr.v0y + s.b1 * tr.v1y + s.b2 * tr.v2y;
  const float pz = s.b0 * tr.v0z + s.b1 * tr.v1z + s.b2 * tr.v2z;
  float nwx = L.wx, nwy = L.wy, nwz = L.wz;
  tr_limited = reemit(q, L.pid, L.hits, tr.nx, tr.ny, tr.nz, nwx, nwy, nwz);
  L.E += (L.wx * L.wx + L.wy * L.wy + L.wz * L.wz) - (nwx * nwx + nwy * nwy + nwz * nwz);
  const float dx = L.wx - nwx, dy = L.wy - nwy, dz = L.wz - nwz;
  const float rx = px - q.c0f[0], ry = py - q.c0f[1], rz = pz - q.c0f[2];
  h.valid = true;
  h.id = id;
  h.dx = dx; h.dy = dy; h.dz = dz;
  h.lx = ry * dz - rz * dy;
  h.ly = rz * dx - rx * dz;
  h.lz = rx * dy - ry * dx;
  L.D += dx * q.Uf[0] + dy * q.Uf[1] + dz * q.Uf[2];
  if (L.hits == 0) first_id = (int32_t)id;
  ++L.hits;
  // The next ray starts at the hit point moved to the side the particle leaves
  // from by 8 FP32 ulps of the triangle's coordinate scale: the rounded
  // barycentric point can lie a few ulps behind the surface, and a ray started
  // there would cross a coplanar or adjacent triangle from the wrong side.
  const float scale = fmaxf(fmaxf(fmaxf(fabsf(tr.v0x), fabsf(tr.v0y)), fmaxf(fabsf(tr.v0z), fabsf(tr.v1x))),
                            fmaxf(fmaxf(fabsf(tr.v1y), fabsf(tr.v1z)),
                                  fmaxf(fmaxf(fabsf(tr.v2x), fabsf(tr.v2y)), fabsf(tr.v2z))));
  const float side = (L.wx * tr.nx + L.wy * tr.ny + L.wz * tr.nz) < 0.0f ? 1.0f : -1.0f;
  const float eps = side * scale * 0x1p-20f;
  L.ox = px + eps * tr.nx; L.oy = py + eps * tr.ny; L.oz = pz + eps * tr.nz;
  L.wx = nwx; L.wy = nwy; L.wz = nwz;
  L.prev = k;
  if (L.hits >= q.rmax) return kOutCapped;
  // the emission side is empty of mesh points (see support_kernel)
  const bool clear = side > 0.0f ? (ow >> 30) & 1u : (ow >> 31) & 1u;
  return clear ? kOutHitLeft : kOutGoOn;
}

// Event counts of a service pass (convergent): lanes with fin set ended a
// segment with outcome out (hit: with a hit; limited: whose re-emission the
// temperature bound limited).
__device__ __forceinline__ void count_pass(Acc& A, bool fin, int out, bool hit, bool limited) {
  A.hits += lanes(fin && hit);
  A.missed += lanes(fin && out == kOutMissed);
  A.escaped += lanes(fin && (out == kOutEscaped || out == kOutHitLeft));
  A.capped += lanes(fin && out == kOutCapped);
  A.tr_capped += lanes(fin && limited);
}

__device__ __forceinline__ void retire(const QueryDev& q, const Lane& L, Acc& A) {
  A.sD += fx(L.D, q.scaleD);
  A.sD2 += fx(L.D * L.D, q.scaleD2);
  A.sE += fx(L.E, q.scaleE);
  A.sE2 += fx(L.E * L.E, q.scaleE2);
}

// Per-triangle sums of a pass's hits, added in device memory with eight lanes to
// a hit: seven consecutive words per triangle go out in one instruction, and
// the L2 takes them as one or two cache-line requests.  With a lane to a hit
// and an instruction to a word every lane is a request of its own: 23e9 atomics/s
// for the chip against 92e9 this way (any number of triangles from 1280 to
// 50000, measured).  4e6 particles on a 1280-triangle sphere: 3.78 ms before,
// 1.10 now, 0.67 with totals alone.  A lane with a hit has no segment in flight, so its column of the
// traversal stack is free: the hit's values are handed over there.  Called by
// every lane of the wave (convergent).
template <int STACK>
__device__ __forceinline__ void tally_rows(const QueryDev& q, const Hit& h, long long* __restrict__ g,
                                           int (*stk)[kBlock]) {
  const uint64_t m = ballot(h.valid);
  if (m == 0ull) return;
  const uint32_t lane = local_lane(), first = threadIdx.x & ~63u;
  if (h.valid) {
    stk[0][threadIdx.x] = (int)rintf(h.dx * q.scaleF);
    stk[1][threadIdx.x] = (int)rintf(h.dy * q.scaleF);
    stk[2][threadIdx.x] = (int)rintf(h.dz * q.scaleF);
    stk[3][threadIdx.x] = (int)rintf(h.lx * q.scaleL);
    stk[4][threadIdx.x] = (int)rintf(h.ly * q.scaleL);
    stk[5][threadIdx.x] = (int)rintf(h.lz * q.scaleL);
    stk[6][threadIdx.x] = 1;
    stk[7][threadIdx.x] = (int)h.id;
  }
  const uint32_t n = (uint32_t)__popcll(m);
  // lane o < n learns the lane of the o-th hit
  const int from = __builtin_amdgcn_ds_permute((int)((h.valid ? below(m) : n + below(~m)) * 4u), (int)lane);
  __builtin_amdgcn_wave_barrier();
  for (uint32_t o = lane >> 3; o - (lane >> 3) < n; o += 8u) {
    const uint32_t col = first + (uint32_t)__builtin_amdgcn_ds_bpermute((int)((o & 63u) * 4u), from), c = lane & 7u;
    if (o < n && c < 7u) atomic_add_i64(g + 7ull * (uint32_t)stk[7][col] + c, (long long)stk[c][col]);
  }
  __builtin_amdgcn_wave_barrier();
}

// Tally of one hit per lane.  Called by every lane of the wave (convergent).
// Totals-only sums go to the wave's LDS slots lds[c][wave] (LDS atomics; the
// few lanes of a pass with a hit share them) when TOT_LDS (the persistent
// kernel, short of registers), else to the lane's registers.
template <int MODE, int STACK, bool TOT_LDS = true>
__device__ __forceinline__ void tally(const QueryDev& q, const Hit& h, long long* __restrict__ g,
                                      unsigned long long* lds, int (*stk)[kBlock], Acc& A) {
  if (STACK >= 8 && (MODE == kTallyGlobal || (MODE == kTallyAuto && q.per_tri))) {
    tally_rows<STACK>(q, h, g, stk);
    return;
  }
  long long v[7];
  // one hit's values are below 2^30 in magnitude after scaling (scale choice)
  v[0] = fx32(h.dx, q.scaleF); v[1] = fx32(h.dy, q.scaleF); v[2] = fx32(h.dz, q.scaleF);
  v[3] = fx32(h.lx, q.scaleL); v[4] = fx32(h.ly, q.scaleL); v[5] = fx32(h.lz, q.scaleL);
  v[6] = 1;
  if ((MODE == kTallyTotals || (MODE == kTallyAuto && !q.per_tri)) && TOT_LDS) {  // the wave's LDS slots [c][wave]
    if (h.valid) {
#pragma unroll
      for (int c = 0; c < 7; ++c) atomicAdd(lds + c * kWaves + (threadIdx.x >> 6), (unsigned long long)v[c]);
    }
  } else if (MODE == kTallyTotals || (MODE == kTallyAuto && !q.per_tri)) {
    if (h.valid) {
#pragma unroll
      for (int c = 0; c < 7; ++c) A.tot[c] += v[c];
    }
  } else if (MODE == kTallyGlobal || MODE == kTallyAuto) {
    if (h.valid) {
#pragma unroll
      for (int c = 0; c < 7; ++c) atomic_add_i64(g + 7ull * h.id + c, v[c]);
    }
  } else if (MODE == kTallyLds) {
    if (h.valid) {
#pragma unroll
      for (int c = 0; c < 7; ++c) atomicAdd(lds + 7u * h.id + c, (unsigned long long)v[c]);
    }
  } else {  // kTallyLane: the lane's own LDS slots [7 * id + c][lane] (meshes of <= 2 triangles)
    if (h.valid) {
#pragma unroll
      for (int c = 0; c < 7; ++c) atomicAdd(lds + (7u * h.id + c) * kBlock + threadIdx.x, (unsigned long long)v[c]);
    }
  }
}

// Wave-uniform 64-bit values, one per lane: lane k holds the k-th (0 if none).
// Written with v_writelane straight from scalar registers: a select per lane
// would have the compiler hold the values in vector registers throughout.
struct LaneSums {
  int lo = 0, hi = 0;
  template <int K>
  __device__ __forceinline__ void put(long long v) {
    // the wait states keep a scalar written, or the VGPR read, by a vector
    // instruction next to it exact
    asm("s_nop 1\n\tv_writelane_b32 %0, %1, %2\n\ts_nop 1" : "+v"(lo) : "s"((uint32_t)v), "i"(K));
    asm("s_nop 1\n\tv_writelane_b32 %0, %1, %2\n\ts_nop 1" : "+v"(hi) : "s"((uint32_t)((unsigned long long)v >> 32)), "i"(K));
  }
  __device__ __forceinline__ long long get() const {
    return (long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
  }
};

template <int... C>
__device__ __forceinline__ void lane_tally_sums(LaneSums& sums, unsigned long long* lds, std::integer_sequence<int, C...>) {
  ((sums.put<C>(wave_sum_uniform((long long)lds[C * kBlock + threadIdx.x])), lds[C * kBlock + threadIdx.x] = 0ull), ...);
}

// Flush (and clear) the calling lane's per-lane tallies of a <= 2-triangle
// mesh: one wave sum per slot, lane k then adds slot k: one atomic instruction
// per wave (convergent).
__device__ __forceinline__ void flush_lane_tally(unsigned long long* lds, long long* __restrict__ g, uint32_t nt) {
  const uint32_t lane = local_lane();
  LaneSums sums;
  lane_tally_sums(sums, lds, std::make_integer_sequence<int, 2 * 7>{});
  const long long mine = sums.get();
  if (lane < 7u * nt && lane < 14u && mine != 0) atomic_add_i64(g + lane, mine);
}

// Wave-reduce the per-lane accumulators into a query's scalar block.  With
// TOTALS the query's force and moment totals come from the lanes' registers,
// or, with TOT_LDS, from (and clearing) the wave's LDS slots wave_tot[c][wave]
// (a compile-time choice, so that the register totals are not kept live
// across the trace loop of a kernel that never uses them).
template <bool TOT_LDS = false>
__device__ __forceinline__ void flush_acc(Acc& A, long long* __restrict__ scal, bool TOTALS,
                                          unsigned long long* wave_tot = nullptr) {
  // one value at a time, each total moved to scalar registers, so that the
  // flush adds little to the kernel's vector-register peak
  const bool lead = (threadIdx.x & 63) == 0;
  auto put = [&](long long total, int slot) {
    if (lead && total) atomic_add_i64(scal + slot, total);
  };
  put(wave_sum_uniform(A.sD), kSD);
  put(wave_sum_uniform(A.sD2), kSD2);
  put((long long)A.hits, kHits);
  put((long long)A.missed, kMissed);
  put((long long)A.escaped, kEscaped);
  put((long long)A.capped, kCapped);
  put((long long)(A.missed + A.escaped + A.capped), kRays);
  put((long long)(A.hits + A.missed + A.escaped), kSegments);
  put(wave_sum_uniform(A.sE), kSE);
  put(wave_sum_uniform(A.sE2), kSE2);
  put((long long)A.tr_capped, kTrCap);
  put((long long)A.guard, kGuard);
  if (TOTALS && TOT_LDS) {
    long long t[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) t[c] = (long long)wave_tot[c * kWaves + (threadIdx.x >> 6)];
#pragma unroll
    for (int c = 0; c < 7; ++c) put(t[c], kFx + c);
    if (lead)  // after every lane of the wave has read them (one wave: LDS in program order)
#pragma unroll
      for (int c = 0; c < 7; ++c) wave_tot[c * kWaves + (threadIdx.x >> 6)] = 0ull;
  } else if (TOTALS) {
#pragma unroll
    for (int c = 0; c < 7; ++c) put(wave_sum_uniform(A.tot[c]), kFx + c);
  }
}

// ---------------------------------------------------------------------------
// a6-a9, plain path: particles read from the SoA.  Each loop iteration advances
// every traversing lane by one BVH step.  Lanes whose segment has ended wait
// until fewer than a.refill lanes are still traversing; then all of them are
// served at once (re-emission, tallies, the next segment, or the wave's next
// particle), so the costly per-hit work runs with many lanes active and no lane
// idles for the rest of a segment's traversal.  A wave has a share of
// consecutive particles, and the lanes that need one take the next ones in
// order, so that a load of the SoA covers whole cache lines and each line is
// fetched once.  With a particle per lane and grid stride every lane was at
// another stride, a line for each: 1e6 particles on a plate 416 us, 52 now; 3e6
// on a cylinder 649, 296 now.
// ---------------------------------------------------------------------------
// Workgroups of a query of n particles in a launch of max_groups a query: a
// particle per lane while they suffice (four per lane at least took 162 us for
// 1e5 particles on the 1280-triangle sphere, on 98 of 256 compute units; 83 so,
// with one traversal step a round).
__host__ __device__ __forceinline__ uint64_t plain_groups(uint64_t n, uint32_t max_groups) {
  const uint64_t g = (n + kBlock - 1) / kBlock;
  return g < max_groups ? g : max_groups;
}

template <int STACK, int MODE, bool COUNT>
__global__ __launch_bounds__(kBlock) void trace_kernel(TraceArgs a) {
  __shared__ int stk[STACK][kBlock];
  extern __shared__ unsigned long long lt[];  // tallies in LDS, sized at launch (tally_lds_bytes)
  const QueryDev& q = a.qs[blockIdx.y];
  const uint64_t groups = plain_groups(q.N, gridDim.x);
  if (blockIdx.x >= groups || (q.per_tri != 0u) != (MODE != kTallyTotals)) return;
  const uint32_t group = blockIdx.y * gridDim.x + blockIdx.x;  // group % 8: the XCD
  long long* const g_tally =
      (a.tally_copies.base ? a.tally_copies.base + (group & ((1u << a.tally_copies.log2) - 1u)) * a.tally_copies.stride
                           : a.tally) + q.tally_offset;
  int32_t* const first_tri = a.first_tri ? a.first_tri + q.p_offset : nullptr;
  if (MODE == kTallyLds) {
    for (uint32_t i = threadIdx.x; i < a.nt * 7u; i += kBlock) lt[i] = 0ull;
    __syncthreads();
  }
  if (MODE == kTallyLane)
    for (int c = 0; c < 2 * 7; ++c) lt[c * kBlock + threadIdx.x] = 0ull;
  Acc A;
  acc_zero(A);
  const uint32_t max_steps = 2u * a.nt + 64u;
  uint64_t next, end;  // the wave's particles not yet taken (uniform)
  {
    const uint64_t waves = groups * kWaves, share = q.N / waves, rest = q.N % waves;
    const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + (threadIdx.x >> 6));
    next = share * w + (w < rest ? w : rest);
    end = next + share + (w < rest ? 1u : 0u);
  }
  Lane L;
  Seg s;
  Ray r;
  seg_begin(s);
  auto load = [&](Lane& l) {
    const uint64_t i = q.p_offset + l.pid;
    l.ox = a.x[0][i]; l.oy = a.x[1][i]; l.oz = a.x[2][i];
    l.wx = a.w[0][i]; l.wy = a.w[1][i]; l.wz = a.w[2][i];
    l.D = 0.0f;
    l.E = 0.0f;
    l.prev = -1;
    l.hits = 0;
  };
  L.pid = next + (threadIdx.x & 63u);
  L.live = L.pid < end;
  next += 64;
  s.cur = kDone;
  if (L.live) {
    load(L);
    seg_begin(s);
  }
  make_ray(r, L.ox, L.oy, L.oz, L.wx, L.wy, L.wz);
  uint32_t guard = 0;  // steps since the last service pass (wave-uniform)
  while (ballot(L.live) != 0ull) {
    uint32_t ntrav = (uint32_t)__popcll(ballot(L.live && seg_traversing(s)));
    if (ntrav < a.refill && ballot(L.live && s.p0 >= 0) != 0ull) {
      leaf_phase<COUNT>(a.tris, a.orig, r, L.prev, s, A.tests);
      ntrav = (uint32_t)__popcll(ballot(L.live && seg_traversing(s)));
    }
    if (ntrav < a.refill) {
      const bool fin = L.live && seg_finished(s);
      if (ballot(fin) != 0ull) {
        Hit h;
        h.valid = false;
        int out = kOutGoOn;
        int32_t fid = -2;
        bool limited = false;
        if (fin) out = finish_segment(a.tris, a.orig, q, L, s, h, fid, limited);
        count_pass(A, fin, out, h.valid, limited);
        tally<MODE, STACK, false>(q, h, g_tally, lt, stk, A);
        if (fin && first_tri && fid != -2) first_tri[L.pid] = fid;
        const bool take = fin && out != kOutGoOn;
        const uint64_t taken = ballot(take);
        if (take) {
          retire(q, L, A);
          L.pid = next + below(taken);
          L.live = L.pid < end;
          if (L.live) load(L);
        }
        next += (uint32_t)__popcll(taken);
        if (fin && L.live) seg_begin(s);
      }
      make_ray(r, L.ox, L.oy, L.oz, L.wx, L.wy, L.wz);
      guard = 0;
    }
    // Between service passes every traversing lane ends its segment within
    // nt - 1 steps and nt leaf phases; the bound only keeps a damaged tree
    // from spinning a wave, and every segment it ends is counted.
    if (++guard > max_steps) {  // rounds: none takes more than the steps
      A.guard += lanes(L.live && s.cur != kDone);
      s.cur = kDone;
    }
    if (L.live && seg_traversing(s))
      trav_step<STACK, COUNT>(a.nodes, a.tris, a.orig, r, L.prev, s, stk, A.nodes, A.tests);
    // a second step before the next round of checks: they are a chain of scalar
    // and vector work that the step's loads do not overlap (satellite of 2e4
    // triangles, 1e6 particles 637 -> 555 us; sphere 1e5 83 -> 70; cylinder 3e6
    // 297 -> 278); 4-slot trees end within one
    if (STACK >= 16 && L.live && seg_traversing(s))
      trav_step<STACK, COUNT>(a.nodes, a.tris, a.orig, r, L.prev, s, stk, A.nodes, A.tests);
  }
  flush_acc(A, a.copies.base ? a.copies.base + (((uint64_t)blockIdx.y << a.copies.log2) +
                                                (group & ((1u << a.copies.log2) - 1u))) * kScalStride
                             : a.scal + q.scalar_offset, MODE == kTallyTotals);
  if (MODE == kTallyLane) flush_lane_tally(lt, g_tally, a.nt);
  if (COUNT) {
    const long long nn = wave_sum((long long)A.nodes), nt2 = wave_sum((long long)A.tests);
    if ((threadIdx.x & 63) == 0) {
      atomic_add_i64(reinterpret_cast<long long*>(a.counters), nn);
      atomic_add_i64(reinterpret_cast<long long*>(a.counters) + 1, nt2);
    }
  }
  if (MODE == kTallyLds) {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < a.nt * 7u; i += kBlock)
      if (lt[i]) atomic_add_i64(g_tally + i, (long long)lt[i]);
  }
}

// ---------------------------------------------------------------------------
// a11: persistent batched kernel.  A wave claims units of one part of a work
// entry (a query, or a range of its tiles) until the part is used up, then
// moves to another part with work left.  It draws 64 particles at a time from
// its unit and seeds them with every lane active (the FP64 seeding is the
// costliest per-particle step) into a wave-private LDS queue; the
// traversal advances one BVH step per iteration as in the plain path, and when
// fewer than a.refill lanes are still traversing, the lanes whose segment has
// ended are served together and lanes whose particle retired take the next
// queued particle.  Particle states never leave the chip.  Partial sums --
// per-lane scalars, per-lane LDS tallies of tiny meshes, the workgroup's
// LDS tally of meshes up to kLdsTallyMaxTris triangles -- stay on chip while
// the workgroup stays on one query and are flushed to HBM with atomics only
// when it changes query or finishes.  Per-particle arithmetic is the plain
// path's, so results match it bit for bit.
// ---------------------------------------------------------------------------

// Seeding in two stages (precull_may_enter) in every instance whose LDS
// leaves room for the survivor rings (not the 64-slot stack).
template <int STACK, int MODE>
constexpr bool kPrecullInstance = STACK <= 32;

// Work is claimed per wave in units of whole 64-particle batches (tpmc_units.hpp): a
// wave's lanes draw particles from its own unit, and when the unit runs out
// while lanes are still busy the wave goes on with another unit of the same
// part instead of draining (lanes in flight keep their absolute particle ids),
// so waves drain only when their part is used up.  Where no tally state is
// shared by the workgroup's waves (global atomics, per-lane LDS tallies, the
// waves' own totals) each wave also chooses its parts alone and never waits
// for the others; with workgroup LDS tallies the workgroup chooses the part
// together and its waves meet at a barrier only when they leave it (the
// tallies are flushed then).
template <int MODE>
constexpr bool kWaveEntries = MODE == kTallyGlobal || MODE == kTallyLane || MODE == kTallyTotals;

constexpr uint32_t kNoEntry = 0xFFFFFFFFu;

// Whether the launch's parts have workgroups that start on them (a whole batch).
__device__ __forceinline__ bool starts_own(const BatchArgs& a) { return (a.start.own | a.start.div) != 0u; }

// The cut of a part into units (tpmc_units.hpp).
__device__ __forceinline__ UnitPlan unit_plan(const BatchArgs& a, uint32_t part) {
  const uint32_t j = part >> a.sub_log2, i = part & ((1u << a.sub_log2) - 1u);
  const uint64_t N = a.qs[a.entry_query ? a.entry_query[j] : j].N;
  const uint64_t e0 = a.entry_tile0 ? a.entry_tile0[j] * a.tile : 0ull;
  uint64_t e1 = a.entry_tiles ? e0 + a.entry_tiles[j] * a.tile : N;
  if (e1 > N) e1 = N;
  const uint64_t ns = (uint64_t)start_groups(a.start, part) * (uint32_t)kWaves;
  return unit_plan_of(e0, e1 > e0 ? e1 - e0 : 0ull, a.sub_log2, i, ns, a.share_log2, a.unit_cap_log2, a.start_cap_log2);
}

// Claim a counted unit of the part (one atomic by lane 0; uniform result).
__device__ __forceinline__ bool claim_counted(const BatchArgs& a, uint32_t part, const UnitPlan& p, uint64_t& b,
                                              uint64_t& e) {
  if (p.ns_end >= p.n) return false;  // starting units only
  unsigned long long t = 0;
  if ((threadIdx.x & 63) == 0) t = atomicAdd(&a.entry_next[part], 1ull);
  t = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)t) |
      ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(t >> 32)) << 32);
  const bool ok = counted_unit(p, t, b, e);
  b += p.lo;
  e += p.lo;
  return ok;
}

// Find a part with counted units left, from part `scan` on, and claim one: 64
// parts are looked at per step, one per lane (called by a whole wave; uniform
// result, kNoEntry when there is none).  A failed claim on a part means that
// it was used up meanwhile.  Where every part has waves that started on it
// (they stay until it is used up), its last units, below kJoinMin particles, are
// left to them: taking up another query, draining and flushing cost more than
// such a unit (kJoinMin 64 / 256 / 512 / 1024: plate sweep 2.17 / 2.10 / 2.06 /
// 2.00 ms, cylinder sweep 6.91 / 6.84 / 6.72 / 6.73).
constexpr uint64_t kJoinMin = 1024;
__device__ __forceinline__ uint32_t claim_any(const BatchArgs& a, uint32_t scan, uint64_t& b, uint64_t& e) {
  const uint32_t parts = a.n_entries << a.sub_log2, lane = threadIdx.x & 63u;
  for (uint32_t k = 0; k < parts; k += 64u) {
    uint32_t part = scan + k + lane;
    if (part >= parts) part -= parts;
    bool has = false;
    if (k + lane < parts) {
      const UnitPlan p = unit_plan(a, part);
      uint64_t x, y;
      has = counted_unit(p, __hip_atomic_load(&a.entry_next[part], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), x, y);
      has = has && (!starts_own(a) || y - x >= kJoinMin);
    }
    uint64_t m = ballot(has);
    while (m != 0ull) {
      uint32_t c = scan + k + (uint32_t)__builtin_ctzll(m);
      m &= m - 1ull;
      if (c >= parts) c -= parts;
      if (claim_counted(a, c, unit_plan(a, c), b, e)) return c;
    }
  }
  return kNoEntry;
}

// The workgroup's place in the dealing of parts.  Workgroups are ordered by XCD, then (where
// the grid fills whole rounds of them) by compute unit, and the parts dealt to
// them in that order, so that a compute unit's waves work on one query or few:
// its rows of the latitude table (10 KB in reach of a query) stay in the
// 32 KB L1.  (The hardware deals workgroups to the XCDs in turn, and within
// an XCD to its compute units in turn; only speed depends on it.)
__device__ __forceinline__ uint32_t dealt_place(const BatchArgs& a) {
  const uint32_t G = gridDim.x, x = blockIdx.x & 7u, y = blockIdx.x >> 3;
  const uint32_t rem8 = G & 7u, cus = a.xcd_cus;
  uint32_t i = x * (G >> 3) + (x < rem8 ? x : rem8);
  if (rem8 == 0u && (G >> 3) % cus == 0u) i += (y % cus) * ((G >> 3) / cus) + y / cus;
  else i += y;
  return i;
}

// The lane's particle of a batch.  Units begin at multiples of 64, so a batch
// shares the high word of its particles' numbers, and the first rounds of
// their Philox blocks are half scalar.
__device__ __forceinline__ uint64_t batch_pid(uint64_t base) {
  return (base & 0xFFFFFFFF00000000ull) | ((uint32_t)base + (threadIdx.x & 63u));
}

// Where the workgroup's waves add a query's sums: the query's block, or one of
// its copies (ScalCopies).
__device__ __forceinline__ long long* scal_block(const BatchArgs& a, uint32_t query, const QueryDev& q) {
  if (a.copies.base == nullptr) return a.scal_base + q.scalar_offset;
  return a.copies.base + (((uint64_t)query << a.copies.log2) + (blockIdx.x & ((1u << a.copies.log2) - 1u))) * kScalStride;
}

// Where the workgroup's waves add a query's per-triangle sums.
__device__ __forceinline__ long long* tally_block(const BatchArgs& a, const QueryDev& q) {
  if (!q.per_tri) return nullptr;
  long long* const base = a.tally_copies.base
                              ? a.tally_copies.base + (blockIdx.x & ((1u << a.tally_copies.log2) - 1u)) * a.tally_copies.stride
                              : a.tally_base;
  return base + q.tally_offset;
}

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32);
}

template <int STACK, int MODE>
__global__ __launch_bounds__(kBlock) PROBE(__attribute__((amdgpu_waves_per_eu(STACK <= 32 && MODE != kTallyAuto ? 4 : 1)))) void batch_kernel(BatchArgs a) {
  constexpr bool kMayLds = MODE == kTallyLds || MODE == kTallyAuto;
  constexpr bool kPre = kPrecullInstance<STACK, MODE>;
  constexpr bool kWave = kWaveEntries<MODE>;
  constexpr uint32_t kSteps = STACK >= 32 ? 2u : 1u;  // traversal steps per round of the trace loop
  constexpr uint32_t kNone = kNoEntry;
  constexpr uint32_t kRing = 128;  // survivors of the estimate awaiting exact seeding (< 64 + 64)
  __shared__ int stk[STACK][kBlock];
  __shared__ float qbuf[kBlock / 64][6][64];
  // queue slot -> particle: its offset in its seeding batch, or (two-stage
  // seeding) in the wave's unit
  __shared__ uint8_t qlane[kPre ? 1 : kBlock / 64][64];
  __shared__ uint16_t qoff[kPre ? kBlock / 64 : 1][64];
  __shared__ uint16_t ring[kPre ? kBlock / 64 : 1][kPre ? kRing : 1];  // survivor offsets in the unit
  extern __shared__ unsigned long long lt[];  // tallies in LDS, sized at launch (tally_lds_bytes)
  // per-wave totals [c][wave]: the start of lt, or after the per-triangle area in the mixed mode
  unsigned long long* const wave_tot = MODE == kTallyAuto ? lt + 7u * a.lds_tris : lt;
  __shared__ unsigned long long unit_sh[2];         // wave 0's claimed unit of the workgroup's part
  __shared__ unsigned long long w_next_sh[kWaves];  // each wave's next unclaimed particle
  __shared__ uint32_t part_sh;
  // each wave's starting parts, in LDS rather than in registers through the trace
  // loop: next and end of its own, the shared one (or kNone) and its rank there
  __shared__ uint32_t own_sh[kWaves][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // where the workgroup's waves look for work: its own parts first
  uint32_t scan;
  if (starts_own(a)) {
    const uint32_t i = dealt_place(a);
    uint32_t part = kNone, rank = 0u;
    if (a.start.div != 0u) start_shared(a.start, i, part, rank);
    scan = i * a.start.own;
    if (lane == 0) {
      own_sh[wave][0] = scan;
      own_sh[wave][1] = scan + a.start.own;
      own_sh[wave][2] = part;
      own_sh[wave][3] = rank;
    }
  } else {
    if (lane == 0) {
      own_sh[wave][0] = own_sh[wave][1] = 0u;
      own_sh[wave][2] = kNone;
    }
    const uint32_t x = blockIdx.x & 7u, lo = a.xcd_start[x], hi = a.xcd_start[x + 1];
    scan = (hi > lo ? lo + (blockIdx.x >> 3) % (hi - lo) : lo) << a.sub_log2;
    scan += (blockIdx.x >> 3) & ((1u << a.sub_log2) - 1u);
  }
  uint32_t held = kNone;                     // entry whose partial sums the wave (and workgroup) holds
  Acc A;
  acc_zero(A);
  PROBE(uint32_t pr = 0u; probe_set<kPrTs>(pr, probe_now()); probe_set<kPrTc>(pr, probe_get(pr, kPrTs));)
  // two-stage seeding, wave-uniform: particles the estimate removed (for the
  // held query), and the estimate's yield so far on it.  A wave that finds
  // more than 60 % of a query's particles surviving the estimate (of at least
  // one batch) stops using it while it stays on the query, since the estimate
  // then costs more than it saves.  Every wave finds out for itself: a flag shared by the
  // launch cost more than the first batches it spared (4096 waves storing to
  // one word take 125 us, measured).  Next to the threshold little depends on it:
  // decided after 64 or 256 particles, launches whose estimate keeps 45 to 62 %
  // differ by 1.5 % at most (a sphere in a CV of 1.7 to 2.4 radii, a cylinder).
  uint64_t pre = 0;
  uint32_t pc_seen = 0, pc_kept = 0;
  auto yields_little = [&]() { return pc_seen >= 64u && 5u * pc_kept > 3u * pc_seen; };
  if (MODE == kTallyLane)
    for (int c = 0; c < 2 * 7; ++c) lt[c * kBlock + threadIdx.x] = 0ull;
  if (MODE == kTallyTotals || (MODE == kTallyAuto && a.wave_totals)) {
    if (kWave) {  // each wave its own slots (no barrier before its first tally)
      if (lane < 7) wave_tot[lane * kWaves + wave] = 0ull;
    } else if (threadIdx.x < 7u * kWaves) {
      wave_tot[threadIdx.x] = 0ull;
    }
  }
  for (;;) {
    uint32_t part;
    uint64_t p_begin = 0, p_end = 0;  // the wave's unit
    bool have = true;                 // the wave holds a unit of the part
    __builtin_amdgcn_wave_barrier();
    const uint32_t wv = __builtin_amdgcn_readfirstlane(wave);
    uint32_t own = __builtin_amdgcn_readfirstlane(own_sh[wv][0]), rank = 0u;
    const bool alone = own != __builtin_amdgcn_readfirstlane(own_sh[wv][1]);
    if (!alone) own = __builtin_amdgcn_readfirstlane(own_sh[wv][2]);
    if (own != kNone) {
      // the wave's starting unit of its next starting part; where the part is too
      // small to have one for the workgroup, it has no counted units either
      if (!alone) rank = __builtin_amdgcn_readfirstlane(own_sh[wv][3]);
      if (lane == 0) own_sh[wv][alone ? 0 : 2] = alone ? own + 1u : kNone;
      scan = own;
      const UnitPlan p = unit_plan(a, scan);
      const uint64_t u = rank * (uint32_t)kWaves + wv;
      const uint64_t b = u << p.s_log2, e = (u + 1ull) << p.s_log2;
      const bool any = kWave ? b < p.n : ((uint64_t)(rank * (uint32_t)kWaves) << p.s_log2) < p.n;
      part = any ? scan : kNone;
      have = b < p.n;
      p_begin = p.lo + b;
      p_end = p.lo + (e < p.n ? e : p.n);
      if (part == kNone) continue;
    } else if (kWave) {
      part = claim_any(a, scan, p_begin, p_end);
      if (part != kNone) scan = part;
    } else {
      if (__builtin_amdgcn_readfirstlane(wave) == 0) {  // the workgroup's part, and wave 0's first unit of it
        part = claim_any(a, scan, p_begin, p_end);
        if (lane == 0) {
          part_sh = part;
          unit_sh[0] = p_begin;
          unit_sh[1] = p_end;
        }
      }
      __syncthreads();
      part = __builtin_amdgcn_readfirstlane(part_sh);  // uniform over the workgroup
      p_begin = uniform_u64(unit_sh[0]);
      p_end = uniform_u64(unit_sh[1]);
      if (part != kNone) {
        scan = part;
        // the waves share the claimed unit in whole batches
        const uint64_t each = (((p_end - p_begin + 3ull) >> 2) + 63ull) & ~63ull;
        const uint64_t first = p_begin + (uint32_t)__builtin_amdgcn_readfirstlane(wave) * each;
        have = first < p_end;
        p_begin = first;
        p_end = first + each < p_end ? first + each : p_end;
      }
    }
    // wave-uniform: kept in scalar registers
    p_begin = uniform_u64(p_begin);
    p_end = uniform_u64(p_end);
    part = __builtin_amdgcn_readfirstlane(part);
    scan = __builtin_amdgcn_readfirstlane(scan);
    const uint32_t j = part == kNone ? kNone : part >> a.sub_log2;
    if (j != held && held != kNone) {
      // leaving the held query: flush its partial sums
      const uint32_t hq = a.entry_query ? a.entry_query[held] : held;
      const QueryDev& qh = a.qs[hq];
      long long* const hscal = scal_block(a, hq, qh);
      long long* htally = tally_block(a, qh);
      flush_acc<MODE == kTallyTotals || MODE == kTallyAuto>(
          A, hscal, MODE == kTallyTotals || (MODE == kTallyAuto && !qh.per_tri), wave_tot);
      if (MODE == kTallyLane) flush_lane_tally(lt, htally, qh.nt);
      acc_zero(A);
      if (kPre) {
        if (lane == 0 && pre != 0) atomic_add_i64(hscal + kPreculled, (long long)pre);
        pre = 0;
        pc_seen = pc_kept = 0;
      }
      if (kMayLds && qh.per_tri && qh.nt <= (uint32_t)kLdsTallyMaxTris)
        for (uint32_t i = threadIdx.x; i < qh.nt * 7u; i += kBlock)
          if (lt[i]) atomic_add_i64(htally + i, (long long)lt[i]);
    }
    if (j == kNone) break;  // uniform (the last claim's cycles are not in the claim slot)
    const QueryDev& q = a.qs[a.entry_query ? a.entry_query[j] : j];
    const bool use_lds = kMayLds && q.per_tri && q.nt <= (uint32_t)kLdsTallyMaxTris;
    if (j != held) {
      if (!kWave) __syncthreads();  // the flush above has read lt
      if (use_lds) {
        for (uint32_t i = threadIdx.x; i < q.nt * 7u; i += kBlock) lt[i] = 0ull;
        __syncthreads();  // cleared before any wave tallies into it
      }
      held = j;
    }
    if (lane == 0) w_next_sh[wave] = p_begin;  // the next unclaimed particle of the wave's unit
    long long* qtally = tally_block(a, q);
    const Node* nodes = uniform_ptr(q.nodes);
    const TriRec* tris = uniform_ptr(q.tris);
    const uint32_t* orig = uniform_ptr(q.orig);
    PROBE(probe_since<kPrClaimCyc>(pr, kPrTc); probe_add<kPrClaims>(pr, 1u);)
    // next 64 particle ids of the wave's unit
    auto claim64 = [&]() -> uint64_t {
      const uint64_t b = uniform_u64(w_next_sh[wave]);
      if (lane == 0) w_next_sh[wave] = b + 64u;
      return b;
    };

    Lane L;
    Seg s;
    Ray r;
    L.live = false;
    seg_begin(s);
    s.cur = kDone;
    const uint32_t max_steps = __builtin_amdgcn_readfirstlane(2u * q.nt + 64u);
    uint32_t guard = 0;                // steps since the last service pass (wave-uniform)
    bool exhausted = !have;            // wave-uniform: the unit has no particles left to claim
    bool dry = !have;                  // wave-uniform: the part has no units left
    uint32_t q_head = 0, q_count = 0;  // wave-uniform queue state
    uint64_t q_pid0 = 0;               // particle id of queue slot 0
    uint32_t s_head = 0, s_count = 0;  // wave-uniform survivor ring state (two-stage seeding)
    bool pc_on = kPre && q.estimate != 0u && !yields_little();  // wave-uniform
    for (;;) {
      uint32_t ntrav = (uint32_t)__popcll(ballot(L.live && seg_traversing(s)));
      if (ntrav < a.refill && ballot(L.live && s.p0 >= 0) != 0ull) {
        PROBE(probe_set<kPrTp>(pr, probe_now()); probe_add<kPrLeafPasses>(pr, 1u);
              probe_add<kPrLeafLanes>(pr, (uint32_t)lanes(L.live && s.p0 >= 0));)
        uint32_t n1 = 0;
        leaf_phase<false>(tris, orig, r, L.prev, s, n1);
        ntrav = (uint32_t)__popcll(ballot(L.live && seg_traversing(s)));
        PROBE(probe_since<kPrLeafCyc>(pr, kPrTp);)
      }
      if (ntrav < a.refill) {
        // serve every lane whose segment has ended
        const bool fin = L.live && seg_finished(s);
        if (ballot(fin) != 0ull) {
          PROBE(probe_set<kPrTp>(pr, probe_now()); probe_add<kPrServes>(pr, 1u);
                probe_add<kPrServeLanes>(pr, (uint32_t)lanes(fin));)
          Hit h;
          h.valid = false;
          int out = kOutGoOn;
          int32_t fid;
          bool limited = false;
          if (fin) out = finish_segment(tris, orig, q, L, s, h, fid, limited);
          count_pass(A, fin, out, h.valid, limited);
          if (use_lds) tally<kTallyLds, STACK>(q, h, qtally, lt, stk, A);
          else tally<MODE, STACK>(q, h, qtally, wave_tot, stk, A);
          if (fin) {
            if (out != kOutGoOn) {
              retire(q, L, A);
              L.live = false;
            } else {
              seg_begin(s);
            }
          }
          PROBE(probe_since<kPrServeCyc>(pr, kPrTp);)
        }
        const uint64_t dead = ballot(!L.live);
        if (dead != 0ull && exhausted && !dry && q_count == 0 && s_count == 0) {
          // the unit is used up (survivor ring and queue empty, so no offset refers to it):
          // go on with the part's next unit while the other lanes are still busy
          if (claim_counted(a, part, unit_plan(a, part), p_begin, p_end)) {
            if (lane == 0) w_next_sh[wave] = p_begin;
            exhausted = false;
            PROBE(probe_add<kPrClaims>(pr, 1u);)
          } else {
            dry = true;
          }
        }
        if (kPre && dead != 0ull) {
          while (q_count == 0 && !(exhausted && s_count == 0)) {  // wave-uniform
            if (s_count < 64 && !exhausted) {
              // stage 1: claim 64 particles, keep those the estimate cannot rule out
              PROBE(probe_set<kPrTp>(pr, probe_now());)
              const uint64_t base = claim64();
              if (base >= p_end) {
                exhausted = true;
              } else {
                const uint64_t pid = batch_pid(base);
                const bool valid = pid < p_end;
                bool maybe = valid;
                if (valid && pc_on) maybe = precull_may_enter(q, g_lat_fine, q.lat_own, g_vn_start, pid);
                const uint64_t mb = ballot(maybe);
                if (maybe) ring[wave][(s_head + s_count + below(mb)) & (kRing - 1)] =
                    (uint16_t)(pid - p_begin);
                const uint32_t nvalid = (uint32_t)__popcll(ballot(valid)), nmaybe = (uint32_t)__popcll(mb);
                s_count += nmaybe;
                pre += nvalid - nmaybe;
                A.missed += nvalid - nmaybe;
                pc_seen += nvalid;
                pc_kept += nmaybe;
                pc_on = pc_on && !yields_little();
                PROBE(probe_add<kPrEstBatches>(pr, 1u); probe_add<kPrEstLanes>(pr, nvalid);
                      probe_add<kPrEstKept>(pr, nmaybe);)
                __builtin_amdgcn_wave_barrier();
              }
              PROBE(probe_since<kPrEstCyc>(pr, kPrTp);)
            } else {
            // stage 2: exact seeding of up to 64 survivors, one per lane; the
            // exact root test as in the one-stage seeding below
            const uint32_t n = s_count < 64u ? s_count : 64u;
            PROBE(probe_set<kPrTp>(pr, probe_now());)
            bool keep = false;
            float xs[3], ws[3];
            if ((uint32_t)lane < n) {
              double x[3], w[3];
              seed_particle(q, g_lat_start, g_lat_fine, q.lat_own, g_vn_start, g_sc_tab, g_ee_tab,
                            p_begin + ring[wave][(s_head + lane) & (kRing - 1)], x, w);
#pragma unroll
              for (int c = 0; c < 3; ++c) {
                xs[c] = (float)x[c];
                ws[c] = (float)w[c];
              }
              keep = STACK <= 4 || ray_enters_root(nodes, xs, ws);
            }
            A.missed += lanes((uint32_t)lane < n && !keep);
            const uint64_t kb = ballot(keep);
            if (keep) {
              const uint32_t slot = below(kb);
#pragma unroll
              for (int c = 0; c < 3; ++c) {
                qbuf[wave][c][slot] = xs[c];
                qbuf[wave][3 + c][slot] = ws[c];
              }
              qoff[wave][slot] = ring[wave][(s_head + lane) & (kRing - 1)];  // read again: not held across the seeding
            }
            s_head += n;
            s_count -= n;
            q_count = (uint32_t)__popcll(kb);
            q_head = 0;
            PROBE(probe_since<kPrSeedCyc>(pr, kPrTp); probe_add<kPrSeedBatches>(pr, 1u);
                  probe_add<kPrSeedLanes>(pr, n); probe_add<kPrSeedKept>(pr, q_count);)
            __builtin_amdgcn_wave_barrier();
            }
          }
        }
        if (!kPre && dead != 0ull) {
          while (q_count == 0 && !exhausted) {  // wave-uniform
            // claim and seed the next (up to) 64 particles, one per lane
            PROBE(probe_set<kPrTp>(pr, probe_now());)
            const uint64_t base = claim64();
            if (base >= p_end) {
              exhausted = true;
            } else {
              // Seed; a particle whose first ray misses both boxes of the root
              // node would end its first traversal step with no hit, so it is
              // counted as missed here and only the others are queued (trees
              // deeper than a 4-slot stack: there it spares the lane its idle
              // wait for the next service pass; in tiny trees every step ends
              // at leaves and the test would only add work).
              const uint64_t pid = base + lane;
              bool keep = false;
              float xs[3], ws[3];
              if (pid < p_end) {
                double x[3], w[3];
                seed_particle(q, g_lat_start, g_lat_fine, q.lat_own, g_vn_start, g_sc_tab, g_ee_tab, pid, x, w);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                  xs[c] = (float)x[c];
                  ws[c] = (float)w[c];
                }
                keep = STACK <= 4 || ray_enters_root(nodes, xs, ws);
              }
              A.missed += lanes(pid < p_end && !keep);
              const uint64_t kb = ballot(keep);
              if (keep) {
                const uint32_t slot = below(kb);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                  qbuf[wave][c][slot] = xs[c];
                  qbuf[wave][3 + c][slot] = ws[c];
                }
                qlane[wave][slot] = (uint8_t)lane;
              }
              q_count = (uint32_t)__popcll(kb);
              q_head = 0;
              q_pid0 = base;
              PROBE(probe_add<kPrSeedBatches>(pr, 1u); probe_add<kPrSeedLanes>(pr, (uint32_t)lanes(pid < p_end));
                    probe_add<kPrSeedKept>(pr, q_count);)
              __builtin_amdgcn_wave_barrier();
            }
            PROBE(probe_since<kPrSeedCyc>(pr, kPrTp);)
          }
        }
        if (dead != 0ull) {
          if (q_count > 0) {
            // dead lanes take queue entries in lane order
            PROBE(probe_set<kPrTp>(pr, probe_now());)
            const uint32_t rank = below(dead);
            if (!L.live && rank < q_count) {
              const uint32_t slot = q_head + rank;
              L.ox = qbuf[wave][0][slot]; L.oy = qbuf[wave][1][slot]; L.oz = qbuf[wave][2][slot];
              L.wx = qbuf[wave][3][slot]; L.wy = qbuf[wave][4][slot]; L.wz = qbuf[wave][5][slot];
              L.pid = kPre ? p_begin + qoff[wave][slot] : q_pid0 + qlane[wave][slot];
              L.D = 0.0f;
              L.E = 0.0f;
              L.prev = -1;
              L.hits = 0;
              L.live = true;
              seg_begin(s);
            }
            const uint32_t ndead = __popcll(dead);
            const uint32_t took = ndead < q_count ? ndead : q_count;
            q_head += took;
            q_count -= took;
            PROBE(probe_since<kPrAssignCyc>(pr, kPrTp); probe_add<kPrAssigns>(pr, 1u);
                  probe_add<kPrAssignLanes>(pr, took);)
            __builtin_amdgcn_wave_barrier();
          }
        }
        // nothing in flight and nothing left: the wave is done with the part.  It
        // stays until the part is dry (with no lane live but particles or units
        // left, the next iteration claims more): others may leave the part's
        // last units to it (claim_any).
        if (ballot(L.live) == 0ull && dry && exhausted && q_count == 0 && s_count == 0) break;
        make_ray(r, L.ox, L.oy, L.oz, L.wx, L.wy, L.wz);
        guard = 0;
      }
      // as in the plain path: a bound only against a damaged tree, counted
      if ((guard += kSteps) > kSteps * max_steps) {
        A.guard += lanes(L.live && s.cur != kDone);
        s.cur = kDone;
      }
      PROBE(const uint32_t nl = (uint32_t)lanes(L.live && seg_traversing(s)); probe_add<kPrTravLanes>(pr, nl);
            probe_add<kPrTravSteps>(pr, nl != 0u ? 1u : 0u); probe_set<kPrTp>(pr, probe_now());)
      if (L.live && seg_traversing(s)) {
        uint32_t n0 = 0, n1 = 0;
        trav_step<STACK, false>(nodes, tris, orig, r, L.prev, s, stk, n0, n1);
      }
      // deep trees (32-slot stacks): a second step before the next round of checks
      // (refill, leaf phase, guard), whose cost there is worth sparing for every
      // other step (attitude sweep -2.4 %, satellite -1.2 %; neutral on shallow trees)
      PROBE(if (kSteps == 2) {
        const uint32_t nl2 = (uint32_t)lanes(L.live && seg_traversing(s));
        probe_add<kPrTravLanes>(pr, nl2);
        probe_add<kPrTravSteps>(pr, nl2 != 0u ? 1u : 0u);
      })
      if (kSteps == 2 && L.live && seg_traversing(s)) {
        uint32_t n0 = 0, n1 = 0;
        trav_step<STACK, false>(nodes, tris, orig, r, L.prev, s, stk, n0, n1);
      }
      PROBE(probe_since<kPrTravCyc>(pr, kPrTp);)
    }
    PROBE(probe_set<kPrTc>(pr, probe_now());)
    if (!kWave) __syncthreads();  // every wave is done with the part; part_sh / unit_sh may be reused
  }
  PROBE(probe_set<kPrWaves>(pr, 1u); probe_set<kPrCycles>(pr, probe_now() - probe_get(pr, kPrTs));
        if (lane < kProbeSlots) atomicAdd(&g_probe[lane], (unsigned long long)pr);)
}

// ---------------------------------------------------------------------------
// a10: reduction and finalisation
// ---------------------------------------------------------------------------
constexpr int kReduceChunk = 1024;  // triangles per workgroup

// The workgroup's sums of triangles [t0, t1) over `copies` copies, `stride`
// words apart: sum k for thread k < 7 (the others get 0).
__device__ __forceinline__ long long sum_triangles(const long long* __restrict__ tally, uint32_t copies, uint64_t stride,
                                                   uint32_t t0, uint32_t t1) {
  __shared__ long long part[kBlock / 64][7];
  long long s[7] = {0, 0, 0, 0, 0, 0, 0};
  // (triangle, copy) pairs over the lanes, so that small meshes with many copies use them all
  const uint32_t items = (t1 - t0) * copies;
  for (uint32_t i = threadIdx.x; i < items; i += kBlock) {
    const uint32_t c = i / (t1 - t0), t = t0 + i % (t1 - t0);
#pragma unroll
    for (int k = 0; k < 7; ++k) s[k] += tally[c * stride + 7ull * t + k];
  }
#pragma unroll
  for (int c = 0; c < 7; ++c) s[c] = wave_sum(s[c]);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int c = 0; c < 7; ++c) part[threadIdx.x >> 6][c] = s[c];
  __syncthreads();
  long long v = 0;
  if (threadIdx.x < 7)
    for (int w = 0; w < kBlock / 64; ++w) v += part[w][threadIdx.x];
  return v;
}

// One query's triangles [chunk], added to its totals.
__device__ __forceinline__ void reduce_one(const long long* __restrict__ tally, uint32_t copies, uint64_t stride,
                                           uint32_t nt, long long* __restrict__ scal, uint32_t chunk) {
  const uint32_t t0 = chunk * kReduceChunk;
  const uint32_t t1 = t0 + kReduceChunk < nt ? t0 + kReduceChunk : nt;
  const long long v = sum_triangles(tally, copies, stride, t0, t1);
  if (threadIdx.x < 7 && v) atomic_add_i64(scal + kFx + threadIdx.x, v);
}

__global__ __launch_bounds__(kBlock) void reduce_batch_kernel(const QueryDev* __restrict__ qs,
                                                              long long* __restrict__ tally_base, TallyCopies copies,
                                                              long long* __restrict__ scal_base) {
  const QueryDev& q = qs[blockIdx.y];
  if (!q.per_tri || blockIdx.x * (uint32_t)kReduceChunk >= q.nt) return;
  const long long* const base = copies.base ? copies.base : tally_base;
  reduce_one(base + q.tally_offset, copies.base ? 1u << copies.log2 : 1u, copies.stride, q.nt,
             scal_base + q.scalar_offset, blockIdx.x);
}

__global__ __launch_bounds__(kBlock) void fold_tally_kernel(long long* __restrict__ tally, TallyCopies copies) {
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < copies.stride; i += (uint64_t)gridDim.x * kBlock) {
    long long v = 0;
    for (uint32_t c = 0; c < (1u << copies.log2); ++c) {
      v += copies.base[c * copies.stride + i];
      copies.base[c * copies.stride + i] = 0;
    }
    tally[i] += v;
  }
}

// F/q = K sum(w - w'), K = 2 Gamma_hat / (N S^2) (eq. drag with the effective
// mass of Sec. II.A); moment about x_ref from the moment about the CV centre.
__device__ __forceinline__ ResultDev converted(const QueryDev& q, const long long* s, double xr, double yr, double zr,
                                               double A_ref) {
  const double N = (double)q.N;
  double F[3], Lc[3];
  for (int k = 0; k < 3; ++k) {
    F[k] = (double)s[kFx + k] * q.inv_scaleF;
    Lc[k] = (double)s[kLx + k] * q.inv_scaleL;
  }
  const double cx = q.c0[0] - xr, cy = q.c0[1] - yr, cz = q.c0[2] - zr;
  const double M[3] = {Lc[0] + (cy * F[2] - cz * F[1]), Lc[1] + (cz * F[0] - cx * F[2]), Lc[2] + (cx * F[1] - cy * F[0])};
  const double nan = __builtin_nan("");
  const double K = q.s_zero ? nan : 2.0 * q.Gamma_hat / (N * q.S * q.S);
  ResultDev r;
  for (int k = 0; k < 3; ++k) {
    r.F_over_q[k] = K * F[k];
    r.M_over_q[k] = K * M[k];
    r.Fhat[k] = q.Gamma_hat / N * F[k];
    r.Mhat[k] = q.Gamma_hat / N * M[k];  // M / (rho c_mp^2), finite at S = 0
  }
  r.CD = (r.F_over_q[0] * q.U[0] + r.F_over_q[1] * q.U[1] + r.F_over_q[2] * q.U[2]) / A_ref;
  const double meanD = (double)s[kSD] * q.inv_scaleD / N;
  double varD = (double)s[kSD2] * q.inv_scaleD2 / N - meanD * meanD;
  if (varD < 0.0) varD = 0.0;
  r.CD_sigma = q.s_zero ? nan : 2.0 * q.Gamma_hat / (q.S * q.S * A_ref) * sqrt(varD / N);
  r.Gamma_hat = q.Gamma_hat;
  // energy: power Q = n c_mp (m c_mp^2 / 2) (Gamma_hat / N) sum E, and
  // C_H = Q / (rho U^3 A_ref / 2) = Gamma_hat sum E / (N S^3 A_ref)
  const double meanE = (double)s[kSE] * q.inv_scaleE / N;
  double varE = (double)s[kSE2] * q.inv_scaleE2 / N - meanE * meanE;
  if (varE < 0.0) varE = 0.0;
  const double S3 = q.S * q.S * q.S;
  r.Qhat = q.Gamma_hat * meanE;
  r.CH = q.s_zero ? nan : q.Gamma_hat * meanE / (S3 * A_ref);
  r.CH_sigma = q.s_zero ? nan : q.Gamma_hat / (S3 * A_ref) * sqrt(varE / N);
  r.rays = (uint64_t)s[kRays];
  r.hits = (uint64_t)s[kHits];
  r.segments = (uint64_t)s[kSegments];
  r.missed = (uint64_t)s[kMissed];
  r.escaped = (uint64_t)s[kEscaped];
  r.capped = (uint64_t)s[kCapped];
  r.tr_capped = (uint64_t)s[kTrCap];
  r.guard_trips = (uint64_t)s[kGuard];
  r.preculled = (uint64_t)s[kPreculled];
  return r;
}

// One workgroup per query: thread (c, k) adds up slot k of copies c, c + 8, ...
// (consecutive words, so a copy is one load of half a wave), thread 0 converts.
// Meshes of at most kFinalizeTris triangles are summed here too (a launch of
// its own took 4.6 us and the clearing of the totals before a plain run's as much;
// 1280 triangles add 2 us here).
__global__ __launch_bounds__(kBlock) void finalize_kernel(const QueryDev* __restrict__ qs,
                                                          const uint32_t* __restrict__ idx,
                                                          const long long* __restrict__ scal_base, ScalCopies copies,
                                                          const long long* __restrict__ tally_base, TallyCopies tc,
                                                          double xr, double yr, double zr, double A_ref,
                                                          ResultDev* __restrict__ out) {
  constexpr uint32_t kRows = kBlock / kScalStride;
  __shared__ long long part[kRows][kScalStride], s[kScalStride];
  __shared__ ResultDev rs;
  const uint32_t i = blockIdx.x, j = idx ? idx[i] : i;
  const QueryDev& q = qs[j];
  const uint32_t k = threadIdx.x % kScalStride, row = threadIdx.x / kScalStride;
  long long v = row == 0 && k < (uint32_t)kScalarSlots ? scal_base[q.scalar_offset + k] : 0;
  if (copies.base) {
    const long long* c = copies.base + ((uint64_t)j << copies.log2) * kScalStride + k;
#pragma unroll 8
    for (uint32_t r = row; r < (1u << copies.log2); r += kRows) v += c[(uint64_t)r * kScalStride];
  }
  part[row][k] = v;
  long long tri = 0;  // thread c < 7: the query's total c
  if (tally_base && q.per_tri) {
    const long long* const base = tc.base ? tc.base : tally_base;
    tri = sum_triangles(base + q.tally_offset, tc.base ? 1u << tc.log2 : 1u, tc.stride, 0, q.nt);
  }
  __syncthreads();
  if (threadIdx.x < (uint32_t)kScalStride) {
    v = 0;
    for (uint32_t r = 0; r < kRows; ++r) v += part[r][threadIdx.x];
    s[threadIdx.x] = v;
  }
  __syncthreads();
  if (threadIdx.x < 7) s[kFx + threadIdx.x] += tri;
  __syncthreads();
  if (threadIdx.x == 0) rs = converted(q, s, xr, yr, zr, A_ref);
  __syncthreads();
  // one store of consecutive words (out may be host memory)
  const uint64_t* const src = reinterpret_cast<const uint64_t*>(&rs);
  uint64_t* const dst = reinterpret_cast<uint64_t*>(out + i);
  if (threadIdx.x < (uint32_t)(sizeof(ResultDev) / 8)) dst[threadIdx.x] = src[threadIdx.x];
}

// Dynamic LDS of the tallies: the workgroup tally of lds_tris triangles, the
// per-lane slots of <= 2-triangle meshes, or per-wave totals (persistent
// kernel only; the plain kernel keeps totals in registers); the mixed mode
// of serving steps holds both a workgroup tally and per-wave totals.
size_t tally_lds_bytes(TallyMode mode, uint32_t lds_tris, bool persistent, bool wave_totals = false) {
  switch (mode) {
    case kTallyLds: return (size_t)lds_tris * 7 * sizeof(unsigned long long);
    case kTallyAuto:  // per-triangle area, then (persistent, if any entry keeps totals only) the per-wave totals
      return ((size_t)lds_tris * 7 + (persistent && wave_totals ? (size_t)7 * kWaves : 0)) * sizeof(unsigned long long);
    case kTallyLane: return (size_t)2 * 7 * kBlock * sizeof(unsigned long long);
    case kTallyTotals: return persistent ? (size_t)7 * kWaves * sizeof(unsigned long long) : 0;
    default: return 0;
  }
}

template <int STACK, bool COUNT>
void launch_trace_mode(const TraceArgs& a, TallyMode mode, dim3 grid, hipStream_t st) {
  const size_t lds = tally_lds_bytes(mode, a.nt, false);
  switch (mode) {
    case kTallyGlobal: trace_kernel<STACK, kTallyGlobal, COUNT><<<grid, kBlock, lds, st>>>(a); break;
    case kTallyLds: trace_kernel<STACK, kTallyLds, COUNT><<<grid, kBlock, lds, st>>>(a); break;
    case kTallyLane: trace_kernel<STACK, kTallyLane, COUNT><<<grid, kBlock, lds, st>>>(a); break;
    default: trace_kernel<STACK, kTallyTotals, COUNT><<<grid, kBlock, lds, st>>>(a); break;
  }
}

template <int STACK>
void launch_trace_stack(const TraceArgs& a, TallyMode mode, dim3 grid, hipStream_t st) {
  if (a.counters) launch_trace_mode<STACK, true>(a, mode, grid, st);
  else launch_trace_mode<STACK, false>(a, mode, grid, st);
}

template <int STACK>
void launch_batch_mode(const BatchArgs& a, TallyMode mode, int grid, hipStream_t st) {
  const size_t lds = tally_lds_bytes(mode, a.lds_tris, true, a.wave_totals != 0u);
  switch (mode) {
    case kTallyLane: batch_kernel<STACK, kTallyLane><<<grid, kBlock, lds, st>>>(a); break;
    case kTallyLds: batch_kernel<STACK, kTallyLds><<<grid, kBlock, lds, st>>>(a); break;
    case kTallyTotals: batch_kernel<STACK, kTallyTotals><<<grid, kBlock, lds, st>>>(a); break;
    case kTallyAuto: batch_kernel<STACK, kTallyAuto><<<grid, kBlock, lds, st>>>(a); break;
    default: batch_kernel<STACK, kTallyGlobal><<<grid, kBlock, lds, st>>>(a); break;
  }
}

static_assert(sizeof(QueryDev) % 8 == 0 && kScalarSlots <= kBlock, "admission copies 8-byte words");

// Serving admission, entry blockIdx.y: the slot's constants and cleared
// scalar block (first workgroup), its per-triangle tally words (all).
__global__ __launch_bounds__(kBlock) void admit_kernel(const AdmitRec* __restrict__ rec, QueryDev* __restrict__ qs,
                                                       long long* __restrict__ scal, ScalCopies copies,
                                                       float* __restrict__ lat_rows, long long* __restrict__ tally) {
  const AdmitRec& r = rec[blockIdx.y];
  if (blockIdx.x == 0) {
    const uint64_t* src = reinterpret_cast<const uint64_t*>(&r.q);
    uint64_t* dst = reinterpret_cast<uint64_t*>(qs + r.slot);
    for (uint32_t w = threadIdx.x; w < sizeof(QueryDev) / 8; w += kBlock) dst[w] = src[w];
    if (threadIdx.x < (uint32_t)kScalarSlots) scal[(uint64_t)r.slot * kScalarSlots + threadIdx.x] = 0;
    if (copies.base)
      for (uint32_t w = threadIdx.x; w < (uint32_t)kScalStride << copies.log2; w += kBlock)
        copies.base[(((uint64_t)r.slot << copies.log2) * kScalStride) + w] = 0;
  }
  if (r.q.lat_own)
    for (int j = blockIdx.x * kBlock + threadIdx.x; j < kLatFNT; j += gridDim.x * kBlock)
      lat_rows[(uint64_t)r.slot * kLatOwnStride + j] = latitude_row(r.q, g_lat_fine, j);
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < r.tally_words; i += (uint64_t)gridDim.x * kBlock)
    tally[r.tally_off + i] = 0;
}

}  // namespace

void launch_admit(const AdmitRec* rec, uint32_t n, uint64_t max_words, QueryDev* qs, long long* scal,
                  const ScalCopies& copies, float* lat_rows, long long* tally, hipStream_t st) {
  const uint64_t gx = std::max<uint64_t>((max_words + kBlock - 1) / kBlock, (kLatFNT + kBlock - 1) / kBlock);
  const dim3 g((uint32_t)(gx < 1 ? 1 : (gx > 1024 ? 1024 : gx)), n);
  admit_kernel<<<g, kBlock, 0, st>>>(rec, qs, scal, copies, lat_rows, tally);
}

// Check of the two-stage seeding's estimate: over particles [0, n) of one
// query, the largest distance between the estimated and the exact ray as a
// fraction of the margin (out[0], the bits of a non-negative double: they
// order as integers), and the number of particles the estimate covered
// (out[1]).  Distance = |o_est - o| + 2 r |w_est / |w_est| - w / |w||: how
// far apart the two rays can get along the at most 2 r of path in the CV.
__global__ __launch_bounds__(kBlock) void precull_check_kernel(const QueryDev* __restrict__ qp, uint64_t n,
                                                               unsigned long long* __restrict__ out) {
  const QueryDev& q = *qp;
  double worst = 0.0;
  unsigned long long cnt = 0;
  for (uint64_t pid = (uint64_t)blockIdx.x * kBlock + threadIdx.x; pid < n; pid += (uint64_t)gridDim.x * kBlock) {
    float o[3], w[3];
    if (!precull_estimate(q, g_lat_fine, nullptr, g_vn_start, pid, o, w)) continue;
    double x[3], we[3];
    seed_particle(q, g_lat_start, g_lat_fine, nullptr, g_vn_start, g_sc_tab, g_ee_tab, pid, x, we);
    double dp = 0.0, nw = 0.0, ne = 0.0, dd = 0.0;
    for (int c = 0; c < 3; ++c) {
      dp += ((double)o[c] - x[c]) * ((double)o[c] - x[c]);
      nw += (double)w[c] * (double)w[c];
      ne += we[c] * we[c];
    }
    nw = sqrt(nw);
    ne = sqrt(ne);
    for (int c = 0; c < 3; ++c) dd += ((double)w[c] / nw - we[c] / ne) * ((double)w[c] / nw - we[c] / ne);
    const double ratio = (sqrt(dp) + 2.0 * q.r * sqrt(dd)) / ((double)kPrecullMargin * q.r);
    worst = ratio == ratio ? fmax(worst, ratio) : __builtin_inf();  // a NaN estimate counts as unbounded
    ++cnt;
  }
  atomicMax(out, (unsigned long long)__double_as_longlong(worst));
  atomicAdd(out + 1, cnt);
}

void launch_precull_check(const QueryDev* d_q, uint64_t n, unsigned long long* out, int grid, hipStream_t st) {
  zero_i64_kernel<<<1, kBlock, 0, st>>>(reinterpret_cast<long long*>(out), 2);
  precull_check_kernel<<<grid, kBlock, 0, st>>>(d_q, n, out);
}

#if TPMC_PHASE_PROBE
bool probe_built() { return true; }

hipError_t probe_read(unsigned long long* out, bool reset, hipStream_t st) {
  unsigned long long* d = nullptr;
  hipError_t e = hipGetSymbolAddress((void**)&d, HIP_SYMBOL(g_probe));
  if (e == hipSuccess) e = hipMemcpyAsync(out, d, kProbeSlots * sizeof(unsigned long long), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess && reset) {
    zero_i64_kernel<<<1, kBlock, 0, st>>>(reinterpret_cast<long long*>(d), kProbeSlots);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  return e;
}
#else
bool probe_built() { return false; }

hipError_t probe_read(unsigned long long*, bool, hipStream_t) { return hipErrorNotSupported; }
#endif

hipError_t init_seed_tables(hipStream_t st) {
  float* tab = nullptr;
  float* lat = nullptr;
  float* fine = nullptr;
  double* sc = nullptr;
  double* ee = nullptr;
  hipError_t e = hipGetSymbolAddress((void**)&tab, HIP_SYMBOL(g_vn_start));
  if (e == hipSuccess) e = hipGetSymbolAddress((void**)&lat, HIP_SYMBOL(g_lat_start));
  if (e == hipSuccess) e = hipGetSymbolAddress((void**)&fine, HIP_SYMBOL(g_lat_fine));
  if (e == hipSuccess) e = hipGetSymbolAddress((void**)&sc, HIP_SYMBOL(g_sc_tab));
  if (e == hipSuccess) e = hipGetSymbolAddress((void**)&ee, HIP_SYMBOL(g_ee_tab));
  if (e != hipSuccess) return e;
  sc_table_kernel<<<1, 256, 0, st>>>(sc);
  ee_table_kernel<<<(kExpErfcN + 255) / 256, 256, 0, st>>>(ee);  // before the solves that read it
  vn_table_kernel<<<(kVnNS * kVnNT + 255) / 256, 256, 0, st>>>(tab, ee);
  lat_table_kernel<<<(kLatNS * kLatNT + 255) / 256, 256, 0, st>>>(lat, ee);
  lat_fine_kernel<<<(kLatFNS * kLatFNT + 255) / 256, 256, 0, st>>>(fine, ee);
  e = hipGetLastError();
  return e != hipSuccess ? e : hipStreamSynchronize(st);
}

void launch_lat_own(const QueryDev* d_qs, uint32_t nq, float* rows, hipStream_t st) {
  lat_own_kernel<<<dim3((kLatFNT + kBlock - 1) / kBlock, nq), kBlock, 0, st>>>(d_qs, rows);
}

void zero_i64(long long* p, uint64_t n, hipStream_t st) {
  if (n) zero_i64_kernel<<<grid_for(n, 4096), kBlock, 0, st>>>(p, n);
}

void clear_ranges(const ClearRanges& r, hipStream_t st) {
  uint64_t n = 0;
  for (int k = 0; k < kClearRanges; ++k) n = std::max(n, r.n[k]);
  if (n) clear_kernel<<<grid_for(n, 4096), kBlock, 0, st>>>(r);
}

void clear_and_upload(const ClearRanges& r, const QueryDev* h_qs, QueryDev* d_qs, uint32_t n, hipStream_t st) {
  uint64_t most = 1;
  for (int k = 0; k < kClearRanges; ++k) most = std::max(most, r.n[k]);
  ArgQueries h;
  std::memcpy(static_cast<void*>(&h), h_qs, n * sizeof(QueryDev));
  std::memset(reinterpret_cast<char*>(&h) + n * sizeof(QueryDev), 0, (kArgQueries - n) * sizeof(QueryDev));
  clear_upload_kernel<<<grid_for(most, 4096), kBlock, 0, st>>>(r, h, d_qs, n);
}

void zero_u32(uint32_t* p, uint64_t n, hipStream_t st) {
  if (n) zero_u32_kernel<<<grid_for(n, 4096), kBlock, 0, st>>>(p, n);
}

int stack_slots_for_depth(uint32_t depth) {
  if (depth <= 4) return 4;
  if (depth <= 8) return 8;
  if (depth <= 16) return 16;
  if (depth <= 32) return 32;
  if (depth <= 64) return 64;
  return 0;
}

void launch_seed(const QueryDev* d_qs, uint32_t nq, uint64_t max_n, float* const planes[6], int n_cu, hipStream_t st) {
  const uint64_t g = std::min<uint64_t>((max_n + kBlock - 1) / kBlock, (uint64_t)n_cu * 16);
  Planes p;
  for (int k = 0; k < 6; ++k) p.p[k] = planes[k];
  seed_kernel<<<dim3((uint32_t)std::max<uint64_t>(g, 1), nq), kBlock, 0, st>>>(d_qs, p);
}

void launch_trace(const TraceArgs& a, uint32_t nq, uint64_t max_n, int stack_slots, TallyMode mode, int max_grid,
                  hipStream_t st) {
  const dim3 grid((uint32_t)std::max<uint64_t>(plain_groups(max_n, (uint32_t)max_grid), 1), nq);
  switch (stack_slots) {
    case 4: launch_trace_stack<4>(a, mode, grid, st); break;
    case 8: launch_trace_stack<8>(a, mode, grid, st); break;
    case 16: launch_trace_stack<16>(a, mode, grid, st); break;
    case 32: launch_trace_stack<32>(a, mode, grid, st); break;
    default: launch_trace_stack<64>(a, mode, grid, st); break;
  }
}

void launch_batch(BatchArgs a, int stack_slots, TallyMode mode, uint64_t total_particles, bool uniform,
                  uint64_t counters, int n_cu, int groups_per_cu, hipStream_t st) {
  // workgroups resident per CU: at most four (four waves per SIMD, every instance
  // has at most 128 VGPRs), and what 160 KB of LDS holds
  const size_t lds = tally_lds_bytes(mode, a.lds_tris, true, a.wave_totals != 0u) + (size_t)stack_slots * kBlock * 4 +
                     (stack_slots <= 32 ? kBatchLdsPrecull : kBatchLds);
  const int resident = std::max(1, std::min((int)((160u << 10) / lds), 4));
  const uint64_t batches = (total_particles + 63) / 64;
  uint64_t grid = (uint64_t)n_cu * (uint64_t)std::min(groups_per_cu, resident);
  // no more than there are batches for, or, where queries are smaller, a workgroup for each
  const uint64_t most = std::max<uint64_t>((batches + kWaves - 1) / kWaves, uniform ? a.n_entries : 1u);
  grid = std::max<uint64_t>(1, std::min<uint64_t>(grid, most));
  const uint64_t waves = grid * kWaves;
  a.sub_log2 = 0;
  if (!uniform || batches > waves)  // more than one batch per wave: units are claimed, from up to 16 counters
    while (((uint64_t)a.n_entries << (a.sub_log2 + 1)) <= std::min<uint64_t>(counters, 16)) ++a.sub_log2;
  const uint64_t parts = (uint64_t)a.n_entries << a.sub_log2;
  a.start = uniform ? start_plan_of((uint32_t)grid, (uint32_t)parts) : StartPlan{0u, 0u, 0u, 0u};
  a.xcd_cus = (uint32_t)std::max(1, n_cu / 8);
  a.share_log2 = 6;
  while ((waves << (a.share_log2 + 1)) <= total_particles) ++a.share_log2;
  // a workgroup's waves alone take the starting units of all its own parts: together at most a quarter of an equal
  // share (a whole one: 3000 queries of 100 to 300000 particles on a cylinder 14.7 ms, 12.9 so)
  a.start_cap_log2 = a.start.own == 0u ? 32u : a.share_log2 > 8u ? a.share_log2 - 8u : 0u;
  for (uint32_t m = a.start.own; m != 0u && a.start_cap_log2 != 0u; m >>= 1) --a.start_cap_log2;
  a.unit_cap_log2 = 0;
  while ((128u << a.unit_cap_log2) <= a.tile / 4 && a.unit_cap_log2 < 8) ++a.unit_cap_log2;
  switch (stack_slots) {
    case 4: launch_batch_mode<4>(a, mode, (int)grid, st); break;
    case 8: launch_batch_mode<8>(a, mode, (int)grid, st); break;
    case 16: launch_batch_mode<16>(a, mode, (int)grid, st); break;
    case 32: launch_batch_mode<32>(a, mode, (int)grid, st); break;
    default: launch_batch_mode<64>(a, mode, (int)grid, st); break;
  }
}

void launch_reduce_batch(const QueryDev* d_qs, uint32_t nq, long long* tally_base, const TallyCopies& copies,
                         long long* scal_base, uint32_t max_nt, hipStream_t st) {
  dim3 g((max_nt + kReduceChunk - 1) / kReduceChunk, nq);
  reduce_batch_kernel<<<g, kBlock, 0, st>>>(d_qs, tally_base, copies, scal_base);
}

void launch_fold_tally(long long* tally, const TallyCopies& copies, hipStream_t st) {
  fold_tally_kernel<<<grid_for(copies.stride, 4096), kBlock, 0, st>>>(tally, copies);
}

void launch_finalize(const QueryDev* d_qs, const uint32_t* d_idx, const long long* scal_base, const ScalCopies& copies,
                     const long long* tally_base, const TallyCopies& tally_copies, uint32_t nq, double xr, double yr,
                     double zr, double A_ref, ResultDev* out, hipStream_t st) {
  // in chunks: a launch holds fewer than 2^32 threads, 2^24 workgroups
  for (uint32_t i = 0; i < nq; i += kMaxFinalize) {
    ScalCopies c = copies;
    if (c.base && !d_idx) c.base += ((uint64_t)i << c.log2) * kScalStride;
    finalize_kernel<<<std::min(kMaxFinalize, nq - i), kBlock, 0, st>>>(d_idx ? d_qs : d_qs + i, d_idx ? d_idx + i : nullptr,
                                                                     scal_base, c, tally_base, tally_copies, xr, yr, zr,
                                                                     A_ref, out + i);
  }
}

// Per-triangle reduction of a list of slots (serving): entry y reduces slot idx[y].
__global__ __launch_bounds__(kBlock) void reduce_slots_kernel(const QueryDev* __restrict__ qs,
                                                              const uint32_t* __restrict__ idx,
                                                              long long* __restrict__ tally_base,
                                                              long long* __restrict__ scal_base) {
  const QueryDev& q = qs[idx[blockIdx.y]];
  if (!q.per_tri || blockIdx.x * (uint32_t)kReduceChunk >= q.nt) return;
  reduce_one(tally_base + q.tally_offset, 1u, 0u, q.nt, scal_base + q.scalar_offset, blockIdx.x);
}

// Clears slots kFx..kCount of the listed per-triangle queries before a reduction.
__global__ void clear_totals_kernel(const QueryDev* __restrict__ qs, const uint32_t* __restrict__ idx,
                                    long long* __restrict__ scal_base, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * 7u) return;
  const QueryDev& q = qs[idx ? idx[i / 7u] : i / 7u];
  if (q.per_tri) scal_base[q.scalar_offset + kFx + i % 7u] = 0;
}

void launch_reduce_slots(const QueryDev* d_qs, const uint32_t* d_idx, uint32_t n, long long* tally_base,
                         long long* scal_base, uint32_t max_nt, hipStream_t st) {
  clear_totals_kernel<<<(n * 7 + 255) / 256, 256, 0, st>>>(d_qs, d_idx, scal_base, n);
  dim3 g((max_nt + kReduceChunk - 1) / kReduceChunk, n);
  reduce_slots_kernel<<<g, kBlock, 0, st>>>(d_qs, d_idx, tally_base, scal_base);
}

void launch_reduce_totals(const QueryDev* d_qs, uint32_t nq, long long* tally_base, long long* scal_base,
                          uint32_t max_nt, hipStream_t st) {
  clear_totals_kernel<<<(nq * 7 + 255) / 256, 256, 0, st>>>(d_qs, nullptr, scal_base, nq);
  launch_reduce_batch(d_qs, nq, tally_base, TallyCopies{nullptr, 0, 0}, scal_base, max_nt, st);
}

}  // namespace tpmc
