// tpmc_bvh.hip -- linear BVH over the triangle mesh, built on the device.
//
// Closest-hit tracing on a triangulation (Sec. II.A) needs an acceleration
// structure; this is an LBVH: 30-bit Morton codes of triangle centroids, a
// stable LSD radix sort (4-bit digits, wave-ballot ranking), the binary radix
// tree of Karras (HPG 2012) and a bottom-up box refit with atomic flags.
// Triangles are then packed in Morton order for locality.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tpmc_device.hpp"
#include "tpmc_launch.h"
#include "tpmc_sah.hpp"

namespace tpmc {

namespace {

constexpr int kSortItems = 4;
constexpr int kSortTile = kBlock * kSortItems;

__device__ __forceinline__ uint32_t spread_bits10(uint32_t v) {
  v = (v * 0x00010001u) & 0xFF0000FFu;
  v = (v * 0x00000101u) & 0x0F00F00Fu;
  v = (v * 0x00000011u) & 0xC30C30C3u;
  v = (v * 0x00000005u) & 0x49249249u;
  return v;
}

__global__ void morton_kernel(const float* __restrict__ xyz, const uint32_t* __restrict__ tri, uint32_t nt, float lox,
                              float loy, float loz, float sx, float sy, float sz, uint32_t* __restrict__ keys,
                              uint32_t* __restrict__ vals) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nt) return;
  const uint32_t a = tri[3 * i], b = tri[3 * i + 1], c = tri[3 * i + 2];
  const float cx = (xyz[3 * a] + xyz[3 * b] + xyz[3 * c]) * (1.0f / 3.0f);
  const float cy = (xyz[3 * a + 1] + xyz[3 * b + 1] + xyz[3 * c + 1]) * (1.0f / 3.0f);
  const float cz = (xyz[3 * a + 2] + xyz[3 * b + 2] + xyz[3 * c + 2]) * (1.0f / 3.0f);
  const uint32_t qx = (uint32_t)fminf(fmaxf((cx - lox) * sx, 0.0f), 1023.0f);
  const uint32_t qy = (uint32_t)fminf(fmaxf((cy - loy) * sy, 0.0f), 1023.0f);
  const uint32_t qz = (uint32_t)fminf(fmaxf((cz - loz) * sz, 0.0f), 1023.0f);
  keys[i] = (spread_bits10(qx) << 2) | (spread_bits10(qy) << 1) | spread_bits10(qz);
  vals[i] = i;
}

// ---- stable LSD radix sort, 4-bit digits ----

__global__ void radix_count_kernel(const uint32_t* __restrict__ keys, uint32_t n, int shift,
                                   uint32_t* __restrict__ counts, uint32_t nblocks) {
  __shared__ uint32_t h[16];
  if (threadIdx.x < 16) h[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t base = blockIdx.x * kSortTile;
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    const uint32_t idx = base + j * kBlock + threadIdx.x;
    if (idx < n) atomicAdd(&h[(keys[idx] >> shift) & 15u], 1u);
  }
  __syncthreads();
  if (threadIdx.x < 16) counts[threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan of m entries by one workgroup of 1024 threads.
__global__ void __launch_bounds__(1024) scan_kernel(uint32_t* __restrict__ a, uint32_t m) {
  __shared__ uint32_t s[1024];
  __shared__ uint32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (uint32_t base = 0; base < m; base += 1024) {
    const uint32_t idx = base + threadIdx.x;
    const uint32_t v = idx < m ? a[idx] : 0u;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const uint32_t add = threadIdx.x >= (uint32_t)o ? s[threadIdx.x - o] : 0u;
      __syncthreads();
      s[threadIdx.x] += add;
      __syncthreads();
    }
    const uint32_t incl = s[threadIdx.x];
    if (idx < m) a[idx] = carry + incl - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry += incl;
    __syncthreads();
  }
}

__global__ void radix_scatter_kernel(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                     uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, uint32_t n, int shift,
                                     const uint32_t* __restrict__ offsets, uint32_t nblocks) {
  __shared__ uint32_t run[16];
  __shared__ uint32_t wc[kBlock / 64][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x < 16) run[threadIdx.x] = offsets[threadIdx.x * nblocks + blockIdx.x];
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const uint32_t base = blockIdx.x * kSortTile;
  for (int j = 0; j < kSortItems; ++j) {
    if (threadIdx.x < kBlock / 64 * 16) wc[threadIdx.x >> 4][threadIdx.x & 15] = 0;
    __syncthreads();
    const uint32_t idx = base + j * kBlock + threadIdx.x;
    const bool valid = idx < n;
    const uint32_t key = valid ? kin[idx] : 0u;
    const uint32_t d = (key >> shift) & 15u;
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint64_t bal = __ballot(valid && ((d >> b) & 1u));
      same &= ((d >> b) & 1u) ? bal : ~bal;
    }
    const uint32_t rank = __popcll(same & lt_mask);
    if (valid && rank == 0) wc[wave][d] = __popcll(same);
    __syncthreads();
    if (threadIdx.x < 16) {
      uint32_t r = run[threadIdx.x];
      for (int w = 0; w < kBlock / 64; ++w) {
        const uint32_t c = wc[w][threadIdx.x];
        wc[w][threadIdx.x] = r;
        r += c;
      }
      run[threadIdx.x] = r;
    }
    __syncthreads();
    if (valid) {
      const uint32_t pos = wc[wave][d] + rank;
      kout[pos] = key;
      vout[pos] = vin[idx];
    }
    __syncthreads();
  }
}

// ---- Karras (2012) binary radix tree over sorted unique keys ----

__device__ __forceinline__ int common_prefix(const uint32_t* __restrict__ k, int n, int i, int j) {
  if (j < 0 || j >= n) return -1;
  const uint32_t a = k[i], b = k[j];
  if (a == b) return 32 + __clz((uint32_t)(i ^ j));
  return __clz(a ^ b);
}

__global__ void karras_kernel(const uint32_t* __restrict__ keys, int n, Node* __restrict__ nodes,
                              int32_t* __restrict__ leaf_parent) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n - 1) return;
  const int d = (common_prefix(keys, n, i, i + 1) - common_prefix(keys, n, i, i - 1)) >= 0 ? 1 : -1;
  const int dmin = common_prefix(keys, n, i, i - d);
  int lmax = 2;
  while (common_prefix(keys, n, i, i + lmax * d) > dmin) lmax <<= 1;
  int l = 0;
  for (int t = lmax >> 1; t >= 1; t >>= 1)
    if (common_prefix(keys, n, i, i + (l + t) * d) > dmin) l += t;
  const int j = i + l * d;
  const int dnode = common_prefix(keys, n, i, j);
  int s = 0;
  int div = 2;
  int t;
  do {
    t = (l + div - 1) / div;
    if (common_prefix(keys, n, i, i + (s + t) * d) > dnode) s += t;
    div <<= 1;
  } while (t > 1);
  const int split = i + s * d + (d < 0 ? -1 : 0);
  const int lo = i < j ? i : j, hi = i < j ? j : i;
  int c0, c1;
  if (lo == split) {
    c0 = ~split;
    leaf_parent[split] = i;
  } else {
    c0 = split;
    nodes[split].parent = i;
  }
  if (hi == split + 1) {
    c1 = ~(split + 1);
    leaf_parent[split + 1] = i;
  } else {
    c1 = split + 1;
    nodes[split + 1].parent = i;
  }
  nodes[i].c0 = c0;
  nodes[i].c1 = c1;
  if (i == 0) nodes[0].parent = -1;
}

// Pack triangles in Morton order with their unit normals (computed in FP64).
__global__ void pack_tris_kernel(const float* __restrict__ xyz, const uint32_t* __restrict__ tri,
                                 const uint32_t* __restrict__ order, uint32_t nt, TriRec* __restrict__ recs,
                                 uint32_t* __restrict__ orig) {
  // Products evaluated without contraction: a component that is exactly zero
  // (e.g. a vertical face) stays zero instead of becoming an FMA residue whose
  // sign would choose a different tangent basis at re-emission.
#pragma clang fp contract(off)
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nt) return;
  const uint32_t id = order[k];
  const uint32_t a = tri[3 * id], b = tri[3 * id + 1], c = tri[3 * id + 2];
  TriRec r;
  r.v0x = xyz[3 * a]; r.v0y = xyz[3 * a + 1]; r.v0z = xyz[3 * a + 2];
  r.v1x = xyz[3 * b]; r.v1y = xyz[3 * b + 1]; r.v1z = xyz[3 * b + 2];
  r.v2x = xyz[3 * c]; r.v2y = xyz[3 * c + 1]; r.v2z = xyz[3 * c + 2];
  const double e1x = (double)r.v1x - r.v0x, e1y = (double)r.v1y - r.v0y, e1z = (double)r.v1z - r.v0z;
  const double e2x = (double)r.v2x - r.v0x, e2y = (double)r.v2y - r.v0y, e2z = (double)r.v2z - r.v0z;
  double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
  const double len = sqrt(nx * nx + ny * ny + nz * nz);
  const double inv = len > 0.0 ? 1.0 / len : 0.0;
  r.nx = (float)(nx * inv);
  r.ny = (float)(ny * inv);
  r.nz = (float)(nz * inv);
  recs[k] = r;
  orig[k] = id | 3u << 30;  // supporting-plane flags, cleared by support_kernel
}

// Supporting-plane flags, used to resolve the segment that leaves a hit
// without tracing it.  For triangle k (Morton order) with exact plane
// through v0 and normal n = (v1 - v0) x (v2 - v0) / |...|: bit 30 of orig[k]
// when no mesh vertex lies above the plane by more than tol, bit 31 when none
// lies below it by more than tol, tol = 2^-22 max|coordinate of triangle k|.
// A particle re-emitted from k leaves from a point 8 ulps of that scale (at
// least 5 once the rounding of the hit point is counted) above the plane on
// its emission side and moves away from the plane (or parallel to it), so
// when the mesh lies within tol of the other side, the outgoing ray cannot hit
// anything: every mesh point is below its starting height.  FP64 distances;
// pack_tris_kernel sets both bits, a vertex found on a side clears that side's.
//
// Two passes.  The first looks at 256 vertices spread over the whole mesh, a
// triangle per lane; on a concave body most triangles have vertices on both
// sides among them and are done.  The rest -- about the facets of the convex
// hull -- are listed, and the second pass runs over their (four triangles,
// 4096 vertices) pairs, a wave each with the lanes over the vertices.  Bound:
// FP64 issue of the second pass.  One lane per triangle over all vertices took
// 900 us on the 50k-triangle satellite (196 workgroups, no early end) and 55 ms
// on the 500k one.  Up to kSupportAll vertices the first pass looks at all of them
// and is the only one: the second's launch and the list's clearing cost as much (LBVH
// builds of 64 soup triangles 226 us with them, 202 without, 642 sphere vertices 279
// and 272).
struct SupportPlane {
  double ox, oy, oz, nx, ny, nz, tol;
  bool area;  // zero-area triangles are never hit and keep no flag
};

__device__ __forceinline__ SupportPlane support_plane(const TriRec& t) {
  SupportPlane p;
  p.ox = t.v0x, p.oy = t.v0y, p.oz = t.v0z;
  const double e1x = (double)t.v1x - p.ox, e1y = (double)t.v1y - p.oy, e1z = (double)t.v1z - p.oz;
  const double e2x = (double)t.v2x - p.ox, e2y = (double)t.v2y - p.oy, e2z = (double)t.v2z - p.oz;
  p.nx = e1y * e2z - e1z * e2y, p.ny = e1z * e2x - e1x * e2z, p.nz = e1x * e2y - e1y * e2x;
  const double len = sqrt(p.nx * p.nx + p.ny * p.ny + p.nz * p.nz);
  p.area = len != 0.0;
  const double inv = len > 0.0 ? 1.0 / len : 0.0;
  p.nx *= inv;
  p.ny *= inv;
  p.nz *= inv;
  const float sc = fmaxf(fmaxf(fmaxf(fabsf(t.v0x), fabsf(t.v0y)), fmaxf(fabsf(t.v0z), fabsf(t.v1x))),
                         fmaxf(fmaxf(fabsf(t.v1y), fabsf(t.v1z)), fmaxf(fmaxf(fabsf(t.v2x), fabsf(t.v2y)), fabsf(t.v2z))));
  p.tol = ldexp((double)sc, -22);
  return p;
}

__device__ __forceinline__ double support_distance(const SupportPlane& p, float x, float y, float z) {
  return p.nx * ((double)x - p.ox) + p.ny * ((double)y - p.oy) + p.nz * ((double)z - p.oz);
}

// orig word without the flags of the sides that have a vertex
__device__ __forceinline__ uint32_t support_keep(bool above, bool below) {
  return ~((above ? 1u << 30 : 0u) | (below ? 1u << 31 : 0u));
}

constexpr uint32_t kSupportAll = 1024, kSupportSpread = 256, kSupportSegment = 4096, kSupportTris = 4;

__global__ __launch_bounds__(kBlock) void support_spread_kernel(const float* __restrict__ xyz, uint32_t nv,
                                                                const TriRec* __restrict__ tris, uint32_t nt,
                                                                uint32_t* __restrict__ orig,
                                                                uint32_t* __restrict__ list,
                                                                uint32_t* __restrict__ n_list,
                                                                const Node* __restrict__ nodes,
                                                                const uint32_t* __restrict__ depth,
                                                                BuildRead* __restrict__ read) {
  __shared__ float v[kSupportAll][3];
  if (blockIdx.x == 0) {  // what the host reads of the build, side by side for one copy
    const uint32_t* const root = reinterpret_cast<const uint32_t*>(nodes);
    uint32_t* const out = reinterpret_cast<uint32_t*>(&read->root);
    if (threadIdx.x < sizeof(Node) / 4u) out[threadIdx.x] = root[threadIdx.x];
    else if (threadIdx.x == sizeof(Node) / 4u) read->depth = depth ? *depth : 0u;
  }
  const uint32_t m = nv <= kSupportAll ? nv : kSupportSpread;
  for (uint32_t i = threadIdx.x; i < ((m + 15u) & ~15u); i += kBlock) {  // whole sixteens, with the last one again
    const uint64_t at = m == nv ? min(i, m - 1u) : (uint64_t)i * nv / m;
    v[i][0] = xyz[3 * at];
    v[i][1] = xyz[3 * at + 1];
    v[i][2] = xyz[3 * at + 2];
  }
  __syncthreads();
  const uint32_t k = blockIdx.x * kBlock + threadIdx.x;
  const bool on = k < nt;
  const SupportPlane p = support_plane(tris[on ? k : nt - 1u]);
  double hi = -__builtin_inf(), lo = __builtin_inf();
  // sixteen at a time, so that their loads overlap
  for (uint32_t j = 0; j < m; j += 16u) {
#pragma unroll
    for (uint32_t i = 0; i < 16u; ++i) {
      const double d = support_distance(p, v[j + i][0], v[j + i][1], v[j + i][2]);
      hi = fmax(hi, d);
      lo = fmin(lo, d);
    }
    if (__all(!on || !p.area || (hi > p.tol && lo < -p.tol))) break;
  }
  const bool above = !p.area || hi > p.tol, below = !p.area || lo < -p.tol;
  if (on && (above || below)) orig[k] &= support_keep(above, below);
  const bool more = on && !(above && below) && nv > m;
  const uint64_t mask = __ballot(more);
  uint32_t at = 0;
  if ((threadIdx.x & 63u) == 0u && mask != 0ull) at = atomicAdd(n_list, (uint32_t)__popcll(mask));
  at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
  if (more) list[at + (uint32_t)__popcll(mask & ((1ull << (threadIdx.x & 63u)) - 1ull))] = k;
}

__global__ __launch_bounds__(kBlock) void support_kernel(const float* __restrict__ xyz, uint32_t nv,
                                                         const TriRec* __restrict__ tris, uint32_t* __restrict__ orig,
                                                         const uint32_t* __restrict__ list,
                                                         const uint32_t* __restrict__ n_list) {
  const uint32_t n = *n_list, lane = threadIdx.x & 63u;
  const uint64_t segs = (nv + kSupportSegment - 1u) / kSupportSegment, items = (n + kSupportTris - 1u) / kSupportTris * segs;
  for (uint64_t it = (uint64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); it < items;
       it += (uint64_t)gridDim.x * (kBlock / 64)) {
    const uint32_t first = (uint32_t)(it / segs) * kSupportTris;
    const uint32_t v0 = (uint32_t)(it % segs) * kSupportSegment, v1 = min(nv, v0 + kSupportSegment);
    SupportPlane p[kSupportTris];
    double hi[kSupportTris], lo[kSupportTris];
#pragma unroll
    for (uint32_t c = 0; c < kSupportTris; ++c) {
      p[c] = support_plane(tris[list[min(first + c, n - 1u)]]);
      hi[c] = -__builtin_inf();
      lo[c] = __builtin_inf();
    }
    for (uint32_t i = v0 + lane; i < v1; i += 64u) {
      const float x = xyz[3ull * i], y = xyz[3ull * i + 1], z = xyz[3ull * i + 2];
#pragma unroll
      for (uint32_t c = 0; c < kSupportTris; ++c) {
        const double d = support_distance(p[c], x, y, z);
        hi[c] = fmax(hi[c], d);
        lo[c] = fmin(lo[c], d);
      }
    }
#pragma unroll
    for (uint32_t c = 0; c < kSupportTris; ++c) {
      const bool above = __any(hi[c] > p[c].tol), below = __any(lo[c] < -p[c].tol);
      if (lane == 0 && (above || below) && first + c < n) atomicAnd(&orig[list[first + c]], support_keep(above, below));
    }
  }
}

__device__ __forceinline__ float ld_relaxed(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void child_box(const Node* nodes, const float* nbox, const TriRec* tris, int c, float b[6]) {
  if (c < 0) {
    const TriRec& t = tris[~c];
    b[0] = fminf(fminf(t.v0x, t.v1x), t.v2x);
    b[1] = fminf(fminf(t.v0y, t.v1y), t.v2y);
    b[2] = fminf(fminf(t.v0z, t.v1z), t.v2z);
    b[3] = fmaxf(fmaxf(t.v0x, t.v1x), t.v2x);
    b[4] = fmaxf(fmaxf(t.v0y, t.v1y), t.v2y);
    b[5] = fmaxf(fmaxf(t.v0z, t.v1z), t.v2z);
  } else {
    for (int k = 0; k < 6; ++k) b[k] = ld_relaxed(nbox + 6 * c + k);
  }
}

// Bottom-up refit: one thread per leaf climbs; the second thread to reach a
// node writes its children's boxes and continues upward.
__global__ void refit_kernel(Node* __restrict__ nodes, const int32_t* __restrict__ leaf_parent,
                             const TriRec* __restrict__ tris, uint32_t nt, uint32_t* __restrict__ flags,
                             float* __restrict__ nbox) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nt) return;
  int p = leaf_parent[k];
  for (int level = 0; p >= 0 && level < 4096; ++level) {  // bounded climb
    __threadfence();
    if (atomicAdd(&flags[p], 1u) == 0u) return;
    __threadfence();
    const int c0 = __hip_atomic_load(&nodes[p].c0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int c1 = __hip_atomic_load(&nodes[p].c1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float b0[6], b1[6];
    child_box(nodes, nbox, tris, c0, b0);
    child_box(nodes, nbox, tris, c1, b1);
    Node& nd = nodes[p];
    nd.lo0x = b0[0]; nd.lo0y = b0[1]; nd.lo0z = b0[2]; nd.hi0x = b0[3]; nd.hi0y = b0[4]; nd.hi0z = b0[5];
    nd.lo1x = b1[0]; nd.lo1y = b1[1]; nd.lo1z = b1[2]; nd.hi1x = b1[3]; nd.hi1y = b1[4]; nd.hi1z = b1[5];
    for (int q = 0; q < 3; ++q) {
      __hip_atomic_store(nbox + 6 * p + q, fminf(b0[q], b1[q]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(nbox + 6 * p + 3 + q, fmaxf(b0[3 + q], b1[3 + q]), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    p = __hip_atomic_load(&nodes[p].parent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Depth of every leaf (root = depth 0), maximum kept.
__global__ void depth_kernel(const Node* __restrict__ nodes, const int32_t* __restrict__ leaf_parent, uint32_t nt,
                             uint32_t* __restrict__ max_depth) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nt) return;
  uint32_t dpt = 0;
  int p = leaf_parent[k];
  while (p >= 0 && dpt < 4096) {  // bounded climb
    ++dpt;
    p = nodes[p].parent;
  }
  atomicMax(max_depth, dpt);
}

// One-triangle mesh: a single node whose two links both name leaf 0.
__global__ void single_node_kernel(Node* nodes, const TriRec* tris) {
  const TriRec& t = tris[0];
  Node nd;
  nd.lo0x = nd.lo1x = fminf(fminf(t.v0x, t.v1x), t.v2x);
  nd.lo0y = nd.lo1y = fminf(fminf(t.v0y, t.v1y), t.v2y);
  nd.lo0z = nd.lo1z = fminf(fminf(t.v0z, t.v1z), t.v2z);
  nd.hi0x = nd.hi1x = fmaxf(fmaxf(t.v0x, t.v1x), t.v2x);
  nd.hi0y = nd.hi1y = fmaxf(fmaxf(t.v0y, t.v1y), t.v2y);
  nd.hi0z = nd.hi1z = fmaxf(fmaxf(t.v0z, t.v1z), t.v2z);
  nd.c0 = ~0;
  nd.c1 = ~0;
  nd.parent = -1;
  nd.pad = 0;
  nodes[0] = nd;
}


// ---- top-down binned SAH build ----
//
// Alternative to the Morton/Karras hierarchy, same node and leaf format.  A
// node's triangles (a contiguous range of an index array) are split where the
// surface-area heuristic (cost of a child = its box area x its triangle count)
// is lowest among kSahBins - 1 planes per axis, planes equally spaced over the
// range of the triangle box centres; the range is then partitioned stably into
// the other index array.  Internal node ids follow Karras's rule, valid for any
// binary tree over ordered leaves: the root is 0, an internal left child takes
// the position of its last triangle and an internal right child that of its
// first, so ids are known before the children are processed and the build is
// deterministic.  Below level kSahMaxLevel (or when every centre coincides)
// ranges are halved by position, so no leaf lies deeper than
// kSahMaxLevel + 30 <= 64 for nt < 2^30.
//
// Three stages by the size m of a node's range, each with its own split of the
// work (the tree is the same whichever does it):
//  * m > kSahBig: chunks of kSahChunk triangles, one workgroup each, bin into
//    the node's bins in global memory, one workgroup per node chooses the
//    plane, and the chunks partition (three launches per level).
//  * kSahWave < m <= kSahBig: one workgroup per node, one launch per level.
//  * m <= kSahWave: one wave builds the whole subtree in registers, a triangle
//    per lane.
// Bound: the length of the chain of levels (each launch 5 to 45 us, almost all
// latency), not the data.
// Task lists and their lengths stay on the device; the host reads them once
// everything has been enqueued.  With one workgroup per
// node and a host read per level, a 50k-triangle build spent 2.6 of its 3.2 ms
// of kernels in the top five levels (1 to 16 workgroups), and 0.7 ms waiting
// for the reads.  Whole builds of satellites, before and now: 1k triangles 0.69
// and 0.39 ms, 20k 2.25 and 0.66, 50k 4.9 and 1.05, 200k 24.6 and 2.1, 500k 81 and 4.4.
constexpr uint32_t kSahWave = 32;
constexpr uint32_t kSahBig = 1024;
constexpr uint32_t kSahChunk = 512;
static_assert(kSahBins == 32 && kSahWave <= 64, "sah_wave_kernel: a triangle per lane, 32 planes of two axes at a time");

struct SahTask {
  uint32_t a, b, id;  // triangle positions [a, b] (b > a), node id
  int32_t parent;
  uint32_t level;
  uint32_t buf;       // which index array holds the range
  uint32_t chunk0;    // first of its chunks (m > kSahBig)
  uint32_t nl;        // left count, axis and plane once chosen (m > kSahBig); nl 0: left to the next stage
  uint32_t ax, split;
  uint32_t child[2];  // list positions of its big children (kNoTask: none)
};
constexpr uint32_t kNoTask = 0xFFFFFFFFu;

// Bins of one big node: centre bounds (lo xyz, hi xyz as ordered ints), counts and box unions.
struct SahBins {
  int cb[6];
  uint32_t cnt[3][kSahBins];
  int lo[3][kSahBins][3], hi[3][kSahBins][3];
};

// List lengths and results, on the device.
struct SahState {
  uint32_t nbig[2], nchunk[2];
  uint32_t nmid[3];  // of mid-stage levels l mod 3: read, filled and emptied in turn
  uint32_t nsmall, depth, err;
};

__device__ __forceinline__ float box_area(float lx, float ly, float lz, float hx, float hy, float hz) {
  const float ex = hx - lx, ey = hy - ly, ez = hz - lz;
  return ex * ey + ey * ez + ez * ex;
}

// Cost of a plane: left boxes L (lo xyz, hi xyz as ordered ints) of nl triangles, right R of nr.
__device__ __forceinline__ float plane_cost(const int L[6], const int R[6], uint32_t nl, uint32_t nr) {
  return box_area(o2f(L[0]), o2f(L[1]), o2f(L[2]), o2f(L[3]), o2f(L[4]), o2f(L[5])) * (float)nl +
         box_area(o2f(R[0]), o2f(R[1]), o2f(R[2]), o2f(R[3]), o2f(R[4]), o2f(R[5])) * (float)nr;
}

__device__ __forceinline__ void empty_box(int b[6]) {
#pragma unroll
  for (int q = 0; q < 6; ++q) b[q] = f2o(q < 3 ? __builtin_inff() : -__builtin_inff());
}

__device__ __forceinline__ float3 box_centre(const float4& lo, const float4& hi) {
  return make_float3(0.5f * (lo.x + hi.x), 0.5f * (lo.y + hi.y), 0.5f * (lo.z + hi.z));
}

__device__ __forceinline__ Node make_node(const int L[6], const int R[6], int c0, int c1, int32_t parent) {
  Node nd;
  nd.lo0x = o2f(L[0]); nd.lo0y = o2f(L[1]); nd.lo0z = o2f(L[2]);
  nd.hi0x = o2f(L[3]); nd.hi0y = o2f(L[4]); nd.hi0z = o2f(L[5]);
  nd.lo1x = o2f(R[0]); nd.lo1y = o2f(R[1]); nd.lo1z = o2f(R[2]);
  nd.hi1x = o2f(R[3]); nd.hi1y = o2f(R[4]); nd.hi1z = o2f(R[5]);
  nd.c0 = c0;
  nd.c1 = c1;
  nd.parent = parent;
  nd.pad = 0;
  return nd;
}

// The children of T split after its first nl triangles (now in index array
// buf), as tasks: appended to the lists of their stages.
__device__ __forceinline__ void emit_children(const SahTask& T, uint32_t nl, uint32_t buf, SahTask* __restrict__ mid,
                                              uint32_t* __restrict__ nmid, SahTask* __restrict__ small,
                                              uint32_t* __restrict__ nsmall) {
  const uint32_t m = T.b - T.a + 1u;
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const uint32_t n = side == 0 ? nl : m - nl;
    if (n < 2u) continue;
    SahTask c{};
    c.a = side == 0 ? T.a : T.a + nl;
    c.b = side == 0 ? T.a + nl - 1u : T.b;
    c.id = side == 0 ? c.b : c.a;
    c.parent = (int32_t)T.id;
    c.level = T.level + 1u;
    c.buf = buf;
    if (n <= kSahWave) small[atomicAdd(nsmall, 1u)] = c;
    else mid[atomicAdd(nmid, 1u)] = c;
  }
}

// Triangle boxes (exact min / max of the FP32 vertices); the box centre is the
// binning key.  With bins, also the bounds of the centres into bins->cb.
__global__ __launch_bounds__(kBlock) void prim_box_kernel(const float* __restrict__ xyz,
                                                          const uint32_t* __restrict__ tri, uint32_t nt,
                                                          float4* __restrict__ plo, float4* __restrict__ phi,
                                                          uint32_t* __restrict__ idx, uint32_t* __restrict__ order,
                                                          SahBins* __restrict__ bins);

__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fminf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

__global__ __launch_bounds__(kBlock) void sah_level_kernel(const float4* __restrict__ plo,
                                                          const float4* __restrict__ phi,
                                                          uint32_t* __restrict__ idx0, uint32_t* __restrict__ idx1,
                                                          uint32_t* __restrict__ order, const SahTask* __restrict__ tasks,
                                                          SahTask* __restrict__ next, SahTask* __restrict__ small,
                                                          uint32_t turn, SahState* __restrict__ st,
                                                          Node* __restrict__ nodes) {
  __shared__ int s_cb[6];  // centre bounds: lo xyz, hi xyz (ordered ints)
  __shared__ uint32_t s_cnt[3][kSahBins];
  __shared__ int s_lo[3][kSahBins][3], s_hi[3][kSahBins][3];
  __shared__ unsigned long long s_best;
  __shared__ int s_box[2][6];  // child boxes: lo xyz, hi xyz
  __shared__ uint32_t s_wl[kBlock / 64], s_wv[kBlock / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  constexpr float kInf = __builtin_inff();

  const uint32_t ntasks = st->nmid[turn];
  uint32_t* const nnext = &st->nmid[turn == 2u ? 0u : turn + 1u];
  if (blockIdx.x == 0 && threadIdx.x == 0) st->nmid[turn == 0u ? 2u : turn - 1u] = 0u;  // worked off by the level before
  for (uint32_t ti = blockIdx.x; ti < ntasks; ti += gridDim.x) {
    const SahTask T = tasks[ti];
    const uint32_t* __restrict__ src = T.buf ? idx1 : idx0;
    uint32_t* __restrict__ dst = T.buf ? idx0 : idx1;
    const uint32_t a = T.a, b = T.b, m = b - a + 1;

    // 1. bounds of the box centres
    if (tid < 6) s_cb[tid] = tid < 3 ? f2o(kInf) : f2o(-kInf);
    if (tid < 12) s_box[tid / 6][tid % 6] = tid % 6 < 3 ? f2o(kInf) : f2o(-kInf);
    for (int e = tid; e < 3 * kSahBins; e += kBlock) {
      (&s_cnt[0][0])[e] = 0u;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        (&s_lo[0][0][0])[3 * e + q] = f2o(kInf);
        (&s_hi[0][0][0])[3 * e + q] = f2o(-kInf);
      }
    }
    if (tid == 0) s_best = ~0ull;
    float cl[3] = {kInf, kInf, kInf}, ch[3] = {-kInf, -kInf, -kInf};
    for (uint32_t i = a + tid; i <= b; i += kBlock) {
      const uint32_t p = src[i];
      const float4 lo = plo[p], hi = phi[p];
      const float c[3] = {0.5f * (lo.x + hi.x), 0.5f * (lo.y + hi.y), 0.5f * (lo.z + hi.z)};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        cl[k] = fminf(cl[k], c[k]);
        ch[k] = fmaxf(ch[k], c[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      cl[k] = wave_min(cl[k]);
      ch[k] = wave_max(ch[k]);
    }
    __syncthreads();
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        atomicMin(&s_cb[k], f2o(cl[k]));
        atomicMax(&s_cb[3 + k], f2o(ch[k]));
      }
    }
    __syncthreads();
    float cmin[3], scale[3];
    bool use[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) use[k] = bin_axis(s_cb[k], s_cb[3 + k], T.level, cmin[k], scale[k]);

    // 2. bins of every usable axis: count and box union
    if (use[0] || use[1] || use[2]) {
      for (uint32_t i = a + tid; i <= b; i += kBlock) {
        const uint32_t p = src[i];
        const float4 lo = plo[p], hi = phi[p];
        const float c[3] = {0.5f * (lo.x + hi.x), 0.5f * (lo.y + hi.y), 0.5f * (lo.z + hi.z)};
        const int ilo[3] = {f2o(lo.x), f2o(lo.y), f2o(lo.z)}, ihi[3] = {f2o(hi.x), f2o(hi.y), f2o(hi.z)};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          if (!use[k]) continue;
          const int bin = sah_bin(c[k], cmin[k], scale[k]);
          atomicAdd(&s_cnt[k][bin], 1u);
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            atomicMin(&s_lo[k][bin][q], ilo[q]);
            atomicMax(&s_hi[k][bin][q], ihi[q]);
          }
        }
      }
      __syncthreads();
      // 3. cost of every plane (axis k, left = bins below s); lowest (cost, k, s) wins
      if (tid < 3 * kSahBins) {
        const int k = tid / kSahBins, s = tid % kSahBins;
        if (s > 0 && use[k]) {
          uint32_t nl = 0, nr = 0;
          int L[6] = {f2o(kInf), f2o(kInf), f2o(kInf), f2o(-kInf), f2o(-kInf), f2o(-kInf)};
          int R[6] = {L[0], L[1], L[2], L[3], L[4], L[5]};
          for (int j = 0; j < s; ++j) {
            nl += s_cnt[k][j];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
              L[q] = min(L[q], s_lo[k][j][q]);
              L[3 + q] = max(L[3 + q], s_hi[k][j][q]);
            }
          }
          for (int j = s; j < kSahBins; ++j) {
            nr += s_cnt[k][j];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
              R[q] = min(R[q], s_lo[k][j][q]);
              R[3 + q] = max(R[3 + q], s_hi[k][j][q]);
            }
          }
          if (nl > 0 && nr > 0) {
            const float cost = plane_cost(L, R, nl, nr);
            atomicMin(&s_best, ((unsigned long long)__float_as_uint(cost) << 32) | (unsigned)tid);
          }
        }
      }
    }
    __syncthreads();
    const unsigned long long best = s_best;
    const bool halve = best == ~0ull;
    int ax = 0, split = 0;
    uint32_t nl = m / 2;
    if (!halve) {
      const int t = (int)(best & 0xFFFFFFFFull);
      ax = t / kSahBins;
      split = t % kSahBins;
      nl = 0;
      for (int j = 0; j < split; ++j) nl += s_cnt[ax][j];
    }

    // 4. stable partition into dst[a..b]: left part first; child boxes
    float bl[2][3] = {{kInf, kInf, kInf}, {kInf, kInf, kInf}};
    float bh[2][3] = {{-kInf, -kInf, -kInf}, {-kInf, -kInf, -kInf}};
    uint32_t baseL = 0, baseR = 0;
    for (uint32_t c0 = a; c0 <= b; c0 += kBlock) {
      const uint32_t i = c0 + tid;
      const bool valid = i <= b;
      uint32_t p = 0;
      bool left = false;
      if (valid) {
        p = src[i];
        const float4 lo = plo[p], hi = phi[p];
        if (halve) {
          left = i - a < nl;
        } else {
          const float c = ax == 0 ? 0.5f * (lo.x + hi.x) : ax == 1 ? 0.5f * (lo.y + hi.y) : 0.5f * (lo.z + hi.z);
          left = sah_bin(c, cmin[ax], scale[ax]) < split;
        }
        const int side = left ? 0 : 1;
        bl[side][0] = fminf(bl[side][0], lo.x); bl[side][1] = fminf(bl[side][1], lo.y);
        bl[side][2] = fminf(bl[side][2], lo.z);
        bh[side][0] = fmaxf(bh[side][0], hi.x); bh[side][1] = fmaxf(bh[side][1], hi.y);
        bh[side][2] = fmaxf(bh[side][2], hi.z);
      }
      const unsigned long long wl = __ballot(left), wv = __ballot(valid);
      if (lane == 0) {
        s_wl[wave] = (uint32_t)__popcll(wl);
        s_wv[wave] = (uint32_t)__popcll(wv);
      }
      __syncthreads();
      uint32_t offL = 0, offV = 0, totL = 0, totV = 0;
#pragma unroll
      for (int w = 0; w < kBlock / 64; ++w) {
        if (w < wave) {
          offL += s_wl[w];
          offV += s_wv[w];
        }
        totL += s_wl[w];
        totV += s_wv[w];
      }
      if (valid) {
        const uint32_t pl = (uint32_t)__popcll(wl & lt_mask), pv = (uint32_t)__popcll(wv & lt_mask);
        const uint32_t pos = left ? a + baseL + offL + pl : a + nl + baseR + (offV - offL) + (pv - pl);
        if (pos >= a && pos <= b) {
          dst[pos] = p;
          if (left ? nl == 1 : m - nl == 1) order[pos] = p;  // a one-triangle child is a leaf
        }
      }
      baseL += totL;
      baseR += totV - totL;
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        bl[s][q] = wave_min(bl[s][q]);
        bh[s][q] = wave_max(bh[s][q]);
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          atomicMin(&s_box[s][q], f2o(bl[s][q]));
          atomicMax(&s_box[s][3 + q], f2o(bh[s][q]));
        }
      }
    }
    __syncthreads();

    // 5. the node, its internal children as tasks of the next level
    if (tid == 0) {
      if (baseL != nl) atomicOr(&st->err, 1u);  // partition disagrees with the bin counts
      const uint32_t nr = m - nl;
      nodes[T.id] = make_node(s_box[0], s_box[1], nl == 1 ? ~(int)a : (int)(a + nl - 1),
                              nr == 1 ? ~(int)b : (int)(a + nl), T.parent);
      emit_children(T, nl, T.buf ^ 1u, next, nnext, small, &st->nsmall);
      atomicMax(&st->depth, T.level + 1u);
    }
    __syncthreads();  // LDS is reused by the next task
  }
}

// ---- big nodes (m > kSahBig): chunks of kSahChunk triangles ----

// Bins of one chunk: LDS first, then the node's bins; the chunk's own counts
// are kept for the partition's offsets.
__global__ __launch_bounds__(kBlock) void sah_big_bins_kernel(const float4* __restrict__ plo,
                                                             const float4* __restrict__ phi,
                                                             const uint32_t* __restrict__ idx0,
                                                             const uint32_t* __restrict__ idx1,
                                                             const SahTask* __restrict__ tasks,
                                                             const uint32_t* __restrict__ chunk_task,
                                                             uint32_t* __restrict__ chunk_cnt, uint32_t par,
                                                             SahState* __restrict__ st, SahBins* __restrict__ bins) {
  __shared__ SahBins s;
  if (blockIdx.x == 0 && threadIdx.x == 0) st->nbig[par ^ 1u] = st->nchunk[par ^ 1u] = 0u;  // the lists this level fills
  const uint32_t nchunk = st->nchunk[par];
  for (uint32_t ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
    const uint32_t ti = chunk_task[ch];
    const SahTask T = tasks[ti];
    const uint32_t* __restrict__ src = T.buf ? idx1 : idx0;
    const uint32_t c0 = T.a + (ch - T.chunk0) * kSahChunk, c1 = min(T.b + 1u, c0 + kSahChunk);
    for (int e = threadIdx.x; e < 3 * kSahBins; e += kBlock) {
      (&s.cnt[0][0])[e] = 0u;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        (&s.lo[0][0][0])[3 * e + q] = f2o(__builtin_inff());
        (&s.hi[0][0][0])[3 * e + q] = f2o(-__builtin_inff());
      }
    }
    float cmin[3], scale[3];
    bool use[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) use[k] = bin_axis(bins[ti].cb[k], bins[ti].cb[3 + k], T.level, cmin[k], scale[k]);
    __syncthreads();
    for (uint32_t i = c0 + threadIdx.x; i < c1; i += kBlock) {
      const uint32_t p = src[i];
      const float4 lo = plo[p], hi = phi[p];
      const float3 cc = box_centre(lo, hi);
      const float c[3] = {cc.x, cc.y, cc.z};
      const int ilo[3] = {f2o(lo.x), f2o(lo.y), f2o(lo.z)}, ihi[3] = {f2o(hi.x), f2o(hi.y), f2o(hi.z)};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (!use[k]) continue;
        const int bin = sah_bin(c[k], cmin[k], scale[k]);
        atomicAdd(&s.cnt[k][bin], 1u);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          atomicMin(&s.lo[k][bin][q], ilo[q]);
          atomicMax(&s.hi[k][bin][q], ihi[q]);
        }
      }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * kSahBins; e += kBlock) {
      const uint32_t n = (&s.cnt[0][0])[e];
      chunk_cnt[ch * (3u * kSahBins) + e] = n;
      if (n == 0u) continue;
      atomicAdd(&bins[ti].cnt[0][0] + e, n);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        atomicMin(&bins[ti].lo[0][0][0] + 3 * e + q, (&s.lo[0][0][0])[3 * e + q]);
        atomicMax(&bins[ti].hi[0][0][0] + 3 * e + q, (&s.hi[0][0][0])[3 * e + q]);
      }
    }
    __syncthreads();  // s is reused by the next chunk
  }
}

// Plane of each big node, its node record and children (big ones into the next
// list with their chunks, their bins cleared), and each chunk's offset among
// the node's left triangles (chunk_left).  A node that cannot be binned goes
// to the mid-stage list as it is.
__global__ __launch_bounds__(kBlock) void sah_big_split_kernel(SahTask* __restrict__ tasks, SahTask* __restrict__ next,
                                                              SahTask* __restrict__ mid, SahTask* __restrict__ small,
                                                              uint32_t* __restrict__ next_chunk_task,
                                                              const uint32_t* __restrict__ chunk_cnt,
                                                              uint32_t* __restrict__ chunk_left, uint32_t par,
                                                              uint32_t turn, SahState* __restrict__ st,
                                                              const SahBins* __restrict__ bins,
                                                              SahBins* __restrict__ next_bins,
                                                              Node* __restrict__ nodes) {
  __shared__ unsigned long long s_best;
  __shared__ uint32_t s_sum[kBlock / 64], s_carry, s_child[2], s_chunk[2];
  __shared__ SahBins B;
  const uint32_t ntasks = st->nbig[par];
  for (uint32_t ti = blockIdx.x; ti < ntasks; ti += gridDim.x) {
    const SahTask T = tasks[ti];
    for (uint32_t w = threadIdx.x; w < sizeof(SahBins) / 4u; w += kBlock)
      reinterpret_cast<uint32_t*>(&B)[w] = reinterpret_cast<const uint32_t*>(&bins[ti])[w];
    const uint32_t m = T.b - T.a + 1u, nch = (m + kSahChunk - 1u) / kSahChunk;
    if (threadIdx.x == 0) {
      s_best = ~0ull;
      s_carry = 0u;
    }
    __syncthreads();
    int L[6], R[6];
    if (threadIdx.x < 3u * kSahBins) {
      const int k = threadIdx.x / kSahBins, sp = threadIdx.x % kSahBins;
      float cmin, scale;
      if (sp > 0 && bin_axis(B.cb[k], B.cb[3 + k], T.level, cmin, scale)) {
        uint32_t nl = 0, nr = 0;
        empty_box(L);
        empty_box(R);
        for (int j = 0; j < kSahBins; ++j) {
          const bool left = j < sp;
          (left ? nl : nr) += B.cnt[k][j];
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const int lo = B.lo[k][j][q], hi = B.hi[k][j][q];
            if (left) {
              L[q] = min(L[q], lo);
              L[3 + q] = max(L[3 + q], hi);
            } else {
              R[q] = min(R[q], lo);
              R[3 + q] = max(R[3 + q], hi);
            }
          }
        }
        if (nl > 0 && nr > 0)
          atomicMin(&s_best, ((unsigned long long)__float_as_uint(plane_cost(L, R, nl, nr)) << 32) | threadIdx.x);
      }
    }
    __syncthreads();
    const unsigned long long best = s_best;
    if (best == ~0ull) {  // uniform
      if (threadIdx.x == 0) {
        tasks[ti].nl = 0u;
        mid[atomicAdd(&st->nmid[turn], 1u)] = T;
      }
      __syncthreads();
      continue;
    }
    const uint32_t t = (uint32_t)best, ax = t / kSahBins, split = t % kSahBins;
    // left triangles of each chunk, and of the chunks before it: a scan per
    // wave of 64 chunks, then the waves' sums
    for (uint32_t c0 = 0; c0 < nch; c0 += kBlock) {
      const uint32_t c = c0 + threadIdx.x;
      uint32_t n = 0;
      if (c < nch)
        for (uint32_t j = 0; j < split; ++j) n += chunk_cnt[(T.chunk0 + c) * (3u * kSahBins) + ax * kSahBins + j];
      uint32_t incl = n;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t add = __shfl_up(incl, o);
        incl += (threadIdx.x & 63u) >= (uint32_t)o ? add : 0u;
      }
      if ((threadIdx.x & 63u) == 63u) s_sum[threadIdx.x >> 6] = incl;
      __syncthreads();
      uint32_t before = s_carry, all = 0;
      for (uint32_t w = 0; w < kBlock / 64; ++w) {
        before += w < (threadIdx.x >> 6) ? s_sum[w] : 0u;
        all += s_sum[w];
      }
      if (c < nch) chunk_left[T.chunk0 + c] = before + incl - n;
      __syncthreads();
      if (threadIdx.x == 0) s_carry += all;
      __syncthreads();
    }
    const uint32_t nl = s_carry;
    if (threadIdx.x == t) {  // holds the plane's boxes
      const uint32_t nr = m - nl;
      nodes[T.id] = make_node(L, R, nl == 1u ? ~(int)T.a : (int)(T.a + nl - 1u),
                              nr == 1u ? ~(int)T.b : (int)(T.a + nl), T.parent);
      atomicMax(&st->depth, T.level + 1u);
      tasks[ti].nl = nl;
      tasks[ti].ax = ax;
      tasks[ti].split = split;
    }
    if (threadIdx.x < 2u) {
      const uint32_t n = threadIdx.x == 0u ? nl : m - nl;
      uint32_t slot = kNoTask;
      if (n >= 2u) {
        SahTask c{};
        c.a = threadIdx.x == 0u ? T.a : T.a + nl;
        c.b = c.a + n - 1u;
        c.id = threadIdx.x == 0u ? c.b : c.a;
        c.parent = (int32_t)T.id;
        c.level = T.level + 1u;
        c.buf = T.buf ^ 1u;
        if (n > kSahBig) {
          c.chunk0 = atomicAdd(&st->nchunk[par ^ 1u], (n + kSahChunk - 1u) / kSahChunk);
          slot = atomicAdd(&st->nbig[par ^ 1u], 1u);
          next[slot] = c;
          s_chunk[threadIdx.x] = c.chunk0;
        } else if (n > kSahWave) {
          mid[atomicAdd(&st->nmid[turn], 1u)] = c;
        } else {
          small[atomicAdd(&st->nsmall, 1u)] = c;
        }
      }
      s_child[threadIdx.x] = slot;
    }
    __syncthreads();
    if (threadIdx.x < 2u) tasks[ti].child[threadIdx.x] = s_child[threadIdx.x];  // for the partition's centre bounds
    for (int side = 0; side < 2; ++side) {
      if (s_child[side] == kNoTask) continue;
      const uint32_t n = side == 0 ? nl : m - nl;
      for (uint32_t c = threadIdx.x; c < (n + kSahChunk - 1u) / kSahChunk; c += kBlock)
        next_chunk_task[s_chunk[side] + c] = s_child[side];
      SahBins& C = next_bins[s_child[side]];
      if (threadIdx.x < 6u) C.cb[threadIdx.x] = f2o(threadIdx.x < 3u ? __builtin_inff() : -__builtin_inff());
      for (int e = threadIdx.x; e < 3 * kSahBins; e += kBlock) {
        (&C.cnt[0][0])[e] = 0u;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          (&C.lo[0][0][0])[3 * e + q] = f2o(__builtin_inff());
          (&C.hi[0][0][0])[3 * e + q] = f2o(-__builtin_inff());
        }
      }
    }
    __syncthreads();
  }
}

// Bounds of box centres, gathered per thread and added to a node's cb by the
// workgroup (one address takes an atomic every 12 ns: with one set of six per
// wave the root's took 57 us).
struct CentreBounds {
  float lo[3], hi[3];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      lo[q] = __builtin_inff();
      hi[q] = -__builtin_inff();
    }
  }
  __device__ __forceinline__ void add(const float3& c) {
    lo[0] = fminf(lo[0], c.x), lo[1] = fminf(lo[1], c.y), lo[2] = fminf(lo[2], c.z);
    hi[0] = fmaxf(hi[0], c.x), hi[1] = fmaxf(hi[1], c.y), hi[2] = fmaxf(hi[2], c.z);
  }
  // Called by the whole workgroup; s: six words of LDS, reused after a barrier.
  __device__ __forceinline__ void flush(int* __restrict__ s, int* __restrict__ cb) {
    if (threadIdx.x < 6u) s[threadIdx.x] = f2o(threadIdx.x < 3u ? __builtin_inff() : -__builtin_inff());
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const float l = wave_min(lo[q]), h = wave_max(hi[q]);
      if ((threadIdx.x & 63u) == 0u) {
        atomicMin(s + q, f2o(l));
        atomicMax(s + 3 + q, f2o(h));
      }
    }
    __syncthreads();
    if (threadIdx.x < 3u) atomicMin(cb + threadIdx.x, s[threadIdx.x]);
    else if (threadIdx.x < 6u) atomicMax(cb + threadIdx.x, s[threadIdx.x]);
    __syncthreads();
  }
};

// Stable partition of a chunk into the other index array, and the bounds of
// the centres of big children.
__global__ __launch_bounds__(kBlock) void sah_big_part_kernel(const float4* __restrict__ plo,
                                                             const float4* __restrict__ phi,
                                                             uint32_t* __restrict__ idx0, uint32_t* __restrict__ idx1,
                                                             uint32_t* __restrict__ order,
                                                             const SahTask* __restrict__ tasks,
                                                             const uint32_t* __restrict__ chunk_task,
                                                             const uint32_t* __restrict__ chunk_left, uint32_t par,
                                                             SahState* __restrict__ st,
                                                             const SahBins* __restrict__ bins,
                                                             SahBins* __restrict__ next_bins) {
  __shared__ uint32_t s_wl[kBlock / 64], s_wv[kBlock / 64];
  __shared__ int s_cb[6];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  const uint32_t nchunk = st->nchunk[par];
  for (uint32_t ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
    const uint32_t ti = chunk_task[ch];
    const SahTask T = tasks[ti];
    if (T.nl == 0u) continue;  // uniform: left to the mid stage
    const uint32_t* __restrict__ src = T.buf ? idx1 : idx0;
    uint32_t* __restrict__ dst = T.buf ? idx0 : idx1;
    const uint32_t m = T.b - T.a + 1u;
    const uint32_t c0 = T.a + (ch - T.chunk0) * kSahChunk, c1 = min(T.b + 1u, c0 + kSahChunk);
    float cmin, scale;
    bin_axis(bins[ti].cb[T.ax], bins[ti].cb[3 + T.ax], T.level, cmin, scale);
    CentreBounds side[2];
    side[0].clear();
    side[1].clear();
    uint32_t baseL = chunk_left[ch], baseR = (ch - T.chunk0) * kSahChunk - baseL;
    for (uint32_t i0 = c0; i0 < c1; i0 += kBlock) {
      const uint32_t i = i0 + threadIdx.x;
      const bool valid = i < c1;
      uint32_t p = 0;
      bool left = false;
      float3 c = make_float3(0.0f, 0.0f, 0.0f);
      if (valid) {
        p = src[i];
        c = box_centre(plo[p], phi[p]);
        left = sah_bin(T.ax == 0u ? c.x : T.ax == 1u ? c.y : c.z, cmin, scale) < (int)T.split;
        if (left) side[0].add(c);
        else side[1].add(c);
      }
      const unsigned long long wl = __ballot(left), wv = __ballot(valid);
      if (lane == 0) {
        s_wl[wave] = (uint32_t)__popcll(wl);
        s_wv[wave] = (uint32_t)__popcll(wv);
      }
      __syncthreads();
      uint32_t offL = 0, offV = 0, totL = 0, totV = 0;
#pragma unroll
      for (int w = 0; w < kBlock / 64; ++w) {
        if (w < wave) {
          offL += s_wl[w];
          offV += s_wv[w];
        }
        totL += s_wl[w];
        totV += s_wv[w];
      }
      if (valid) {
        const uint32_t pl = (uint32_t)__popcll(wl & lt_mask), pv = (uint32_t)__popcll(wv & lt_mask);
        const uint32_t pos = left ? T.a + baseL + offL + pl : T.a + T.nl + baseR + (offV - offL) + (pv - pl);
        if (pos >= T.a && pos <= T.b) {
          dst[pos] = p;
          if (left ? T.nl == 1u : m - T.nl == 1u) order[pos] = p;  // a one-triangle child is a leaf
        }
      }
      baseL += totL;
      baseR += totV - totL;
      __syncthreads();
    }
    if (T.child[0] != kNoTask) side[0].flush(s_cb, next_bins[T.child[0]].cb);
    if (T.child[1] != kNoTask) side[1].flush(s_cb, next_bins[T.child[1]].cb);
    if (threadIdx.x == 0 && c1 == T.b + 1u && baseL != T.nl) atomicOr(&st->err, 1u);
  }
}

// ---- small nodes (m <= kSahWave): one wave per subtree, a triangle per lane ----
//
// Lane l holds the triangle at position l of the subtree's range.  Nodes are
// worked off one after another from a stack in LDS: the bounds of the centres
// and the sums of every plane run over the node's triangles one at a time (their
// values in scalar registers), each lane summing for its own plane -- 32 planes
// of two axes in a first pass, of the third in a second -- so no bins are kept
// and no barrier is needed.  A pair needs no sums (pair_plane).  kSahWave: a wave
// takes longer the larger its subtree (64: 267 us on the 50k satellite, one level
// launch of 25 us less).
__global__ __launch_bounds__(kBlock) void sah_wave_kernel(const float4* __restrict__ plo,
                                                          const float4* __restrict__ phi,
                                                          const uint32_t* __restrict__ idx0,
                                                          const uint32_t* __restrict__ idx1,
                                                          uint32_t* __restrict__ order,
                                                          const SahTask* __restrict__ small,
                                                          SahState* __restrict__ st, Node* __restrict__ nodes) {
  __shared__ uint32_t s_node[kBlock / 64][64], s_parent[kBlock / 64][64];  // waiting nodes: (first, last, level), parent
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t ntasks = st->nsmall;
  uint32_t depth = 0;
  for (uint32_t ti = blockIdx.x * (kBlock / 64) + wave; ti < ntasks; ti += gridDim.x * (kBlock / 64)) {
    const SahTask T = small[ti];
    const uint32_t base = __builtin_amdgcn_readfirstlane(T.a);
    const uint32_t m = __builtin_amdgcn_readfirstlane(T.b) - base + 1u;
    uint32_t p = 0;
    int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0}, oc[3] = {0, 0, 0};  // box and centre as ordered ints
    if (lane < m) {
      p = (T.buf ? idx1 : idx0)[base + lane];
      const float4 l4 = plo[p], h4 = phi[p];
      const float3 c = box_centre(l4, h4);
      lo[0] = f2o(l4.x); lo[1] = f2o(l4.y); lo[2] = f2o(l4.z);
      hi[0] = f2o(h4.x); hi[1] = f2o(h4.y); hi[2] = f2o(h4.z);
      oc[0] = f2o(c.x); oc[1] = f2o(c.y); oc[2] = f2o(c.z);
    }
    uint32_t sp = 1;
    if (lane == 0) {
      s_node[wave][0] = (m - 1u) << 8 | T.level << 16;
      s_parent[wave][0] = (uint32_t)T.parent;
    }
    __builtin_amdgcn_wave_barrier();
    bool root = true;
    while (sp > 0u) {
      --sp;
      const uint32_t w = __builtin_amdgcn_readfirstlane(s_node[wave][sp]);
      const int32_t parent = (int32_t)__builtin_amdgcn_readfirstlane(s_parent[wave][sp]);
      const uint32_t s = w & 255u, e = (w >> 8) & 255u, level = (w >> 16) & 0x7FFFu;  // positions [s, e]
      const uint32_t n = e - s + 1u;
      const bool in = lane >= s && lane <= e;
      // 1. bounds of the centres
      int cb[6];
      empty_box(cb);
      for (uint32_t j = s; j <= e; ++j) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const int c = __builtin_amdgcn_readlane(oc[q], j);
          cb[q] = min(cb[q], c);
          cb[3 + q] = max(cb[3 + q], c);
        }
      }
      // 2. bins of the lane's triangle
      float cmin[3], scale[3];
      bool use[3];
      uint32_t bins = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        use[k] = bin_axis(cb[k], cb[3 + k], level, cmin[k], scale[k]);
        if (use[k] && in) bins |= (uint32_t)sah_bin(o2f(oc[k]), cmin[k], scale[k]) << (8 * k);
      }
      // 3. every plane: lane (k, sp) of pass 0 axes 0 and 1, of pass 1 axis 2
      unsigned long long best = ~0ull;
      int L[2][6], R[2][6];
      const bool pair = n == 2u;
      if (!pair)
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
        const int k = pass == 0 ? (int)(lane >> 5) : 2;
        const uint32_t plane = lane & 31u, shift = 8u * (uint32_t)k;
        empty_box(L[pass]);
        empty_box(R[pass]);
        uint32_t nl = 0;
        for (uint32_t j = s; j <= e; ++j) {
          const uint32_t bj = (uint32_t)__builtin_amdgcn_readlane((int)bins, j);
          const bool left = ((bj >> shift) & 255u) < plane;
          nl += left ? 1u : 0u;
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const int jl = __builtin_amdgcn_readlane(lo[q], j), jh = __builtin_amdgcn_readlane(hi[q], j);
            L[pass][q] = left ? min(L[pass][q], jl) : L[pass][q];
            L[pass][3 + q] = left ? max(L[pass][3 + q], jh) : L[pass][3 + q];
            R[pass][q] = left ? R[pass][q] : min(R[pass][q], jl);
            R[pass][3 + q] = left ? R[pass][3 + q] : max(R[pass][3 + q], jh);
          }
        }
        const bool usable = pass == 0 ? (lane < 32u ? use[0] : use[1]) : (lane < 32u && use[2]);
        if (usable && plane > 0u && nl > 0u && nl < n) {
          const unsigned long long key =
              ((unsigned long long)__float_as_uint(plane_cost(L[pass], R[pass], nl, n - nl)) << 32) |
              ((uint32_t)k * kSahBins + plane);
          best = key < best ? key : best;
        }
      }
      if (!pair)
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long other = __shfl_xor(best, o);
        best = other < best ? other : best;
      }
      else {
        const uint32_t plane = pair_plane((uint32_t)__builtin_amdgcn_readlane((int)bins, s),
                                          (uint32_t)__builtin_amdgcn_readlane((int)bins, e));
        if (plane != kNoPlane) best = plane;
      }
      const bool halve = best == ~0ull;  // uniform
      const uint32_t t = __builtin_amdgcn_readfirstlane((uint32_t)best);
      // 4. left side, stable positions, child boxes
      const bool left = in && (halve ? lane - s < n / 2u : ((bins >> (8u * (t / kSahBins))) & 255u) < t % kSahBins);
      const uint64_t lm = __ballot(left), im = __ballot(in);
      const uint32_t nl = (uint32_t)__popcll(lm);
      int bl[6], br[6];
      if (halve || pair) {
        empty_box(bl);
        empty_box(br);
        for (uint32_t j = s; j <= e; ++j) {
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const int jl = __builtin_amdgcn_readlane(lo[q], j), jh = __builtin_amdgcn_readlane(hi[q], j);
            if (lm >> j & 1ull) {
              bl[q] = min(bl[q], jl);
              bl[3 + q] = max(bl[3 + q], jh);
            } else {
              br[q] = min(br[q], jl);
              br[3 + q] = max(br[3 + q], jh);
            }
          }
        }
      } else {
        const uint32_t from = t & 63u;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          bl[q] = t < 64u ? __builtin_amdgcn_readlane(L[0][q], from) : __builtin_amdgcn_readlane(L[1][q], from);
          br[q] = t < 64u ? __builtin_amdgcn_readlane(R[0][q], from) : __builtin_amdgcn_readlane(R[1][q], from);
        }
      }
      const uint64_t below = (1ull << lane) - 1ull;
      const uint32_t nleft = (uint32_t)__popcll(lm & below), nin = (uint32_t)__popcll(im & below);
      const uint32_t to = !in ? lane : (left ? s + nleft : s + nl + (nin - nleft));
      const int addr = (int)(to * 4u);
      p = (uint32_t)__builtin_amdgcn_ds_permute(addr, (int)p);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        lo[q] = __builtin_amdgcn_ds_permute(addr, lo[q]);
        hi[q] = __builtin_amdgcn_ds_permute(addr, hi[q]);
        oc[q] = __builtin_amdgcn_ds_permute(addr, oc[q]);
      }
      // 5. the node and its internal children
      const uint32_t nr = n - nl, a = base + s, b = base + e;
      const uint32_t id = root ? T.id : (w & 0x80000000u ? b : a);
      if (lane == 0) {
        nodes[id] = make_node(bl, br, nl == 1u ? ~(int)a : (int)(a + nl - 1u), nr == 1u ? ~(int)b : (int)(a + nl),
                              parent);
        uint32_t at = sp;
        if (nr > 1u) {
          s_node[wave][at] = (s + nl) | e << 8 | (level + 1u) << 16;
          s_parent[wave][at++] = id;
        }
        if (nl > 1u) {
          s_node[wave][at] = s | (s + nl - 1u) << 8 | (level + 1u) << 16 | 0x80000000u;  // a left child
          s_parent[wave][at] = id;
        }
      }
      sp += (nl > 1u ? 1u : 0u) + (nr > 1u ? 1u : 0u);
      __builtin_amdgcn_wave_barrier();
      depth = max(depth, level + 1u);
      root = false;
    }
    if (lane < m) order[base + lane] = p;
  }
  if (lane == 0 && depth > 0u) atomicMax(&st->depth, depth);
}

__global__ __launch_bounds__(kBlock) void prim_box_kernel(const float* __restrict__ xyz,
                                                          const uint32_t* __restrict__ tri, uint32_t nt,
                                                          float4* __restrict__ plo, float4* __restrict__ phi,
                                                          uint32_t* __restrict__ idx, uint32_t* __restrict__ order,
                                                          SahBins* __restrict__ bins) {
  __shared__ int s_cb[6];
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool on = i < nt;
  float lo[3] = {0.0f, 0.0f, 0.0f}, hi[3] = {0.0f, 0.0f, 0.0f};
  if (on) {
    const uint32_t a = tri[3 * i], b = tri[3 * i + 1], c = tri[3 * i + 2];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float x = xyz[3 * a + k], y = xyz[3 * b + k], z = xyz[3 * c + k];
      lo[k] = fminf(fminf(x, y), z);
      hi[k] = fmaxf(fmaxf(x, y), z);
    }
    plo[i] = make_float4(lo[0], lo[1], lo[2], 0.0f);
    phi[i] = make_float4(hi[0], hi[1], hi[2], 0.0f);
    idx[i] = i;
    order[i] = i;  // names a triangle from the start: the packing may run before every leaf is placed
  }
  if (bins) {  // uniform
    CentreBounds c;
    c.clear();
    if (on) c.add(box_centre(make_float4(lo[0], lo[1], lo[2], 0.0f), make_float4(hi[0], hi[1], hi[2], 0.0f)));
    c.flush(s_cb, bins->cb);
  }
}

// The root task in its stage's list, and the empty state.
__global__ __launch_bounds__(kBlock) void sah_root_kernel(SahState* __restrict__ st, SahTask* __restrict__ big,
                                                          SahTask* __restrict__ mid, SahTask* __restrict__ small,
                                                          uint32_t* __restrict__ chunk_task, SahBins* __restrict__ bins,
                                                          uint32_t nt) {
  const SahTask T{0u, nt - 1u, 0u, -1, 0u, 0u, 0u, 0u, 0u, 0u, {kNoTask, kNoTask}};
  const uint32_t nch = (nt + kSahChunk - 1u) / kSahChunk;
  if (threadIdx.x == 0) {
    *st = SahState{};
    if (nt > kSahBig) {
      big[0] = T;
      st->nbig[0] = 1u;
      st->nchunk[0] = nch;
    } else if (nt > kSahWave) {
      mid[0] = T;
      st->nmid[0] = 1u;
    } else {
      small[0] = T;
      st->nsmall = 1u;
    }
  }
  if (nt <= kSahBig) return;
  for (uint32_t c = threadIdx.x; c < nch; c += kBlock) chunk_task[c] = 0u;
  if (threadIdx.x < 6u) bins->cb[threadIdx.x] = f2o(threadIdx.x < 3u ? __builtin_inff() : -__builtin_inff());
  for (int e = threadIdx.x; e < 3 * kSahBins; e += kBlock) {
    (&bins->cnt[0][0])[e] = 0u;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      (&bins->lo[0][0][0])[3 * e + q] = f2o(__builtin_inff());
      (&bins->hi[0][0][0])[3 * e + q] = f2o(-__builtin_inff());
    }
  }
}

}  // namespace

void mark_support(const float* d_xyz, uint64_t nv, const TriRec* d_tris, uint64_t nt, uint32_t* d_orig,
                  const Node* d_nodes, const uint32_t* d_depth, BuildRead* d_read, void* scratch, hipStream_t st) {
  uint32_t* n_list = static_cast<uint32_t*>(scratch);
  uint32_t* list = n_list + 64;
  if (nv > kSupportAll) zero_u32(n_list, 1, st);
  support_spread_kernel<<<(uint32_t)((nt + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      d_xyz, (uint32_t)nv, d_tris, (uint32_t)nt, d_orig, list, n_list, d_nodes, d_depth, d_read);
  if (nv <= kSupportAll) return;
  const uint64_t pairs = (nt + kSupportTris - 1) / kSupportTris * ((nv + kSupportSegment - 1) / kSupportSegment);
  support_kernel<<<(uint32_t)std::min<uint64_t>(2048, pairs / 4 + 1), kBlock, 0, st>>>(d_xyz, (uint32_t)nv, d_tris, d_orig,
                                                                                   list, n_list);
}

size_t support_scratch_bytes(uint64_t nt) { return (nt + 64) * sizeof(uint32_t); }

size_t bvh_scratch_bytes(uint64_t nt) {
  const uint64_t nblocks = (nt + kSortTile - 1) / kSortTile;
  // xyz/tri copies are separate; here: keys x2, vals x2, counts, leaf_parent, flags, nbox, depth
  return (4 * nt + 16 * nblocks + 2 * nt + 6 * nt + 64) * sizeof(uint32_t) + 4096;
}

hipError_t build_bvh(const float* d_xyz, const uint32_t* d_tri, uint64_t nt64, const float box_lo[3],
                     const float box_hi[3], void* scratch, Node* d_nodes, TriRec* d_tris, uint32_t* d_orig,
                     uint32_t* h_depth, const uint32_t** d_depth, hipStream_t st) {
  *d_depth = nullptr;
  const uint32_t nt = (uint32_t)nt64;
  const uint32_t nblocks = (nt + kSortTile - 1) / kSortTile;
  uint32_t* k0 = static_cast<uint32_t*>(scratch);
  uint32_t* v0 = k0 + nt;
  uint32_t* k1 = v0 + nt;
  uint32_t* v1 = k1 + nt;
  uint32_t* counts = v1 + nt;
  int32_t* leaf_parent = reinterpret_cast<int32_t*>(counts + 16 * nblocks);
  uint32_t* flags = reinterpret_cast<uint32_t*>(leaf_parent + nt);
  float* nbox = reinterpret_cast<float*>(flags + nt);
  uint32_t* depth = reinterpret_cast<uint32_t*>(nbox + 6 * nt);

  float ext[3], sc[3];
  for (int k = 0; k < 3; ++k) {
    ext[k] = box_hi[k] - box_lo[k];
    sc[k] = ext[k] > 0.0f ? 1024.0f / ext[k] : 0.0f;
  }
  const uint32_t g = (nt + kBlock - 1) / kBlock;
  morton_kernel<<<g, kBlock, 0, st>>>(d_xyz, d_tri, nt, box_lo[0], box_lo[1], box_lo[2], sc[0], sc[1], sc[2], k0, v0);
  for (int shift = 0; shift < 30; shift += 4) {
    radix_count_kernel<<<nblocks, kBlock, 0, st>>>(k0, nt, shift, counts, nblocks);
    scan_kernel<<<1, 1024, 0, st>>>(counts, 16 * nblocks);
    radix_scatter_kernel<<<nblocks, kBlock, 0, st>>>(k0, v0, k1, v1, nt, shift, counts, nblocks);
    uint32_t* t = k0; k0 = k1; k1 = t;
    t = v0; v0 = v1; v1 = t;
  }
  pack_tris_kernel<<<g, kBlock, 0, st>>>(d_xyz, d_tri, v0, nt, d_tris, d_orig);
  hipError_t e;
  if (nt == 1) {
    single_node_kernel<<<1, 1, 0, st>>>(d_nodes, d_tris);
    *h_depth = 1;
    return hipGetLastError();
  }
  zero_u32(flags, nt, st);
  zero_u32(depth, 1, st);
  e = hipMemsetAsync(leaf_parent, 0xFF, nt * sizeof(int32_t), st);  // -1: no parent yet
  if (e != hipSuccess) return e;
  const uint32_t gi = (nt - 1 + kBlock - 1) / kBlock;
  karras_kernel<<<gi, kBlock, 0, st>>>(k0, (int)nt, d_nodes, leaf_parent);
  refit_kernel<<<g, kBlock, 0, st>>>(d_nodes, leaf_parent, d_tris, nt, flags, nbox);
  depth_kernel<<<g, kBlock, 0, st>>>(d_nodes, leaf_parent, nt, depth);
  *d_depth = depth;
  return hipGetLastError();
}

namespace {

// Scratch of a SAH build: base null gives the size alone.
struct SahScratch {
  float4 *plo, *phi;
  uint32_t *idx[2], *order, *chunk_task[2], *chunk_cnt, *chunk_left;
  SahTask *big[2], *mid[2], *small;
  SahBins* bins[2];
  SahState* st;
  size_t bytes;
};

SahScratch sah_scratch(uint64_t nt, char* base) {
  SahScratch x{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* q = base + off;
    off += (bytes + 255) & ~size_t(255);
    return q;
  };
  // disjoint ranges: at most nt / (kSahBig + 1) big nodes at a time, with a
  // part chunk each, and nt / (kSahWave + 1) mid ones; a small one has two
  // triangles or more
  const size_t nbig = nt / (kSahBig + 1) + 1, nchunk = nt / kSahChunk + nbig + 1, nmid = nt / (kSahWave + 1) + 1;
  x.plo = reinterpret_cast<float4*>(take(nt * sizeof(float4)));
  x.phi = reinterpret_cast<float4*>(take(nt * sizeof(float4)));
  for (int k = 0; k < 2; ++k) {
    x.idx[k] = reinterpret_cast<uint32_t*>(take(nt * sizeof(uint32_t)));
    x.chunk_task[k] = reinterpret_cast<uint32_t*>(take(nchunk * sizeof(uint32_t)));
    x.big[k] = reinterpret_cast<SahTask*>(take(nbig * sizeof(SahTask)));
    x.mid[k] = reinterpret_cast<SahTask*>(take(nmid * sizeof(SahTask)));
    x.bins[k] = reinterpret_cast<SahBins*>(take(nbig * sizeof(SahBins)));
  }
  x.order = reinterpret_cast<uint32_t*>(take(nt * sizeof(uint32_t)));
  x.chunk_cnt = reinterpret_cast<uint32_t*>(take(nchunk * 3 * kSahBins * sizeof(uint32_t)));
  x.chunk_left = reinterpret_cast<uint32_t*>(take(nchunk * sizeof(uint32_t)));
  x.small = reinterpret_cast<SahTask*>(take((nt / 2 + 1) * sizeof(SahTask)));
  x.st = reinterpret_cast<SahState*>(take(sizeof(SahState)));
  x.bytes = off;
  return x;
}

// Levels from n triangles down to a node of at most `to` in a balanced tree.
uint32_t levels_to(uint32_t n, uint32_t to) {
  uint32_t l = 0;
  while (n > to) {
    n = (n + 1) / 2;
    ++l;
  }
  return l;
}

}  // namespace

size_t sah_scratch_bytes(uint64_t nt) { return sah_scratch(nt, nullptr).bytes; }

hipError_t build_bvh_sah(const float* d_xyz, const uint32_t* d_tri, uint64_t nt64, void* scratch, Node* d_nodes,
                         TriRec* d_tris, uint32_t* d_orig, uint32_t* h_depth, hipStream_t st) {
  const uint32_t nt = (uint32_t)nt64;
  const SahScratch x = sah_scratch(nt64, static_cast<char*>(scratch));
  const uint32_t g = (nt + kBlock - 1) / kBlock;
  hipError_t e;
  if (nt == 1) {
    prim_box_kernel<<<g, kBlock, 0, st>>>(d_xyz, d_tri, nt, x.plo, x.phi, x.idx[0], x.order, nullptr);
    pack_tris_kernel<<<1, kBlock, 0, st>>>(d_xyz, d_tri, x.idx[0], 1u, d_tris, d_orig);
    single_node_kernel<<<1, 1, 0, st>>>(d_nodes, d_tris);
    *h_depth = 1;
    return hipGetLastError();
  }
  sah_root_kernel<<<1, kBlock, 0, st>>>(x.st, x.big[0], x.mid[0], x.small, x.chunk_task[0], x.bins[0], nt);
  prim_box_kernel<<<g, kBlock, 0, st>>>(d_xyz, d_tri, nt, x.plo, x.phi, x.idx[0], x.order,
                                      nt > kSahBig ? x.bins[0] : nullptr);
  // All stages are enqueued before the state is read, with 1.5 times the levels
  // of a balanced tree (an empty level costs 5 to 20 us, a read 60 us).  Where
  // that was not enough the loop goes round again; the small stage and what
  // follows may run twice on the same tasks, to the same effect.  Every stage
  // ends: a node's children are smaller than it, and below kSahMaxLevel ranges
  // are halved, so no list outlives level 64.
  const uint32_t gc = std::min(1024u, nt / kSahChunk + 1u), gt = std::min(1024u, nt / kSahBig + 1u);
  const uint32_t gm = std::min(2048u, nt / kSahWave + 1u), gw = std::min(2048u, nt / 8u + 1u);
  uint32_t par = 0, mid = 0;  // levels done
  uint32_t big_burst = nt > kSahBig ? levels_to(nt, kSahBig) * 3u / 2u + 1u : 0u;
  uint32_t mid_burst = nt > kSahWave ? levels_to(std::min(nt, kSahBig), kSahWave) * 3u / 2u + 2u : 0u;
  for (int round = 0; round < 64; ++round) {
    for (uint32_t l = 0; l < big_burst; ++l, par ^= 1u) {
      sah_big_bins_kernel<<<gc, kBlock, 0, st>>>(x.plo, x.phi, x.idx[0], x.idx[1], x.big[par], x.chunk_task[par],
                                                 x.chunk_cnt, par, x.st, x.bins[par]);
      sah_big_split_kernel<<<gt, kBlock, 0, st>>>(x.big[par], x.big[par ^ 1u], x.mid[mid & 1u], x.small,
                                                  x.chunk_task[par ^ 1u], x.chunk_cnt, x.chunk_left, par, mid % 3u, x.st,
                                                  x.bins[par], x.bins[par ^ 1u], d_nodes);
      sah_big_part_kernel<<<gc, kBlock, 0, st>>>(x.plo, x.phi, x.idx[0], x.idx[1], x.order, x.big[par],
                                                 x.chunk_task[par], x.chunk_left, par, x.st, x.bins[par],
                                                 x.bins[par ^ 1u]);
    }
    for (uint32_t l = 0; l < mid_burst; ++l, ++mid)
      sah_level_kernel<<<gm, kBlock, 0, st>>>(x.plo, x.phi, x.idx[0], x.idx[1], x.order, x.mid[mid & 1u],
                                              x.mid[(mid & 1u) ^ 1u], x.small, mid % 3u, x.st, d_nodes);
    sah_wave_kernel<<<gw, kBlock, 0, st>>>(x.plo, x.phi, x.idx[0], x.idx[1], x.order, x.small, x.st, d_nodes);
    pack_tris_kernel<<<g, kBlock, 0, st>>>(d_xyz, d_tri, x.order, nt, d_tris, d_orig);
    SahState h{};
    e = hipMemcpyAsync(&h, x.st, sizeof h, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (h.err != 0u || h.depth > 64u) return hipErrorUnknown;  // partition inconsistent with the bin counts
    if (h.nbig[par] == 0u && h.nmid[mid % 3u] == 0u) {
      *h_depth = h.depth;  // internal nodes on the longest root-to-leaf path
      return h.depth != 0u ? hipSuccess : hipErrorUnknown;
    }
    big_burst = h.nbig[par] != 0u ? 4u : 0u;
    mid_burst = 4u;
  }
  return hipErrorUnknown;
}

}  // namespace tpmc
