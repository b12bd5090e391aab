// tpmc_sah.hpp -- the binning rule of the SAH build: which axes of a node can be
// binned, a triangle's bin, and the plane of a node of two triangles.
#ifndef TPMC_SAH_HPP
#define TPMC_SAH_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tpmc {

constexpr int kSahBins = 32;
constexpr uint32_t kSahMaxLevel = 32;
constexpr uint32_t kNoPlane = 0xFFFFFFFFu;

// Order-preserving map of floats (no NaN) to int32 (for LDS integer min / max).
__host__ __device__ __forceinline__ int f2o(float f) {
  const int i = __builtin_bit_cast(int, f);
  return i >= 0 ? i : i ^ 0x7FFFFFFF;
}
__host__ __device__ __forceinline__ float o2f(int i) {
  return __builtin_bit_cast(float, i >= 0 ? i : i ^ 0x7FFFFFFF);
}

__host__ __device__ __forceinline__ int sah_bin(float c, float cmin, float scale) {
  const int b = (int)((c - cmin) * scale);
  return b < kSahBins - 1 ? b : kSahBins - 1;
}

// Whether an axis of a node can be binned, and the bins' origin and scale: not
// where every centre coincides, nor where the extent is beyond FP32 (scale 0
// would put every triangle into bin 0).
__host__ __device__ __forceinline__ bool bin_axis(int cb_lo, int cb_hi, uint32_t level, float& cmin, float& scale) {
  cmin = o2f(cb_lo);
  const float ext = o2f(cb_hi) - cmin;
  scale = (float)kSahBins / ext;
  return level < kSahMaxLevel && ext > 0.0f && ext < __builtin_inff() && scale < __builtin_inff();
}

// Plane (axis * kSahBins + first bin of its right side) of a node of two
// triangles with bins a and b, eight bits per axis (0 on an axis that cannot be
// binned): every plane between their bins costs the same, so the lowest one of the
// first axis where the bins differ.  kNoPlane where none separates them: the
// range is halved.
__host__ __device__ __forceinline__ uint32_t pair_plane(uint32_t a, uint32_t b) {
#pragma unroll
  for (uint32_t k = 0; k < 3u; ++k) {
    const uint32_t ka = (a >> (8u * k)) & 255u, kb = (b >> (8u * k)) & 255u;
    if (ka != kb) return k * kSahBins + 1u + (ka < kb ? ka : kb);
  }
  return kNoPlane;
}

}  // namespace tpmc

#endif  // TPMC_SAH_HPP
