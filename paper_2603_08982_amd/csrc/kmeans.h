// What the two k-means paths (kmeans.hip, kmeans_small.hip) share.
#pragma once

#include "common.h"

namespace svgear {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kCentChunk = 64;  // the centroid tables are padded to a multiple of this

// x[row][2s + h] for s = 0..D/2-1 into xb[] (the B operand of k-step s for lane (row, h))
template <int D>
__device__ __forceinline__ void load_row_operands(const float* xr, int h, float (&xb)[D / 2]) {
#pragma unroll
  for (int t = 0; t < D / 4; ++t) {
    const float4 v = *reinterpret_cast<const float4*>(xr + 4 * t);
    xb[2 * t] = h ? v.y : v.x;
    xb[2 * t + 1] = h ? v.w : v.z;
  }
}
template <int D>
__device__ __forceinline__ void load_row_operands(const bf16_t* xr, int h, float (&xb)[D / 2]) {
#pragma unroll
  for (int t = 0; t < D / 8; ++t) {
    const uint4 v = *reinterpret_cast<const uint4*>(xr + 8 * t);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) xb[4 * t + i] = __uint_as_float(h ? (w[i] & 0xffff0000u) : (w[i] << 16));
  }
}

// Parts per cluster of the centroid update: about 128 members per part on average, at most 8.
static inline int means_parts(int64_t n, int C) {
  const int64_t p = (n / C + 64) / 128;
  return (int)(p < 1 ? 1 : (p > 8 ? 8 : p));
}

// ---- small calls (kmeans_small.hip)
// One call's arguments; tables as prep_centroids_kernel lays them out (kmeans.hip).
struct SmallKmeans {
  const void* x;
  const void* x2;
  Strides st;
  int BH, H, n, C, Cpad, iters;
  float* cent;
  float* cent2;
  int32_t* labels;
  int32_t* labels2;  // [BH][n] scratch: the labels of every second iteration
  int32_t* counts;
  float* cperm;
  float* norms;    // [BH][4 Cpad]: |c|^2, eight to a line; padding +inf
  int32_t* state;  // kSmallState int32 per head, cleared before the launch
  // the shape of the work: waves over the rows (32 each) and the centroids of a tile, tiles and update groups a
  // head, parts a cluster
  int row_waves, col_waves, tiles, groups, parts;
};
// Counters of a head, each in a cache line of its own: claimed tasks, then finished tiles and finished
// updates, eight counters each (additions to one line from all XCDs follow each other at some 57 ns).
constexpr int kSmallLine = 64, kSmallSpread = 8;
constexpr int kSmallState = kSmallLine * (1 + 2 * kSmallSpread);

constexpr int kSmallRows = 16384;  // most rows a head (the member lists of a group lie in LDS, two bytes a row)

constexpr int kSmallIterations = 1 << 16;  // most iterations (tasks are counted in 32 bits)

// Whether a call of these sizes takes the small path.
bool kmeans_small_takes(int64_t BH, int64_t nv, int C, int iters, bool bf16);
int launch_kmeans_small(SmallKmeans a, int d, bool bf16, hipStream_t s);

}  // namespace svgear
