// Sums of what several workgroups left, as device functions of 256 threads each.
#pragma once

#include "common.h"

namespace gnn {

__device__ __forceinline__ void store_partial_sum(const PartialSum& j, int64_t i, float v) {
  if (j.quads > 0) {
    if (i < 4 * j.quads) ((i & 2) == 0 ? j.c : j.c2)[i / 4 * 2 + (i & 1)] = v;
  } else if (j.c2 != nullptr && i >= j.cut) {
    j.c2[i - j.cut] = v;
  } else {
    j.c[i] = v;
  }
}

__device__ __forceinline__ void sum_partials_thin(const PartialSum& j, int64_t block, int t) {
  const int64_t i = block * 256 + t;
  if (i >= j.count) return;
  // four interleaved running sums keep four loads in flight; their order is fixed
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  int z = 0;
  for (; z + 4 <= j.parts; z += 4) {
    const float* p = j.partials + (int64_t)z * j.stride + i;
    const float v0 = p[0], v1 = p[j.stride], v2 = p[2 * j.stride], v3 = p[3 * j.stride];
    s0 += v0; s1 += v1; s2 += v2; s3 += v3;
  }
  for (; z < j.parts; ++z) s0 += j.partials[(int64_t)z * j.stride + i];
  store_partial_sum(j, i, (s0 + s1) + (s2 + s3));
}

// Same sum for short outputs and many parts: 8 threads share one output element, each
// adds every 8th part of its range (in four interleaved running sums), then the 8 subtotals are
// added in order through LDS.  `range` selects `chunk` consecutive parts, whose subtotal goes
// to row `range` of the output (a second call then adds the rows).
// The grouping is fixed, so the result is reproducible.  All threads of the workgroup have to call it; sub is [8][32].
__device__ __forceinline__ void sum_partials_wide(const PartialSum& j, int64_t block, int range, int chunk, int t, float (*sub)[32]) {
  const int col = t & 31, lane8 = t >> 5;
  const int64_t i = block * 32 + col;
  const int z0 = range * chunk;
  const int z1 = z0 + chunk < j.parts ? z0 + chunk : j.parts;
  float s = 0.f;
  if (i < j.count) {
    // four interleaved running sums keep four loads in flight; their order is fixed
    float s1 = 0.f, s2 = 0.f, s3 = 0.f;
    int z = z0 + lane8;
    for (; z + 24 < z1; z += 32) {
      const float* p = j.partials + (int64_t)z * j.stride + i;
      const float v0 = p[0], v1 = p[8 * j.stride], v2 = p[16 * j.stride], v3 = p[24 * j.stride];
      s += v0; s1 += v1; s2 += v2; s3 += v3;
    }
    for (; z < z1; z += 8) s += j.partials[(int64_t)z * j.stride + i];
    s = (s + s1) + (s2 + s3);
  }
  sub[lane8][col] = s;
  __syncthreads();
  if (lane8 == 0 && i < j.count) {
    float tot = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) tot += sub[q][col];
    store_partial_sum(j, (int64_t)range * j.count + i, tot);
  }
}

inline bool sums_wide(const PartialSum& j) { return j.count < 32768 && j.parts >= 16; }
inline unsigned sum_blocks(const PartialSum& j) { return (unsigned)cdiv(j.count, sums_wide(j) ? 32 : 256); }  // of 256 threads

}  // namespace gnn
