// k-nearest-neighbour graph of batched point clouds, built on the GPU (the EdgeConv model of
// Sec. 7.2 derives its graph from the points: k = 20 / 40 neighbours inside each cloud of a
// batch; the paper counts this construction as part of an end-to-end step).
//
// Definition: for every point the k points of its own cloud with the smallest squared
// Euclidean distance, itself included, ties towards the lower index; edges run from the
// neighbours to the point, so the result is the CSR by destination with k sources per row,
// ascending.  Floating point decides integers here, so the arithmetic is pinned down: the
// squared distance is accumulated in float32, coordinate by coordinate in index order: every
// subtraction is rounded, the first square is rounded, and each further square is added by one fused
// multiply-add.  (Written out as an intrinsic: from a product and a sum the compiler makes a fused form
// of its own choice, also out of __fmul_rn and __fadd_rn, and not the same one in every loop.)
//
// One wavefront per query point: lane l keeps the distance bits of candidates l, l+64, ... in
// registers (non-negative floats order like unsigned integers).
// The k-th smallest distance is built bit by bit from the top: a bit is set if fewer than k candidates lie below the value that has it;
// each probe is one wave-wide vote and a scalar population count per register slot, and a probe that separates exactly k
// ends the search.  Everything below is chosen, and of the candidates exactly at T the lowest indices fill up to k.  Positions
// in the output row come from the same votes (candidates before me that are chosen), which leaves the row in ascending index
// order because index = lane + 64 * slot.
//
// The votes of 16 slots in 32 probes are most of that work.  So for k <= 64 the k-th smallest of the
// 64 lanes' minima comes first, to its upper bits: at least k candidates lie at or below it, seldom more than a few
// dozen beyond, and these are packed into one or two slots (in index order) for the search proper.
// Bound by the instructions issued, some 430 to a point of 1024, a third of them to pack the candidates; occupancy (4 or 8 wavefronts a
// SIMD) and several points to a wavefront change little.  us, with a bisection between moving ends, 64-bit addresses, every slot
// checked against the cloud's end and the row pointers in a launch of their own -> this: 32 x 1024 points, k = 20
// 39 -> 23; 64 x 1024, 40 70 -> 45; 64 x 512, 30 31 -> 19; 16 x 2048, 20 59 -> 36; 48 x 200, 10 12 -> 8.
#include <algorithm>

#include "common.h"
#include "rowgroup.h"

namespace gnn {

constexpr int kKnnThreads = 256;
constexpr int kKnnWaves = kKnnThreads / kWave;
constexpr int kKnnMaxPoints = 2048;  // 32 register slots per lane
constexpr int kKnnBatch = 8;   // slots whose loads travel together
constexpr int kKnnRough = 18;  // low bits of the first bound that are not looked for: at most 2^-5 of a distance
constexpr uint32_t kKeyNone = 0xFFFFFFFFu;  // above every distance pattern

__device__ __forceinline__ int votes(unsigned long long v) { return __popcll(v); }
// lanes before this one that voted, added to n
__device__ __forceinline__ int votes_before(unsigned long long v, int n) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(v >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)v, n));
}

// The k-th smallest of the wavefront's keys, or a pattern above it that still has exactly k at or below it; LAST > 0: with
// its lowest LAST bits set instead, and no shorter search.  The counts are uniform over the wavefront, so this is scalar
// control flow.
template <int NSLOT, int LAST>
__device__ __forceinline__ uint32_t kth_smallest(const uint32_t* key, int k) {
  uint32_t T = 0u;
#pragma unroll
  for (int bit = 31; bit >= LAST; --bit) {
    const uint32_t probe = T | (1u << bit);
    int cnt = 0;
#pragma unroll
    for (int t = 0; t < NSLOT; ++t) cnt += votes(__ballot(key[t] < probe));
    if (LAST == 0 && cnt == k) return probe - 1u;
    T = cnt < k ? probe : T;
  }
  return T | ((1u << LAST) - 1u);
}

// the k nearest: every key below T, and of those at T the first ones; id ascends with (slot, lane)
template <int NSLOT>
__device__ __forceinline__ void write_nearest(const uint32_t* key, const uint32_t* id, int k, uint32_t T,
                                              int64_t base, int32_t* __restrict__ out) {
  int below = 0;
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) below += votes(__ballot(key[t] < T));
  const int ties_wanted = k - below;
  int ties_seen = 0, chosen_seen = 0;
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) {
    const bool tie = key[t] == T;
    const unsigned long long tie_vote = __ballot(tie);
    const bool chosen = key[t] < T || (tie && votes_before(tie_vote, ties_seen) < ties_wanted);
    const unsigned long long vote = __ballot(chosen);
    if (chosen) out[votes_before(vote, chosen_seen)] = (int32_t)(base + id[t]);
    ties_seen += votes(tie_vote);
    chosen_seen += votes(vote);
  }
}

// DIM: 2 or 3 coordinates (all slots' loads travel together), or 0: `dim` of them, one after the other
template <int NSLOT, int DIM>
__global__ __launch_bounds__(kKnnThreads) void k_knn(int64_t n, int points, int dim, int k, const float* __restrict__ coords,
                                                     int32_t* __restrict__ indptr, int32_t* __restrict__ indices) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t q = (int64_t)blockIdx.x * kKnnWaves + w;
  if (q == 0 && lane == 0) indptr[n] = (int32_t)(n * k);
  if (q >= n) return;  // whole wavefront
  const int64_t base = (int64_t)((uint32_t)q / (uint32_t)points) * points;
  if (lane == 0) indptr[q] = (int32_t)(q * k);
  int32_t* out = indices + q * k;
  const float* cloud = coords + base * dim;  // a scalar base, and with 2 or 3 coordinates 32-bit offsets from it
  const float* a = coords + q * dim;

  uint32_t key[NSLOT];
  auto squared_distance = [&](const float* x, const float* y) {
    float acc = 0.f;
    auto add = [&](float u, float v, bool start) {
      const float diff = u - v;
      acc = start ? diff * diff : __builtin_fmaf(diff, diff, acc);
    };
    if constexpr (DIM > 0) {
#pragma unroll
      for (int d = 0; d < DIM; ++d) add(x[d], y[d], d == 0);
    } else {
      for (int d = 0; d < dim; ++d) add(x[d], y[d], d == 0);
    }
    return __float_as_uint(acc);
  };
  // more than half of the slots are needed, so the first half is full
  constexpr int kFull = NSLOT / 2;
  int from = lane;
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) {
    const int j = from + kWave * t, at = t < kFull ? j : min(j, points - 1);  // past the cloud's end: its last point, for nothing
    const uint32_t bits = squared_distance(a, cloud + (DIM > 0 ? (uint64_t)((uint32_t)at * (uint32_t)DIM) : (uint64_t)at * dim));
    key[t] = t < kFull || j < points ? bits : kKeyNone;
    // the next slots' addresses wait for this one's distance: all 48 coordinates at once would cost wavefronts, or spill
    if ((t + 1) % kKnnBatch == 0) asm volatile("" : "+v"(from) : "v"(key[t]));
  }

  if constexpr (NSLOT >= 4) {  // more than 128 points: every lane has a candidate
    if (k <= kWave) {
      __shared__ uint2 packed[kKnnWaves][2 * kWave];  // (distance bits, candidate)
      uint32_t least = key[0];
#pragma unroll
      for (int t = 1; t < NSLOT; ++t) least = min(least, key[t]);
      const uint32_t bound = min((kth_smallest<1, kKnnRough>(&least, k)), kKeyNone - 1u);
      int cnt = 0;
#pragma unroll
      for (int t = 0; t < NSLOT; ++t) {
        const unsigned long long vote = __ballot(key[t] <= bound);
        if (key[t] <= bound)  // past two slots: anywhere, the count tells
          packed[w][min(votes_before(vote, cnt), 2 * kWave - 1)] = make_uint2(key[t], (uint32_t)(lane + kWave * t));
        cnt += votes(vote);
      }
      if (cnt <= 2 * kWave) {  // uniform over the wavefront
        wave_lds_fence();
        uint32_t near[2], id[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const bool ok = lane + kWave * t < cnt;
          const uint2 c = packed[w][lane + kWave * t];
          near[t] = ok ? c.x : kKeyNone;
          id[t] = c.y;
        }
        if (cnt <= kWave) write_nearest<1>(near, id, k, kth_smallest<1, 0>(near, k), base, out);
        else write_nearest<2>(near, id, k, kth_smallest<2, 0>(near, k), base, out);
        return;
      }
    }
  }
  uint32_t id[NSLOT];
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) id[t] = (uint32_t)(lane + kWave * t);
  write_nearest<NSLOT>(key, id, k, kth_smallest<NSLOT, 0>(key, k), base, out);
}

}  // namespace gnn

using namespace gnn;

extern "C" gnn_status_t gnn_knn_graph(int clouds, int points, int dim, int k, const float* coords,
                                      int32_t* indptr, int32_t* indices, void* stream) {
  clear_error();
  GNN_REQUIRE(clouds >= 0 && points > 0 && dim > 0 && k > 0, GNN_ERR_INVALID_ARG,
              "gnn_knn_graph: sizes must be positive");
  GNN_REQUIRE(k <= points, GNN_ERR_UNSUPPORTED, "gnn_knn_graph: k = %d exceeds the cloud size %d", k, points);
  GNN_REQUIRE(points <= kKnnMaxPoints, GNN_ERR_UNSUPPORTED, "gnn_knn_graph: %d points per cloud exceed %d",
              points, kKnnMaxPoints);
  const int64_t n = (int64_t)clouds * points;
  GNN_REQUIRE(n * k < (int64_t)INT32_MAX, GNN_ERR_UNSUPPORTED, "gnn_knn_graph: edge count does not fit 32 bits");
  GNN_REQUIRE(indptr != nullptr, GNN_ERR_INVALID_ARG, "gnn_knn_graph: indptr is null");
  hipStream_t st = static_cast<hipStream_t>(stream);
  GNN_REQUIRE(n == 0 || (coords && indices), GNN_ERR_INVALID_ARG, "gnn_knn_graph: null pointer");
  ProfScope p("knn_graph", st);
  const unsigned grid = (unsigned)std::max<int64_t>(cdiv(n, kKnnWaves), 1);  // without points: for indptr[0]
#define GNN_KNN_CASE(NSLOT_)                                                                                       \
  do {                                                                                                             \
    if (dim == 3) k_knn<NSLOT_, 3><<<grid, kKnnThreads, 0, st>>>(n, points, dim, k, coords, indptr, indices);      \
    else if (dim == 2) k_knn<NSLOT_, 2><<<grid, kKnnThreads, 0, st>>>(n, points, dim, k, coords, indptr, indices); \
    else k_knn<NSLOT_, 0><<<grid, kKnnThreads, 0, st>>>(n, points, dim, k, coords, indptr, indices);               \
  } while (0)
  const int slots = (int)cdiv(points, kWave);  // register slots a lane needs
  if (slots <= 1) GNN_KNN_CASE(1);
  else if (slots <= 2) GNN_KNN_CASE(2);
  else if (slots <= 4) GNN_KNN_CASE(4);
  else if (slots <= 8) GNN_KNN_CASE(8);
  else if (slots <= 16) GNN_KNN_CASE(16);
  else GNN_KNN_CASE(32);
#undef GNN_KNN_CASE
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}
