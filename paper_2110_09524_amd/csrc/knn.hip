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
// registers (non-negative floats order like unsigned integers).  The k-th smallest distance is found
// by bisection on the 32-bit pattern; each probe counts the candidates at or below it with one
// wave-wide vote and a scalar population count per register slot, and the search ends early when a
// probe separates exactly k.  Everything below is chosen, and of the candidates exactly at T the
// lowest indices fill up to k.  Positions in the output row come from the same votes (candidates
// before me that are chosen), which leaves the row in ascending index order because index = lane +
// 64 * slot.
//
// The votes of 16 slots in 32 probes are most of that work.  So for k <= 64 the k-th smallest of the
// 64 lanes' minima comes first: at least k candidates lie at or below it, seldom more than a few
// dozen beyond, and these are packed into two slots (in index order) for the search proper.
// 32 x 1024 points, k = 20: 114 -> 45 us (84 us with the coordinates loaded one after the other).
#include "common.h"
#include "rowgroup.h"

namespace gnn {

constexpr int kKnnThreads = 256;
constexpr int kKnnQueries = kKnnThreads / kWave;
constexpr int kKnnMaxPoints = 2048;  // 32 register slots per lane
constexpr uint32_t kKeyNone = 0xFFFFFFFFu;  // above every distance pattern

// The smallest pattern with at least k of the wavefront's keys at or below it, or one above it that
// still has exactly k there; at least k keys are at or below `hi`.  The counts are uniform over the
// wavefront, so this loop is scalar control flow.
template <int NSLOT>
__device__ __forceinline__ uint32_t kth_smallest(const uint32_t* key, int k, uint32_t hi) {
  uint32_t lo = 0u;
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    int cnt = 0;
#pragma unroll
    for (int t = 0; t < NSLOT; ++t) cnt += __popcll(__ballot(key[t] <= mid));
    if (cnt == k) return mid;
    if (cnt > k) hi = mid; else lo = mid + 1u;
  }
  return lo;
}

// the k nearest: every key below T, and of those at T the first ones; id ascends with (slot, lane)
template <int NSLOT>
__device__ __forceinline__ void write_nearest(const uint32_t* key, const uint32_t* id, int k, uint32_t T,
                                              int64_t base, int32_t* __restrict__ out) {
  int below = 0;
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) below += __popcll(__ballot(key[t] < T));
  const int ties_wanted = k - below;
  const unsigned long long before_me = (1ull << (threadIdx.x & 63)) - 1ull;
  int ties_seen = 0, chosen_seen = 0;
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) {
    const bool tie = key[t] == T;
    const unsigned long long tie_vote = __ballot(tie);
    const int tie_rank = ties_seen + __popcll(tie_vote & before_me);
    const bool chosen = key[t] < T || (tie && tie_rank < ties_wanted);
    const unsigned long long vote = __ballot(chosen);
    if (chosen) out[chosen_seen + __popcll(vote & before_me)] = (int32_t)(base + id[t]);
    ties_seen += __popcll(tie_vote);
    chosen_seen += __popcll(vote);
  }
}

// DIM: 2 or 3 coordinates (all slots' loads travel together), or 0: `dim` of them, one after the other
template <int NSLOT, int DIM>
__global__ __launch_bounds__(kKnnThreads) void k_knn(int64_t n, int points, int dim, int k,
                                                     const float* __restrict__ coords,
                                                     int32_t* __restrict__ indices) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t q = (int64_t)blockIdx.x * kKnnQueries + w;
  if (q >= n) return;  // whole wavefront
  const int64_t base = q / points * points;
  const float* a = coords + q * dim;

  uint32_t key[NSLOT];
  auto squared_distance = [&](const float* p) {
    float acc = 0.f;
    auto add = [&](float x, float y, bool first) {
      const float diff = x - y;
      acc = first ? diff * diff : __builtin_fmaf(diff, diff, acc);
    };
    if constexpr (DIM > 0) {
#pragma unroll
      for (int d = 0; d < DIM; ++d) add(a[d], p[d], d == 0);
    } else {
      for (int d = 0; d < dim; ++d) add(a[d], p[d], d == 0);
    }
    return __float_as_uint(acc);
  };
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) {
    const int j = lane + kWave * t;  // past the cloud's end: its first point, for nothing
    const uint32_t bits = squared_distance(coords + (base + (j < points ? j : 0)) * dim);
    key[t] = j < points ? bits : kKeyNone;
  }

  if constexpr (NSLOT >= 4) {  // more than 128 points: every lane has a candidate
    if (k <= kWave) {
      __shared__ uint2 packed[kKnnQueries][2 * kWave];  // (distance bits, candidate)
      uint32_t least = key[0];
#pragma unroll
      for (int t = 1; t < NSLOT; ++t) least = min(least, key[t]);
      const uint32_t bound = kth_smallest<1>(&least, k, kKeyNone - 1u);
      int cnt = 0;
#pragma unroll
      for (int t = 0; t < NSLOT; ++t) cnt += __popcll(__ballot(key[t] <= bound));
      if (cnt <= 2 * kWave) {  // uniform over the wavefront
        int at = 0;
#pragma unroll
        for (int t = 0; t < NSLOT; ++t) {
          const unsigned long long vote = __ballot(key[t] <= bound);
          if (key[t] <= bound)
            packed[w][at + __popcll(vote & ((1ull << lane) - 1ull))] = make_uint2(key[t], (uint32_t)(lane + kWave * t));
          at += __popcll(vote);
        }
        wave_lds_fence();
        uint32_t near[2], id[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const bool ok = lane + kWave * t < cnt;
          const uint2 c = packed[w][lane + kWave * t];
          near[t] = ok ? c.x : kKeyNone;
          id[t] = c.y;
        }
        write_nearest<2>(near, id, k, kth_smallest<2>(near, k, bound), base, indices + q * k);
        return;
      }
    }
  }
  uint32_t id[NSLOT];
#pragma unroll
  for (int t = 0; t < NSLOT; ++t) id[t] = (uint32_t)(lane + kWave * t);
  write_nearest<NSLOT>(key, id, k, kth_smallest<NSLOT>(key, k, kKeyNone - 1u), base, indices + q * k);
}

__global__ void k_knn_indptr(int64_t n, int k, int32_t* __restrict__ indptr) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i <= n) indptr[i] = (int32_t)(i * k);
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
  ProfScope p("knn_graph", st);
  k_knn_indptr<<<(unsigned)cdiv(n + 1, 256), 256, 0, st>>>(n, k, indptr);
  GNN_LAUNCH_CHECK();
  if (n == 0) return GNN_OK;
  GNN_REQUIRE(coords && indices, GNN_ERR_INVALID_ARG, "gnn_knn_graph: null pointer");
  const unsigned grid = (unsigned)cdiv(n, kKnnQueries);
#define GNN_KNN_CASE(NSLOT_)                                                                           \
  do {                                                                                                 \
    if (dim == 3) k_knn<NSLOT_, 3><<<grid, kKnnThreads, 0, st>>>(n, points, dim, k, coords, indices);      \
    else if (dim == 2) k_knn<NSLOT_, 2><<<grid, kKnnThreads, 0, st>>>(n, points, dim, k, coords, indices); \
    else k_knn<NSLOT_, 0><<<grid, kKnnThreads, 0, st>>>(n, points, dim, k, coords, indices);               \
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
