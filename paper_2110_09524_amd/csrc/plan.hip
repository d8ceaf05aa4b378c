// Graph plan: device-side validation of the CSR arrays, tiles (runs of vertices that no edge leaves), the CSC
// transpose (per tile, or rows filled and sorted in place, or a stable radix sort by source), and the degree order / degree
// buckets of both sides.  Integer work only; every table is a pure function of the input.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <unordered_map>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "common.h"

namespace gnn {

// largest value over the wavefront (all 64 lanes take part), then one atomic per wavefront
__device__ __forceinline__ void wave_atomic_max(int* __restrict__ dst, int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  if ((threadIdx.x & 63) == 0 && v > 0) atomicMax(dst, v);
}

// the row that contains CSR position p: the largest v with indptr[v] <= p (rows may be empty, so take the upper bound)
__device__ __forceinline__ int32_t row_of_position(const int32_t* __restrict__ indptr, int32_t p, int32_t lo, int32_t hi) {
  while (hi - lo > 1) {  // invariant: indptr[lo] <= p < indptr[hi]
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (indptr[mid] <= p) lo = mid; else hi = mid;
  }
  return lo;
}

// What the first kernels leave for the host and for those behind them, zeroed before.
struct PlanHead {
  int flags;           // errors: see the message in build()
  int max_degree[2];
  int open;            // some row is too long or reaches too far for tiles
  int arrivals;        // workgroups of k_check_rows that have finished
  int n_tiles;         // 0 without tiles
  int max_tile;
  int apart;           // there are tiles, but not all were transposed: some have too many edges or a hub
  int near, far;       // sampled edges by the distance of their ends (kNearRows)
};

// the transpose is, or will be, made tile by tile: the kernels for other graphs have nothing to do
__device__ __forceinline__ bool by_tile(const PlanHead* head, bool tried) {
  return tried && head->n_tiles != 0 && head->apart == 0;
}

// ---- validation of indptr, and tiles: runs of vertices that no edge leaves ---------------------
// A batch of point clouds is block-diagonal: no edge crosses from one cloud to the next.  Position p is a cut when
// every vertex before p hears from vertices before p only, and those from p on from p on only.  A tile starts at the first cut
// at or after each multiple of kTileRows; there are tiles if none is longer than kTileMost.  Kernels whose
// rows hear from their own tile only can hold it in LDS.
//
// One workgroup to a block of kTileRows rows, 16 lanes to a row.  It finds how far the block reaches to either side and
// which of its positions are cuts as far as its own rows go (a mask); the workgroup that arrives last
// lets the blocks' reaches veto each other's cuts and writes the tile starts.  An index outside [0, n) is
// an error here only in graphs that may have tiles, whose rows are all read; others are read edge by edge below.
// 32 768 vertices of 20 in-edges: 13 us, of which the check of indptr alone took 7.
constexpr int kTileRows = 256;
constexpr int kTileMost = 2048;
constexpr int kTileMaxInRow = 256;
constexpr int kTileMaxBlocks = 1024;  // one thread of the last workgroup to each
constexpr int kTileWords = kTileRows / 32;
struct TileBlock {
  int before;  // n - 1 - lowest vertex that the block's rows touch
  int beyond;  // highest
  uint32_t cuts[kTileWords];
};

__device__ __forceinline__ int wave_scan_max(int v, bool from_above) {  // inclusive; all 64 lanes take part
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int other = from_above ? __shfl_down(v, o, 64) : __shfl_up(v, o, 64);
    if (from_above ? lane + o < 64 : lane >= o) v = max(v, other);
  }
  return v;
}

// Exclusive scans over the first W wavefronts of a workgroup, all of whose threads call this: x is the largest `up` of
// the threads below, y the largest `down` of those above; -1 where there are none.
template <int W>
__device__ __forceinline__ int2 group_scan_max(int up, int down, int* l_up /* [W] */, int* l_down /* [W] */) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int u = wave_scan_max(up, false), d = wave_scan_max(down, true);
  if (w < W) {
    if (lane == 63) l_up[w] = u;
    if (lane == 0) l_down[w] = d;
  }
  __syncthreads();
  const int u1 = __shfl_up(u, 1, 64), d1 = __shfl_down(d, 1, 64);
  int2 r = make_int2(lane == 0 ? -1 : u1, lane == 63 ? -1 : d1);
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const int wu = l_up[i], wd = l_down[i];
    r.x = i < w && wu > r.x ? wu : r.x;
    r.y = i > w && wd > r.y ? wd : r.y;
  }
  __syncthreads();
  return r;
}

// blocks == nullptr: no tiles are looked for
__global__ __launch_bounds__(1024) void k_check_rows(int32_t n, int64_t nnz, const int32_t* __restrict__ indptr,
                                                     const int32_t* __restrict__ indices, TileBlock* __restrict__ blocks,
                                                     int32_t* __restrict__ tile_start, PlanHead* __restrict__ head) {
  __shared__ int l_before[kTileRows], l_beyond[kTileRows], l_up[16], l_down[16], l_count[16];
  __shared__ uint32_t l_cuts[kTileWords];
  __shared__ int l_flags, l_longest, l_open, l_last;
  const int t = threadIdx.x, li = t & 15, lane = t & 63, w = t >> 6;
  if (t == 0) l_flags = l_longest = l_open = l_last = 0;
  if (t < kTileWords) l_cuts[t] = 0;
  __syncthreads();
  const int64_t first = (int64_t)blockIdx.x * kTileRows;
  int longest = 0;
  // 2^32 threads are more than a launch may have: where no tiles are looked for, workgroups may take further blocks
  for (int64_t v0 = first; v0 <= n; v0 += (int64_t)gridDim.x * kTileRows) {
    constexpr int kTurns = kTileRows / 64;
    int32_t beg[kTurns], end[kTurns], near[kTurns][2];  // the first 32 sources of every row travel together
    int deg[kTurns];
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
      const int64_t v = v0 + i * 64 + (t >> 4);
      beg[i] = v <= n ? indptr[v] : 0;
      end[i] = v < n ? indptr[v + 1] : beg[i];
    }
    int flags = 0;
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
      const int64_t v = v0 + i * 64 + (t >> 4), len = (int64_t)end[i] - beg[i];
      if (v == 0 && beg[i] != 0) flags |= 1;
      if (v == n && (int64_t)beg[i] != nnz) flags |= 2;
      if (beg[i] < 0 || (int64_t)beg[i] > nnz || len < 0) flags |= 4;
      longest = max(longest, (int)min(max(len, (int64_t)0), (int64_t)INT32_MAX));
      // a row that may be read: inside [0, nnz)
      deg[i] = blocks != nullptr && v < n && beg[i] >= 0 && len >= 0 && end[i] <= nnz ? (int)len : 0;
#pragma unroll
      for (int k = 0; k < 2; ++k) near[i][k] = li + 16 * k < deg[i] ? indices[beg[i] + li + 16 * k] : (int)min(v, (int64_t)n - 1);
    }
    if (flags != 0) atomicOr(&l_flags, flags);
    bool open = longest > kTileMaxInRow;
#pragma unroll
    for (int i = 0; i < kTurns; ++i) {
      const int r = i * 64 + (t >> 4);
      int before = -1, beyond = -1;
      if (blocks != nullptr && v0 + r < n) {
        before = n - 1 - (int)(v0 + r);
        beyond = (int)(v0 + r);
        auto touch = [&](int32_t u) {
          open |= u < 0 || u >= n;
          before = max(before, n - 1 - max(u, 0));
          beyond = max(beyond, u);
        };
        touch(near[i][0]);
        touch(near[i][1]);
        if (deg[i] <= kTileMaxInRow)
          for (int j = li + 32; j < deg[i]; j += 16) touch(indices[beg[i] + j]);
      }
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        before = max(before, __shfl_xor(before, o, 64));
        beyond = max(beyond, __shfl_xor(beyond, o, 64));
      }
      if (li == 0) l_before[r] = before, l_beyond[r] = beyond;
    }
    if (open) l_open = 1;
  }
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) longest = max(longest, __shfl_xor(longest, o, 64));
  if (lane == 0 && longest > 0) atomicMax(&l_longest, longest);
  __syncthreads();
  if (t == 0) {
    if (l_flags != 0) atomicOr(&head->flags, l_flags);
    if (l_longest > 0) atomicMax(&head->max_degree[0], l_longest);
  }
  if (blocks == nullptr) return;

  // cuts as far as this block's rows go; thread r answers for the position before row r
  const bool mine = t < kTileRows;
  const int before = mine ? l_before[t] : -1, beyond = mine ? l_beyond[t] : -1;
  const int2 rest = group_scan_max<kTileRows / 64>(beyond, before, l_up, l_down);
  const int64_t p = first + t;
  if (mine && p < n && rest.x < p && n - 1 - max(rest.y, before) >= p) atomicOr(l_cuts + t / 32, 1u << (t & 31));
  if (t == kTileRows - 1) l_up[0] = max(rest.x, beyond);
  if (t == 0) l_down[0] = max(rest.y, before);
  __syncthreads();
  TileBlock* out = blocks + blockIdx.x;
  if (t == 0) {
    auto publish = [](auto* dst, auto v) { __hip_atomic_store(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    publish(&out->before, l_down[0]);
    publish(&out->beyond, l_up[0]);
#pragma unroll
    for (int i = 0; i < kTileWords; ++i) publish(out->cuts + i, l_cuts[i]);
    const bool far = l_up[0] >= first + kTileRows + kTileMost || n - 1 - l_down[0] < first - kTileMost;
    if (far || l_open || l_flags) atomicOr(&head->open, 1);
    // Everything that the last workgroup reads is written and read past the caches (relaxed, agent scope), so it is enough
    // that it has arrived; a fence would write back what the L2 holds of the kernels before.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    l_last = __hip_atomic_fetch_add(&head->arrivals, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!l_last) return;
  if (__hip_atomic_load(&head->open, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;

  // thread b: block b
  const int nb = (n + kTileRows - 1) / kTileRows;
  auto read = [](const auto* src) { return __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  const int block_beyond = t < nb ? read(&blocks[t].beyond) : -1, block_before = t < nb ? read(&blocks[t].before) : -1;
  uint32_t cuts[kTileWords];
#pragma unroll
  for (int i = 0; i < kTileWords; ++i) cuts[i] = t < nb ? read(blocks[t].cuts + i) : 0;
  const int2 others = group_scan_max<16>(block_beyond, block_before, l_up, l_down);
  int cut = n;
#pragma unroll
  for (int i = kTileWords - 1; i >= 0; --i) {
    // positions after everything that earlier blocks touch, up to the first that later ones do
    const int64_t at = (int64_t)t * kTileRows + 32 * i;
    const int64_t lo = max((int64_t)others.x + 1 - at, (int64_t)0), hi = min((int64_t)(n - 1 - others.y) - at, (int64_t)31);
    const uint32_t ok = lo > 31 || hi < lo ? 0u : (0xFFFFFFFFu << lo) & (0xFFFFFFFFu >> (31 - hi));
    if (cuts[i] & ok) cut = (int)at + __ffs((int)(cuts[i] & ok)) - 1;
  }
  // the first cut at or after this block's start, and the one at or after the next block's
  const int next = n - max(group_scan_max<16>(-1, n - cut, l_up, l_down).y, 0), start = min(cut, next);
  const bool keep = t < nb && start != next;
  int most = keep ? next - start : 0;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) most = max(most, __shfl_xor(most, o, 64));
  const unsigned long long vote = __ballot(keep);
  if (lane == 0) l_count[w] = __popcll(vote), l_up[w] = most;
  __syncthreads();
  int at = __popcll(vote & ((1ull << lane) - 1ull)), all = 0;
  for (int i = 0; i < 16; ++i) {
    if (i < w) at += l_count[i];
    all += l_count[i];
    most = max(most, l_up[i]);
  }
  if (keep) tile_start[at] = start;
  if (t == 0 && most <= kTileMost) {
    tile_start[all] = n;
    head->max_tile = most;
    head->n_tiles = all;
  }
}

// the largest out-degree; tried: k_transpose_tiles has run
// sample: 64 neighbouring rows of each of some 64 workgroups say whether their middle edge is near or far (all workgroups:
// 300 000 vertices 704 -> 723 us, a million 2905 -> 3015).  near: 2^11 rows of 512 bytes are a quarter of an L2, and of 16 384
// vertices drawn evenly less than a quarter are as near.
constexpr int kNearRows = 2048;
constexpr unsigned kNearBlocks = 64;
__global__ __launch_bounds__(256) void k_max_out_degree(int64_t count, const int32_t* __restrict__ v, bool tried, bool sample, int64_t nnz,
                                                        const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                                        PlanHead* __restrict__ head) {
  if (by_tile(head, tried)) return;
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  wave_atomic_max(&head->max_degree[1], i < count ? v[i] : 0);
  if (!sample || threadIdx.x >= 64 || blockIdx.x % max(gridDim.x / kNearBlocks, 1u) != 0) return;
  // whether indptr is sound has been looked at, but the host has yet to hear of it
  const int64_t beg = i < count ? indptr[i] : 0, end = i < count ? indptr[i + 1] : 0;
  const bool seen = 0 <= beg && beg < end && end <= nnz;
  const int64_t apart = seen ? llabs((int64_t)indices[(beg + end) / 2] - i) : 0;
  const unsigned long long far = __ballot(seen && apart >= kNearRows), near = __ballot(seen && apart < kNearRows);
  if (threadIdx.x != 0) return;
  if (near != 0) atomicAdd(&head->near, __popcll(near));
  if (far != 0) atomicAdd(&head->far, __popcll(far));
}

__global__ void k_validate_indices_and_count(int32_t n, int64_t nnz,
                                             const int32_t* __restrict__ indices,
                                             int32_t* __restrict__ outdeg, bool tried, PlanHead* __restrict__ head) {
  if (by_tile(head, tried)) return;
  int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  int32_t u = indices[e];
  if (u < 0 || u >= n) {
    atomicOr(&head->flags, 8);
    return;
  }
  atomicAdd(&outdeg[u], 1);  // integer count: the result does not depend on the order
}

__global__ void k_iota(int64_t count, int32_t* __restrict__ out) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < count) out[i] = (int32_t)i;
}

// indices_t[i] = destination row that contains CSR position eid_t[i]
__global__ void k_dst_of_position(int32_t n, int64_t nnz, const int32_t* __restrict__ indptr,
                                  const int32_t* __restrict__ eid_t, int32_t* __restrict__ indices_t) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nnz) return;
  indices_t[i] = row_of_position(indptr, eid_t[i], 0, n);
}

// ---- CSC transpose of graphs without very long out-rows: place, then sort each row ---------
// A radix sort of the edges by source is a dozen launches of a few microseconds each on a small graph
// (a k-nearest-neighbour graph of 655 000 edges, rebuilt every training step: 24 launches, 150 us on the
// device; 2 launches and 43 us here).  Every edge goes to the next free slot of its source's row, in whatever order the
// atomics fall, and one wavefront per row then sorts the row's CSR positions.  They are distinct, so
// the table is the same whatever the order was.  Sorting by counting smaller entries costs len^2 / 64
// steps and a slot counter serves one edge at a time, so long rows are left to the radix sort.  Whole
// plan, us, radix sort -> this: 5 10^3 vertices and 10^5 edges with out-degrees up to 38 189 -> 91,
// 2 10^5 edges up to 113 185 -> 133, 233 10^3 vertices and 10^7 edges up to 79 1969 -> 1511; beyond the
// limit it would lose: 10^5 edges up to 324 157 -> 240, 2 10^6 up to 1403 630 -> 2260.
constexpr int kPlaceMaxRow = 128;

// Workgroups for kernels that give several threads to a row: a launch may not have 2^32 threads along a dimension,
// so such a kernel goes on with the row gridDim.x workgroups further (2^21 workgroups of 1024 threads are 2^31).
static unsigned row_grid(int64_t n, int rows_per_block) {
  return (unsigned)std::min(cdiv(n, rows_per_block), (int64_t)1 << 21);
}

// left[u]: out-degree of u, counted down to 0 here
__device__ __forceinline__ void place_edge(int32_t e, int32_t v, const int32_t* __restrict__ indices,
                                           const int32_t* __restrict__ indptr_t, int32_t* __restrict__ left,
                                           int2* __restrict__ placed /* (CSR position, destination) */) {
  const int32_t u = indices[e];
  const int32_t slot = indptr_t[u] + atomicAdd(left + u, -1) - 1;
  placed[slot] = make_int2(e, v);
}

// 16 lanes per in-row.  A row of d edges takes d / 16 turns of 0.6 us one after the other, so graphs with a longer
// in-row than kPlaceMaxInRow go by edge.  Whole plan, us, by row -> by edge: 655 000 edges in rows of 20 145 -> 152,
// 2.6 10^6 in rows of 40 297 -> 329, 10^5 edges and one row of 256 98 -> 99, of 512 106 -> 98, of 4096 262 -> 159;
// 10^6 edges in one row 35440 -> 738 (radix sort 737).
constexpr int kPlaceMaxInRow = 256;
__global__ __launch_bounds__(256) void k_place_rows(int32_t n, const int32_t* __restrict__ indptr,
                                                    const int32_t* __restrict__ indices,
                                                    const int32_t* __restrict__ indptr_t, int32_t* __restrict__ left,
                                                    int2* __restrict__ placed) {
  const int li = threadIdx.x & 15;
  for (int64_t v = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); v < n; v += (int64_t)gridDim.x * 16) {
    const int32_t beg = indptr[v], len = indptr[v + 1] - beg;  // counted from the row's start: beg + len + 16 may
    for (int i = li; i < len; i += 16)                         // not fit 32 bits
      place_edge(beg + i, (int32_t)v, indices, indptr_t, left, placed);
  }
}

// One thread per edge: a workgroup takes kPlaceEdges consecutive edges, finds the rows of the first and the last of
// them, and its threads search between those.
constexpr int kPlaceEdges = 1024;
__global__ __launch_bounds__(256) void k_place_edges(int32_t n, int64_t nnz, const int32_t* __restrict__ indptr,
                                                     const int32_t* __restrict__ indices,
                                                     const int32_t* __restrict__ indptr_t, int32_t* __restrict__ left,
                                                     int2* __restrict__ placed) {
  const int64_t first = (int64_t)blockIdx.x * kPlaceEdges;
  const int64_t last = first + kPlaceEdges < nnz ? first + kPlaceEdges - 1 : nnz - 1;
  const int32_t r0 = row_of_position(indptr, (int32_t)first, 0, n);
  const int32_t r1 = row_of_position(indptr, (int32_t)last, r0, n);
#pragma unroll
  for (int t = 0; t < kPlaceEdges / 256; ++t) {
    const int64_t e = first + t * 256 + threadIdx.x;
    if (e <= last)
      place_edge((int32_t)e, row_of_position(indptr, (int32_t)e, r0, r1 + 1), indices, indptr_t, left, placed);
  }
}

__global__ __launch_bounds__(256) void k_sort_rows(int32_t n, const int32_t* __restrict__ indptr_t,
                                                   const int2* __restrict__ placed, int32_t* __restrict__ eid_t,
                                                   int32_t* __restrict__ indices_t) {
  const int lane = threadIdx.x & 63;
  for (int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); u < n; u += (int64_t)gridDim.x * 4) {
    const int32_t beg = indptr_t[u], len = indptr_t[u + 1] - beg;
    const int2* row = placed + beg;
    for (int i0 = 0; i0 < len; i0 += kWave) {
      const bool ok = i0 + lane < len;
      const int2 mine = ok ? row[i0 + lane] : make_int2(0, 0);
      int rank = 0;
      for (int j0 = 0; j0 < len; j0 += kWave) {
        const int other = j0 == i0 ? mine.x : j0 + lane < len ? row[j0 + lane].x : 0;
        const int cnt = min(kWave, len - j0);
        for (int j = 0; j < cnt; ++j) rank += __builtin_amdgcn_readlane(other, j) < mine.x ? 1 : 0;
      }
      if (ok) {
        eid_t[beg + rank] = mine.x;
        indices_t[beg + rank] = mine.y;
      }
    }
  }
}

// ---- CSC transpose of graphs with tiles ----------------------------------------------------------
// The edges into a tile are the edges out of it, and they are consecutive.  A workgroup takes kTransposeRows sources and
// reads the edges of the tiles that these lie in twice: first it counts each source's edges and those of smaller
// sources, then it collects the sources' edges in LDS.  There each is ranked among those of its source (16 lanes to a source)
// and goes to its place.  No global atomics, no tables in between.  32 768 vertices of 20 in-edges in tiles of 1024, us: count,
// maximum, scan, place, sort 78 -> 18; a training step that builds the plan anew 404 -> 350 with both.
// Ranking takes d * d / 16 LDS reads for a source of d edges, so longer rows are collected in order instead: the workgroup goes
// through the tiles' edges once more for each of them.  A graph in which that, or the edges of some 128 sources, is beyond
// the limits is left to the kernels for other graphs.  Whole plan, us, without tiles -> this: 64 stars of 1024 vertices 264 -> 175,
// 4 of 2040 128 -> 96, 256 of 300 244 -> 144; 16 clouds of 1024 points and 90 neighbours 492 -> 385.
constexpr int kTransposeRows = 128;
constexpr int kTransposeEdges = 12288;
constexpr int kTransposeRanked = 192;
constexpr int kTransposeReread = 1 << 18;
constexpr int kTransposeSpan = kTransposeRows + 2 * kTileMost;
typedef int int4_u __attribute__((ext_vector_type(4), aligned(4)));  // four ints at any int's address

constexpr int kTransposeThreads = 1024;

__global__ __launch_bounds__(kTransposeThreads) void k_transpose_tiles(int32_t n, int64_t nnz, const int32_t* __restrict__ indptr,
                                                         const int32_t* __restrict__ indices,
                                                         const int32_t* __restrict__ tile_start, PlanHead* __restrict__ head,
                                                         int32_t* __restrict__ indptr_t, int32_t* __restrict__ indices_t,
                                                         int32_t* __restrict__ eid_t) {
  extern __shared__ int l_edge[];  // [kTransposeEdges] positions in the tiles' list of edges, [kTransposeSpan + 1] its rows
  int* l_ptr = l_edge + kTransposeEdges;
  constexpr int kThreads = kTransposeThreads, kWaves = kThreads / 64;
  __shared__ int l_count[kTransposeRows], l_first[kTransposeRows + 1], l_less[kWaves], l_a, l_b, l_long;
  const int n_tiles = head->n_tiles;
  if (n_tiles == 0) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // neighbouring sources, which read the same edges, on one XCD; the grid is a multiple of kXcds
  const int64_t source = (int64_t)(blockIdx.x % kXcds * (gridDim.x / kXcds) + blockIdx.x / kXcds) * kTransposeRows;
  if (source >= n) return;
  const int32_t s0 = (int32_t)source, s1 = min(s0 + kTransposeRows, n);
  if (t == 0) l_a = 0, l_b = n;
  __syncthreads();
  for (int i = t; i < n_tiles; i += kThreads) {
    const int32_t start = tile_start[i];
    if (start <= s0) atomicMax(&l_a, start);
    if (start >= s1) atomicMin(&l_b, start);
  }
  __syncthreads();
  const int32_t a = l_a, b = l_b;
  const int32_t beg = indptr[a];
  const int rows = b - a, m = indptr[b] - beg;
  for (int i = t; i <= rows; i += kThreads) l_ptr[i] = indptr[a + i] - beg;
  if (t < kTransposeRows) l_count[t] = 0;
  __syncthreads();
  auto for_edges = [&](auto&& visit) {  // four fours of edges to a thread at a time
    constexpr int kFours = 4;
    int i = 4 * t;
    for (; i + 4 * kThreads * (kFours - 1) + 4 <= m; i += 4 * kThreads * kFours) {
      int4_u u[kFours];
#pragma unroll
      for (int f = 0; f < kFours; ++f) u[f] = *reinterpret_cast<const int4_u*>(indices + beg + i + 4 * kThreads * f);
#pragma unroll
      for (int f = 0; f < kFours; ++f)
#pragma unroll
        for (int k = 0; k < 4; ++k) visit(i + 4 * kThreads * f + k, u[f][k] - s0);
    }
    for (; i < m; i += 4 * kThreads) {
      int32_t u[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = i + k < m ? indices[beg + i + k] : INT32_MAX;  // beyond every source
#pragma unroll
      for (int k = 0; k < 4; ++k) visit(i + k, u[k] - s0);
    }
  };
  int less = 0;
  for_edges([&](int, int u) {
    if (u < 0) ++less;
    else if (u < kTransposeRows) atomicAdd(l_count + u, 1);
  });
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) less += __shfl_xor(less, o, 64);
  if (lane == 0) l_less[w] = less;
  __syncthreads();
  less = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) less += l_less[i];
  if (w == 0) {  // running sums of the 128 counts, two to a lane
    const int c0 = l_count[2 * lane], c1 = l_count[2 * lane + 1];
    int sum = c0 + c1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int other = __shfl_up(sum, o, 64);
      if (lane >= o) sum += other;
    }
    const int before = sum - c0 - c1;
    l_first[2 * lane] = before;
    l_first[2 * lane + 1] = before + c0;
    if (lane == 63) l_first[kTransposeRows] = sum;
    int most = max(c0, c1);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) most = max(most, __shfl_xor(most, o, 64));
    const int longer = __popcll(__ballot(c0 > kTransposeRanked)) + __popcll(__ballot(c1 > kTransposeRanked));
    if (lane == 0) {
      if (most > head->max_degree[1]) atomicMax(&head->max_degree[1], most);
      l_long = longer;
    }
  }
  __syncthreads();
  if (l_first[kTransposeRows] > kTransposeEdges || (int64_t)l_long * m > kTransposeReread) {
    if (t == 0) atomicOr(&head->apart, 1);
    return;
  }
  const int32_t to = beg + less;  // where the edges of source s0 start
  if (t < s1 - s0) indptr_t[s0 + t] = to + l_first[t];
  if (t == 0 && s1 == n) indptr_t[n] = (int32_t)nnz;
  const float per_edge = (float)rows / (float)m * 1.000001f;
  auto put = [&](int at, int edge) {
    eid_t[to + at] = beg + edge;
    int lo = (int)(edge * per_edge);  // right at once where all rows are equally long
    if (lo >= rows || edge < l_ptr[lo] || edge >= l_ptr[lo + 1]) {
      lo = 0;
      for (int hi = rows; hi - lo > 1;) {  // invariant: l_ptr[lo] <= edge < l_ptr[hi]
        const int mid = (lo + hi) >> 1;
        if (l_ptr[mid] <= edge) lo = mid; else hi = mid;
      }
    }
    indices_t[to + at] = a + lo;
  };
  for_edges([&](int i, int u) {
    if (u >= 0 && u < kTransposeRows) l_edge[l_first[u] + atomicAdd(l_count + u, -1) - 1] = i;
  });
  __syncthreads();
  for (int u = t >> 4; u < s1 - s0; u += kThreads / 16) {
    const int first = l_first[u], len = l_first[u + 1] - first;
    if (len > kTransposeRanked) continue;
    for (int i = t & 15; i < len; i += 16) {
      const int mine = l_edge[first + i];
      int rank = 0;
#pragma unroll 4
      for (int j = 0; j < len; ++j) rank += l_edge[first + j] < mine ? 1 : 0;
      put(first + rank, mine);
    }
  }
  if (l_long == 0) return;
  const int share = (m + kThreads - 1) / kThreads * 64, from = min(w * share, m), until = min(from + share, m);  // a wavefront's
  for (int u = 0; u < s1 - s0; ++u) {
    if (l_first[u + 1] - l_first[u] <= kTransposeRanked) continue;
    auto for_hits = [&](auto&& visit) {
      for (int i0 = from; i0 < until; i0 += 64) {
        const bool hit = i0 + lane < until && indices[beg + i0 + lane] == s0 + u;
        visit(i0, hit, __ballot(hit));
      }
    };
    int hits = 0;
    for_hits([&](int, bool, unsigned long long vote) { hits += __popcll(vote); });
    __syncthreads();  // the last row's counts have been read
    if (lane == 0) l_less[w] = hits;
    __syncthreads();
    int at = l_first[u];
    for (int i = 0; i < w; ++i) at += l_less[i];
    for_hits([&](int i0, bool hit, unsigned long long vote) {
      if (hit) put(at + __popcll(vote & ((1ull << lane) - 1ull)), i0 + lane);
      at += __popcll(vote);
    });
  }
}

// ---- degree order by counting: stable, descending ------------------------------------------
// One pass over blocks of 256 vertices for both sides (blockIdx.y): histograms of the degrees, laid out
// so that their running sum in memory order is the position of each (degree, block) in the order.
// Takes over from the radix sorts (two of ten launches, 55 us each) where the largest degree is below
// kCountMaxBins, so that a workgroup's counters fit its LDS, and the table of all blocks' histograms is no
// larger than a scan of a few microseconds (whole plan of 2 10^4 vertices, degrees up to 330: 240 -> 172 us).
constexpr int kCountMaxBins = 2048;
constexpr int64_t kCountMaxTable = 1 << 19;
struct DegreeSides {
  const int32_t* ptr[2];
  int32_t* bucket[2];
  int32_t* order[2];
  int4* rows[2];
};

__global__ __launch_bounds__(256) void k_degree_histograms(int32_t n, int bins, DegreeSides sides,
                                                           int32_t* __restrict__ table, int32_t* __restrict__ hist) {
  extern __shared__ int l_bins[];  // [bins]
  __shared__ int l_bucket[GNN_NUM_BUCKETS];
  const int side = blockIdx.y;
  for (int b = threadIdx.x; b < bins; b += 256) l_bins[b] = 0;
  if (threadIdx.x < GNN_NUM_BUCKETS) l_bucket[threadIdx.x] = 0;
  __syncthreads();
  const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (v < n) {
    const int d = sides.ptr[side][v + 1] - sides.ptr[side][v];
    sides.bucket[side][v] = d == 0 ? 32 : __clz(d);
    atomicAdd(l_bins + d, 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < bins; b += 256) {
    const int cnt = l_bins[b];
    table[((int64_t)side * bins + (bins - 1 - b)) * gridDim.x + blockIdx.x] = cnt;
    if (cnt != 0) atomicAdd(l_bucket + (b == 0 ? 32 : __clz(b)), cnt);
  }
  __syncthreads();
  if (threadIdx.x < GNN_NUM_BUCKETS && l_bucket[threadIdx.x] != 0)
    atomicAdd(hist + side * GNN_NUM_BUCKETS + threadIdx.x, l_bucket[threadIdx.x]);
}

__global__ __launch_bounds__(256) void k_degree_scatter(int32_t n, int bins, DegreeSides sides,
                                                        const int32_t* __restrict__ first /* exclusive sum of table */) {
  extern __shared__ int l_bins[];  // [4 wavefronts][bins]
  const int side = blockIdx.y;
  for (int b = threadIdx.x; b < 4 * bins; b += 256) l_bins[b] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const bool ok = v < n;
  const int32_t beg = ok ? sides.ptr[side][v] : 0, end = ok ? sides.ptr[side][v + 1] : -1;
  const int d = end - beg;
  int rank = 0;
  unsigned long long todo = __ballot(ok);
  while (todo) {  // uniform over the wavefront: one turn per distinct degree
    const int dd = __builtin_amdgcn_readlane(d, __ffsll((long long)todo) - 1);
    const unsigned long long same = __ballot(d == dd);
    if (d == dd) {
      rank = __popcll(same & ((1ull << lane) - 1ull));
      l_bins[w * bins + d] = __popcll(same);  // the same value from all of them
    }
    todo &= ~same;
  }
  __syncthreads();
  if (!ok) return;
  for (int q = 0; q < w; ++q) rank += l_bins[q * bins + d];
  const int64_t at = first[((int64_t)side * bins + (bins - 1 - d)) * gridDim.x + blockIdx.x] - (int64_t)side * n;
  sides.order[side][at + rank] = (int32_t)v;
  sides.rows[side][at + rank] = make_int4((int32_t)v, beg, end, 0);
}

__global__ void k_row_table(int32_t n, const int32_t* __restrict__ order, const int32_t* __restrict__ ptr,
                            int4* __restrict__ rows) {
  const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (r >= n) return;
  const int32_t v = order[r];
  rows[r] = make_int4(v, ptr[v], ptr[v + 1], 0);
}

// The histogram is counted per workgroup in LDS first, one vote per distinct bucket of a
// wavefront: graphs whose vertices all have the same degree (k-nearest-neighbour graphs) would
// otherwise send every vertex's atomic to one address.
__global__ __launch_bounds__(256) void k_degree_and_bucket(int32_t n, const int32_t* __restrict__ ptr,
                                                           uint32_t* __restrict__ deg,
                                                           int32_t* __restrict__ bucket,
                                                           int32_t* __restrict__ hist) {
  __shared__ int l_hist[GNN_NUM_BUCKETS];
  if (threadIdx.x < GNN_NUM_BUCKETS) l_hist[threadIdx.x] = 0;
  __syncthreads();
  const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const bool ok = v < n;
  int b = -1;
  if (ok) {
    const uint32_t d = (uint32_t)(ptr[v + 1] - ptr[v]);
    b = d == 0 ? 32 : __clz((int)d);
    deg[v] = d;
    bucket[v] = b;
  }
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(ok);
  while (todo) {  // uniform over the wavefront
    const int first = __ffsll((long long)todo) - 1;
    const int bb = __shfl(b, first, 64);
    const unsigned long long same = __ballot(ok && b == bb);
    if (lane == first) atomicAdd(&l_hist[bb], __popcll(same));
    todo &= ~same;
  }
  __syncthreads();
  if (threadIdx.x < GNN_NUM_BUCKETS && l_hist[threadIdx.x] != 0) atomicAdd(&hist[threadIdx.x], l_hist[threadIdx.x]);
}

// key of an edge for the column-blocked order: (block of its column) * n + its row.
// One wavefront per row, lanes strided over the row's edges (coalesced, no search).
// disorder: set where a row's edges are not in the order of their blocks.
__global__ void k_block_keys(int32_t n, int64_t nnz, const int32_t* __restrict__ ptr,
                             const int32_t* __restrict__ cols, int32_t block_cols,
                             uint64_t* __restrict__ keys, int32_t* __restrict__ counts, int32_t* __restrict__ disorder) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (row >= n) return;
  const int32_t beg = ptr[row], end = ptr[row + 1];
  // The lanes of a wavefront share the row, and within a row equal blocks usually sit next to each
  // other (sorted columns): only the first lane of a run of equal blocks adds the run's length
  // (one atomic per run instead of one per edge; integer counts, so the order does not matter).
  int32_t b_last = -1;  // of the edge before i0
  bool falls = false;
  for (int32_t i0 = beg; i0 < end; i0 += 64) {
    const int32_t i = i0 + lane;
    const bool valid = i < end;
    const int32_t b = valid ? cols[i] / block_cols : -1;
    const uint64_t key = (uint64_t)(uint32_t)b * (uint64_t)n + (uint64_t)row;
    if (valid) keys[i] = key;
    const int32_t b_prev = __shfl_up(b, 1, 64);
    falls |= valid && b < (lane == 0 ? b_last : b_prev);
    b_last = __shfl(b, 63, 64);
    const bool head = valid && (lane == 0 || b != b_prev);
    const uint64_t heads = __ballot(head);
    const int nvalid = min(64, end - i0);  // the valid lanes are a prefix
    if (head) {
      const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1);
      const int next = later != 0 ? lane + 1 + __builtin_ctzll(later) : nvalid;
      atomicAdd(&counts[key], next - lane);
    }
  }
  if (falls) *disorder = 1;
}

// bseg[b*n + r] = (bptr[b*n + row], bptr[b*n + row + 1]) with row = order[r]: the blocked
// kernels hand out rows in degree order and read their bounds with one coalesced load
__global__ void k_block_segments(int32_t n, int32_t nblk, const int32_t* __restrict__ bptr,
                                 const int32_t* __restrict__ order, int2* __restrict__ bseg) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= (int64_t)n * nblk) return;
  const int64_t b = i / n, r = i - b * n;
  const int64_t j = b * n + order[r];
  bseg[i] = make_int2(bptr[j], bptr[j + 1]);
}

// dst[i] = src[i * stride]
__global__ void k_gather_strided(int count, const int32_t* __restrict__ src, int64_t stride,
                                 int32_t* __restrict__ dst) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src[(int64_t)i * stride];
}

// ---- device memory for plan tables and temporaries ---------------------------------------
// Graphs that are rebuilt all the time (a k-nearest-neighbour graph per training step) would
// otherwise spend more time in hipMalloc / hipFree than in the plan kernels.  Blocks of up to
// 64 MB are rounded up to a power of two and, when released, kept on a free list (at most
// 512 MB in total) for the next plan of a similar size; larger blocks go straight to the
// driver.  A block is only released once nothing on the device can still touch it (the
// callers below synchronise first), so handing it out again needs no further care.
constexpr size_t kPoolMaxBlock = (size_t)64 << 20;
constexpr size_t kPoolMaxCached = (size_t)512 << 20;
static std::mutex g_pool_mu;  // guards the three objects below
static std::unordered_multimap<size_t, void*> g_pool_free;  // capacity -> idle block
static std::unordered_map<void*, size_t> g_pool_capacity;   // every pooled block, idle or in use
static size_t g_pool_cached = 0;

static void pool_trim();

static hipError_t pool_alloc(void** out, size_t bytes) {
  *out = nullptr;
  if (bytes == 0) bytes = 1;
  if (bytes > kPoolMaxBlock) {
    hipError_t e = hipMalloc(out, bytes);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      pool_trim();
      e = hipMalloc(out, bytes);
    }
    return e;
  }
  size_t cap = 256;
  while (cap < bytes) cap <<= 1;
  {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    auto it = g_pool_free.find(cap);
    if (it != g_pool_free.end()) {
      *out = it->second;
      g_pool_free.erase(it);
      g_pool_cached -= cap;
      return hipSuccess;
    }
  }
  hipError_t e = hipMalloc(out, cap);
  if (e == hipErrorOutOfMemory) {
    // idle blocks of other sizes may be what fills the device: hand them back and try once more
    (void)hipGetLastError();
    pool_trim();
    e = hipMalloc(out, cap);
  }
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    g_pool_capacity[*out] = cap;
  }
  return e;
}

// the block must be idle on the device
static void pool_free(void* p) {
  if (!p) return;
  {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    auto it = g_pool_capacity.find(p);
    if (it != g_pool_capacity.end()) {
      if (g_pool_cached + it->second <= kPoolMaxCached) {
        g_pool_free.emplace(it->second, p);
        g_pool_cached += it->second;
        return;
      }
      g_pool_capacity.erase(it);
    }
  }
  (void)hipFree(p);
}

// returns every idle block to the driver
static void pool_trim() {
  std::unordered_multimap<size_t, void*> idle;
  {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    idle.swap(g_pool_free);
    for (auto& kv : idle) g_pool_capacity.erase(kv.second);
    g_pool_cached = 0;
  }
  for (auto& kv : idle) (void)hipFree(kv.second);
}

static void free_all(gnn_graph* g) {
  if (!g) return;
  (void)hipDeviceSynchronize();  // kernels that read the tables have finished (hipFree used to wait, too)
  pool_free(g->indptr_t);
  pool_free(g->indices_t);
  pool_free(g->eid_t);
  for (int s = 0; s < 2; ++s) {
    pool_free(g->bucket_of[s]);
    pool_free(g->order[s]);
    pool_free(g->rows[s]);
    pool_free(g->bucket_offsets[s]);
    pool_free(g->bptr[s]);
    pool_free(g->bcol[s]);
    pool_free(g->bseg[s]);
  }
  pool_free(g->tile_start);
  pool_free(g->phase_clock);
  delete g;
}

struct TempBuffers {
  void* p[24] = {};
  int count = 0;
  hipStream_t st;
  explicit TempBuffers(hipStream_t stream) : st(stream) {}
  ~TempBuffers() {
    if (count) (void)hipStreamSynchronize(st);  // also on error paths: nothing may still be writing
    for (int i = 0; i < count; ++i) pool_free(p[i]);
  }
  template <typename T>
  hipError_t alloc(T** out, size_t elems) {
    void* q = nullptr;
    *out = nullptr;
    if (count == 24) return hipErrorOutOfMemory;  // more temporaries than slots: a bug, not a device state
    hipError_t e = pool_alloc(&q, elems ? elems * sizeof(T) : sizeof(T));
    if (e == hipSuccess) p[count++] = q;
    *out = static_cast<T*>(q);
    return e;
  }
};

static int bits_for(uint32_t max_value) {
  int b = 1;
  while (b < 32 && (max_value >> b) != 0) ++b;
  return b;
}

// Small results the host needs (error flags, bucket histograms, largest degrees) are copied into
// pinned memory, so that the copies are asynchronous and one wait at the end of the build
// serves all of them.  One staging block per host thread, allocated on first use and kept.
struct PlanStage {
  int32_t hist[2][GNN_NUM_BUCKETS];
  PlanHead head;
};
static PlanStage* plan_stage() {
  static thread_local PlanStage* stage = nullptr;
  if (!stage) {
    void* p = nullptr;
    if (hipHostMalloc(&p, sizeof(PlanStage), hipHostMallocDefault) != hipSuccess) return nullptr;
    stage = static_cast<PlanStage*>(p);
  }
  return stage;
}

// hist is [2][GNN_NUM_BUCKETS]; thread s serves side s
__global__ void k_bucket_offsets(const int32_t* __restrict__ hist, int32_t* __restrict__ offsets0,
                                 int32_t* __restrict__ offsets1) {
  if (threadIdx.x >= 2) return;
  const int32_t* h = hist + threadIdx.x * GNN_NUM_BUCKETS;
  int32_t* o = threadIdx.x ? offsets1 : offsets0;
  int32_t run = 0;
  o[0] = 0;
  for (int b = 0; b < GNN_NUM_BUCKETS; ++b) {
    run += h[b];
    o[b + 1] = run;
  }
}

// enqueues the degree order and buckets of one side with a radix sort; hist: the side's zeroed histogram
static gnn_status_t sort_side(gnn_graph* g, int side, const int32_t* ptr, int32_t* hist, TempBuffers& tmp,
                              hipStream_t st) {
  // the sort's keys are as wide as the largest degree (one 8-bit pass for a kNN graph instead of four)
  const int key_bits = bits_for((uint32_t)g->max_degree[side]);
  const int32_t n = g->n;
  const int thr = 256;
  uint32_t *deg = nullptr, *deg_sorted = nullptr;
  int32_t* ids = nullptr;
  GNN_HIP(tmp.alloc(&deg, n));
  GNN_HIP(tmp.alloc(&deg_sorted, n));
  GNN_HIP(tmp.alloc(&ids, n));
  k_degree_and_bucket<<<cdiv(n, thr), thr, 0, st>>>(n, ptr, deg, g->bucket_of[side], hist);
  GNN_LAUNCH_CHECK();
  k_iota<<<cdiv(n, thr), thr, 0, st>>>(n, ids);
  GNN_LAUNCH_CHECK();
  // stable descending sort by degree: ties keep ascending vertex id
  size_t bytes = 0;
  GNN_HIP(rocprim::radix_sort_pairs_desc(nullptr, bytes, deg, deg_sorted, ids, g->order[side],
                                         (size_t)n, 0, key_bits, st));
  void* scratch = nullptr;
  GNN_HIP(tmp.alloc((char**)&scratch, bytes));
  GNN_HIP(rocprim::radix_sort_pairs_desc(scratch, bytes, deg, deg_sorted, ids, g->order[side],
                                         (size_t)n, 0, key_bits, st));
  k_row_table<<<cdiv(n, thr), thr, 0, st>>>(n, g->order[side], ptr, g->rows[side]);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

// enqueues the degree orders and buckets of both sides; finish_side completes them after the wait.
// hist: [2][GNN_NUM_BUCKETS], zeroed
static gnn_status_t build_sides(gnn_graph* g, int32_t* hist, TempBuffers& tmp, PlanStage* stage, hipStream_t st) {
  const int32_t n = g->n;
  const int32_t* ptr[2] = {g->indptr, g->indptr_t};
  for (int side = 0; side < 2; ++side) {
    GNN_HIP(pool_alloc((void**)&g->bucket_of[side], sizeof(int32_t) * (n ? n : 1)));
    GNN_HIP(pool_alloc((void**)&g->order[side], sizeof(int32_t) * (n ? n : 1)));
    GNN_HIP(pool_alloc((void**)&g->rows[side], sizeof(int4) * (n ? n : 1)));
    GNN_HIP(pool_alloc((void**)&g->bucket_offsets[side], sizeof(int32_t) * (GNN_NUM_BUCKETS + 1)));
  }
  const int bins = std::max(g->max_degree[0], g->max_degree[1]) + 1;
  const int64_t blocks = cdiv(n, 256), table_len = 2 * (int64_t)bins * blocks;
  if (n > 0 && bins <= kCountMaxBins && table_len <= kCountMaxTable) {
    const DegreeSides sides{{ptr[0], ptr[1]}, {g->bucket_of[0], g->bucket_of[1]}, {g->order[0], g->order[1]},
                            {g->rows[0], g->rows[1]}};
    int32_t *table = nullptr, *first = nullptr;
    GNN_HIP(tmp.alloc(&table, (size_t)table_len));
    GNN_HIP(tmp.alloc(&first, (size_t)table_len));
    const dim3 grid((unsigned)blocks, 2);
    k_degree_histograms<<<grid, 256, sizeof(int) * bins, st>>>(n, bins, sides, table, hist);
    GNN_LAUNCH_CHECK();
    size_t bytes = 0;
    GNN_HIP(rocprim::exclusive_scan(nullptr, bytes, table, first, (int32_t)0, (size_t)table_len,
                                    rocprim::plus<int32_t>(), st));
    void* scratch = nullptr;
    GNN_HIP(tmp.alloc((char**)&scratch, bytes));
    GNN_HIP(rocprim::exclusive_scan(scratch, bytes, table, first, (int32_t)0, (size_t)table_len,
                                    rocprim::plus<int32_t>(), st));
    k_degree_scatter<<<grid, 256, 4 * sizeof(int) * bins, st>>>(n, bins, sides, first);
    GNN_LAUNCH_CHECK();
  } else if (n > 0) {
    for (int side = 0; side < 2; ++side)
      GNN_TRY(sort_side(g, side, ptr[side], hist + side * GNN_NUM_BUCKETS, tmp, st));
  }
  k_bucket_offsets<<<1, 64, 0, st>>>(hist, g->bucket_offsets[0], g->bucket_offsets[1]);
  GNN_LAUNCH_CHECK();
  GNN_HIP(hipMemcpyAsync(stage->hist, hist, sizeof(stage->hist), hipMemcpyDeviceToHost, st));
  return GNN_OK;
}

// after the stream has been waited for: the host copies of the bucket table
static void finish_side(gnn_graph* g, int side, const PlanStage* stage) {
  g->h_bucket_offsets[side][0] = 0;
  for (int b = 0; b < GNN_NUM_BUCKETS; ++b)
    g->h_bucket_offsets[side][b + 1] = g->h_bucket_offsets[side][b] + stage->hist[side][b];
}

// Column-blocked copy of one side's edge list: edges stable-sorted by
// (column / block_cols, row); bptr[b*n + r] .. bptr[b*n + r + 1] is the range of
// row r inside block b.  Only built when the vertex set spans several blocks.

// Launch groups of the column-blocked kernels.  One launch over w adjacent blocks costs, in units
// of one gathered edge per row: a fixed part (the row's running sums are read and written once,
// its segment bounds and scalars fetched) plus d * (1 + spill * log2(columns / 24576)) for its d
// edges per row, because a wider set of gathered row slices no longer sits in the L2.  Measured
// with the Reddit-scale GAT layer (1 KB rows): the per-edge part grows from 0.076 ms per million
// edges at 24576 columns to 0.099 at twice and 0.128 at four times that; the fixed part that
// gives the fastest partition is worth 8 to 12 gathered rows per row for kernels with two running
// sums (of 4, 8, 12, 16, 24 tried), about half of that with one.  The partition of the block
// sequence with the least total cost comes from a dynamic programme; it merges the sparse tail
// blocks of a power-law graph and leaves dense blocks alone.
static std::vector<int32_t> launch_groups(const std::vector<int32_t>& begin, int32_t n, int32_t block_cols,
                                          bool merge, double kFixed) {
  constexpr double kSpill = 0.32, kFitCols = 24576.0;
  const int nb = (int)begin.size() - 1;
  std::vector<int32_t> groups;
  if (nb < 1) return groups;
  if (!merge || n <= 0) {
    for (int b = 0; b <= nb; ++b) groups.push_back(b);
    return groups;
  }
  std::vector<double> best((size_t)nb + 1, 0.0);
  std::vector<int> width((size_t)nb + 1, 1);
  for (int e = 1; e <= nb; ++e) {
    best[e] = -1.0;
    for (int w = 1; w <= kMaxMerge && w <= e; ++w) {
      const double d = (double)((int64_t)begin[e] - begin[e - w]) / (double)n;
      const double over = std::log2((double)w * (double)block_cols / kFitCols);
      const double c = best[e - w] + kFixed + d * (1.0 + kSpill * (over > 0.0 ? over : 0.0));
      if (best[e] < 0.0 || c < best[e]) {
        best[e] = c;
        width[e] = w;
      }
    }
  }
  for (int e = nb; e > 0; e -= width[e]) groups.push_back(e);
  groups.push_back(0);
  std::reverse(groups.begin(), groups.end());
  return groups;
}

static gnn_status_t build_blocked(gnn_graph* g, int side, const int32_t* ptr, const int32_t* cols,
                                  hipStream_t st) {
  const int32_t n = g->n;
  const int64_t nnz = g->nnz;
  const int thr = 256;
  const int64_t slots = (int64_t)g->nblk * n;
  TempBuffers tmp(st);
  uint64_t *keys = nullptr, *keys_sorted = nullptr;
  int32_t* counts = nullptr;
  GNN_HIP(tmp.alloc(&keys, (size_t)nnz));
  GNN_HIP(tmp.alloc(&keys_sorted, (size_t)nnz));
  GNN_HIP(tmp.alloc(&counts, (size_t)slots + 1));
  GNN_HIP(pool_alloc((void**)&g->bptr[side], sizeof(int32_t) * ((size_t)slots + 1)));
  GNN_HIP(pool_alloc((void**)&g->bcol[side], sizeof(int32_t) * (size_t)nnz));
  GNN_HIP(hipMemsetAsync(counts, 0, sizeof(int32_t) * ((size_t)slots + 1), st));
  int32_t* starts = nullptr;  // of the blocks; then whether edges are out of their order
  GNN_HIP(tmp.alloc(&starts, (size_t)g->nblk + 2));
  GNN_HIP(hipMemsetAsync(starts + g->nblk + 1, 0, sizeof(int32_t), st));
  k_block_keys<<<cdiv((int64_t)n * 64, thr), thr, 0, st>>>(n, nnz, ptr, cols, g->block_cols, keys, counts, starts + g->nblk + 1);
  GNN_LAUNCH_CHECK();
  {
    size_t bytes = 0;
    GNN_HIP(rocprim::exclusive_scan(nullptr, bytes, counts, g->bptr[side], (int32_t)0,
                                    (size_t)slots + 1, rocprim::plus<int32_t>(), st));
    void* scratch = nullptr;
    GNN_HIP(tmp.alloc((char**)&scratch, bytes));
    GNN_HIP(rocprim::exclusive_scan(scratch, bytes, counts, g->bptr[side], (int32_t)0,
                                    (size_t)slots + 1, rocprim::plus<int32_t>(), st));
  }
  {
    int end_bit = 1;
    while (end_bit < 64 && ((uint64_t)(slots - 1) >> end_bit) != 0) ++end_bit;
    size_t bytes = 0;
    GNN_HIP(rocprim::radix_sort_pairs(nullptr, bytes, keys, keys_sorted, cols, g->bcol[side],
                                      (size_t)nnz, 0, end_bit, st));
    void* scratch = nullptr;
    GNN_HIP(tmp.alloc((char**)&scratch, bytes));
    GNN_HIP(rocprim::radix_sort_pairs(scratch, bytes, keys, keys_sorted, cols, g->bcol[side],
                                      (size_t)nnz, 0, end_bit, st));
  }
  GNN_HIP(pool_alloc((void**)&g->bseg[side], sizeof(int32_t) * 2 * (size_t)slots));
  k_block_segments<<<cdiv(slots, thr), thr, 0, st>>>(n, g->nblk, g->bptr[side], g->order[side],
                                                     reinterpret_cast<int2*>(g->bseg[side]));
  GNN_LAUNCH_CHECK();
  // edges per block, for the host's choice of kernel variant: bptr[b * n], b = 0 .. nblk
  g->h_block_begin[side].assign((size_t)g->nblk + 2, 0);
  k_gather_strided<<<cdiv((int64_t)g->nblk + 1, thr), thr, 0, st>>>(g->nblk + 1, g->bptr[side], n, starts);
  GNN_LAUNCH_CHECK();
  GNN_HIP(hipMemcpyAsync(g->h_block_begin[side].data(), starts, sizeof(int32_t) * ((size_t)g->nblk + 2),
                         hipMemcpyDeviceToHost, st));
  GNN_HIP(hipStreamSynchronize(st));
  g->in_block_order[side] = g->h_block_begin[side].back() == 0;
  g->h_block_begin[side].pop_back();
  const bool merge = config_get(kCfgMergeBlocks) != 0;
  g->h_group[side][0] = launch_groups(g->h_block_begin[side], n, g->block_cols, merge, 6.0);
  g->h_group[side][1] = launch_groups(g->h_block_begin[side], n, g->block_cols, merge, 10.0);
  return GNN_OK;
}

// CSC transpose of a graph that does not go by tiles; outdeg: the out-degrees, [n + 1], the last one 0
static gnn_status_t transpose(gnn_graph* g, int32_t* outdeg, TempBuffers& tmp, hipStream_t st) {
  const int32_t n = g->n;
  const int64_t nnz = g->nnz;
  const int thr = 256;
  // indptr_t = exclusive prefix sum of the out-degrees (n+1 entries; the last input is 0)
  {
    size_t bytes = 0;
    GNN_HIP(rocprim::exclusive_scan(nullptr, bytes, outdeg, g->indptr_t, (int32_t)0, (size_t)n + 1,
                                    rocprim::plus<int32_t>(), st));
    void* scratch = nullptr;
    GNN_HIP(tmp.alloc((char**)&scratch, bytes));
    GNN_HIP(rocprim::exclusive_scan(scratch, bytes, outdeg, g->indptr_t, (int32_t)0, (size_t)n + 1,
                                    rocprim::plus<int32_t>(), st));
  }
  if (nnz > 0 && g->max_degree[1] <= kPlaceMaxRow) {
    int2* placed = nullptr;
    GNN_HIP(tmp.alloc(&placed, (size_t)nnz));
    if (g->max_degree[0] <= kPlaceMaxInRow)
      k_place_rows<<<row_grid(n, 16), thr, 0, st>>>(n, g->indptr, g->indices, g->indptr_t, outdeg, placed);
    else
      k_place_edges<<<(unsigned)cdiv(nnz, kPlaceEdges), thr, 0, st>>>(n, nnz, g->indptr, g->indices, g->indptr_t,
                                                                      outdeg, placed);
    GNN_LAUNCH_CHECK();
    k_sort_rows<<<row_grid(n, 4), thr, 0, st>>>(n, g->indptr_t, placed, g->eid_t, g->indices_t);
    GNN_LAUNCH_CHECK();
  } else if (nnz > 0) {
    // stable sort of (source, CSR position): positions stay ascending inside a source
    uint32_t* keys_out = nullptr;
    int32_t* pos = nullptr;
    GNN_HIP(tmp.alloc(&keys_out, (size_t)nnz));
    GNN_HIP(tmp.alloc(&pos, (size_t)nnz));
    k_iota<<<cdiv(nnz, thr), thr, 0, st>>>(nnz, pos);
    GNN_LAUNCH_CHECK();
    const uint32_t* keys_in = reinterpret_cast<const uint32_t*>(g->indices);
    const int end_bit = bits_for(n > 0 ? (uint32_t)(n - 1) : 0u);
    size_t bytes = 0;
    GNN_HIP(rocprim::radix_sort_pairs(nullptr, bytes, keys_in, keys_out, pos, g->eid_t, (size_t)nnz,
                                      0, end_bit, st));
    void* scratch = nullptr;
    GNN_HIP(tmp.alloc((char**)&scratch, bytes));
    GNN_HIP(rocprim::radix_sort_pairs(scratch, bytes, keys_in, keys_out, pos, g->eid_t, (size_t)nnz,
                                      0, end_bit, st));
    k_dst_of_position<<<cdiv(nnz, thr), thr, 0, st>>>(n, nnz, g->indptr, g->eid_t, g->indices_t);
    GNN_LAUNCH_CHECK();
  }
  return GNN_OK;
}

static gnn_status_t build(gnn_graph* g, hipStream_t st) {
  const int32_t n = g->n;
  const int64_t nnz = g->nnz;
  const int thr = 256;
  TempBuffers tmp(st);
  PlanStage* stage = plan_stage();
  GNN_REQUIRE(stage != nullptr, GNN_ERR_HIP, "gnn_graph_create: no pinned staging memory");
  std::memset(stage, 0, sizeof(PlanStage));
  // zeroed together: head | bucket histograms | out-degrees
  int* zeroed = nullptr;
  constexpr int kHead = sizeof(PlanHead) / sizeof(int);
  // whole 256 bytes: a remainder would be a launch of its own
  const size_t zeroed_bytes = ws_granule(sizeof(int) * ((size_t)kHead + 2 * GNN_NUM_BUCKETS + n + 1));
  GNN_HIP(tmp.alloc((char**)&zeroed, zeroed_bytes));
  GNN_HIP(hipMemsetAsync(zeroed, 0, zeroed_bytes, st));
  PlanHead* head = reinterpret_cast<PlanHead*>(zeroed);
  int32_t *hist = zeroed + kHead, *outdeg = hist + 2 * GNN_NUM_BUCKETS;
  const bool look_for_tiles = nnz > 0 && cdiv(n, kTileRows) <= kTileMaxBlocks;
  TileBlock* blocks = nullptr;
  if (look_for_tiles) {
    GNN_HIP(tmp.alloc(&blocks, (size_t)n / kTileRows + 1));
    GNN_HIP(pool_alloc((void**)&g->tile_start, sizeof(int32_t) * ((size_t)cdiv(n, kTileRows) + 1)));
  }

  GNN_HIP(pool_alloc((void**)&g->indptr_t, sizeof(int32_t) * (size_t)(n + 1)));
  GNN_HIP(pool_alloc((void**)&g->indices_t, sizeof(int32_t) * (size_t)(nnz ? nnz : 1)));
  GNN_HIP(pool_alloc((void**)&g->eid_t, sizeof(int32_t) * (size_t)(nnz ? nnz : 1)));

  // one row more than there are vertices, for indptr[n]
  k_check_rows<<<row_grid((int64_t)n + 1, kTileRows), 1024, 0, st>>>(n, nnz, g->indptr, g->indices, blocks, g->tile_start, head);
  GNN_LAUNCH_CHECK();
  // more edges per vertex than this are, on average, more than a workgroup takes
  const bool transpose_tiles = look_for_tiles && nnz <= (int64_t)n * (kTransposeEdges / kTransposeRows);
  if (transpose_tiles) {
    constexpr int kLds = sizeof(int) * (kTransposeEdges + kTransposeSpan + 1);
    static std::atomic<bool> allowed{false};
    if (!allowed.load(std::memory_order_acquire)) {
      GNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_transpose_tiles),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kLds));
      allowed.store(true, std::memory_order_release);
    }
    const unsigned grid = (unsigned)(cdiv(cdiv(n, kTransposeRows), kXcds) * kXcds);
    k_transpose_tiles<<<grid, kTransposeThreads, kLds, st>>>(n, nnz, g->indptr, g->indices, g->tile_start,
                                                                            head, g->indptr_t, g->indices_t, g->eid_t);
    GNN_LAUNCH_CHECK();
  }
  if (nnz > 0) {
    k_validate_indices_and_count<<<cdiv(nnz, thr), thr, 0, st>>>(n, nnz, g->indices, outdeg, transpose_tiles, head);
    GNN_LAUNCH_CHECK();
    const bool sample = n >= kScatterRows && nnz >= kScatterDegree * (int64_t)n;
    k_max_out_degree<<<cdiv((int64_t)n, thr), thr, 0, st>>>(n, outdeg, transpose_tiles, sample, nnz, g->indptr, g->indices, head);
    GNN_LAUNCH_CHECK();
  }
  // the kernels below index with the source ids, so this one has to be waited for
  GNN_HIP(hipMemcpyAsync(&stage->head, head, sizeof(stage->head), hipMemcpyDeviceToHost, st));
  GNN_HIP(hipStreamSynchronize(st));
  const int h_bad = stage->head.flags;
  g->max_degree[0] = stage->head.max_degree[0];
  g->max_degree[1] = stage->head.max_degree[1];
  GNN_REQUIRE(h_bad == 0, GNN_ERR_BAD_GRAPH,
              "gnn_graph_create: malformed CSR (%s%s%s%s)", (h_bad & 1) ? "indptr[0] != 0; " : "",
              (h_bad & 2) ? "indptr[n] != nnz; " : "", (h_bad & 4) ? "indptr not monotone; " : "",
              (h_bad & 8) ? "source id outside [0, n)" : "");
  g->n_tiles = stage->head.n_tiles;
  g->max_tile = stage->head.max_tile;
  g->scattered = stage->head.far > stage->head.near;
  g->transposed_by_tile = transpose_tiles && g->n_tiles != 0 && stage->head.apart == 0;
  if (!g->transposed_by_tile) GNN_TRY(transpose(g, outdeg, tmp, st));
  GNN_TRY(build_sides(g, hist, tmp, stage, st));
  g->block_cols = (int32_t)config_get(kCfgBlockCols);
  g->nblk = 1;
  // the (block, row) pointer table has nblk * n entries: keep it below 2^28.  A graph too sparse
  // for the column-blocked kernels to pay (fewer than "blocked_min_edges" edges per row and block:
  // a kNN graph rebuilt every step, say) gets no lists, which are most of a small plan's launches.
  if (g->block_cols > 0 && n > g->block_cols && nnz > 0 &&
      cdiv(n, g->block_cols) * (int64_t)n < ((int64_t)1 << 28) &&
      nnz >= config_get(kCfgBlockedMinEdges) * (int64_t)n * cdiv(n, g->block_cols)) {
    g->nblk = (int32_t)cdiv(n, g->block_cols);
    GNN_TRY(build_blocked(g, 0, g->indptr, g->indices, st));
    GNN_TRY(build_blocked(g, 1, g->indptr_t, g->indices_t, st));
    GNN_HIP(pool_alloc((void**)&g->phase_clock, sizeof(int32_t) * kXcds * kClockStride));
  }
  GNN_HIP(hipStreamSynchronize(st));
  finish_side(g, 0, stage);
  finish_side(g, 1, stage);
  return GNN_OK;
}

}  // namespace gnn

using namespace gnn;

extern "C" gnn_status_t gnn_release_cached_memory(void) {
  clear_error();
  pool_trim();
  return GNN_OK;
}

extern "C" gnn_status_t gnn_graph_create(int32_t n, int64_t nnz, const int32_t* indptr,
                                         const int32_t* indices, void* stream, gnn_graph_t** graph) {
  clear_error();
  GNN_REQUIRE(graph != nullptr, GNN_ERR_INVALID_ARG, "gnn_graph_create: graph is null");
  *graph = nullptr;
  GNN_REQUIRE(n >= 0 && nnz >= 0, GNN_ERR_INVALID_ARG, "gnn_graph_create: negative size");
  GNN_REQUIRE(nnz < (int64_t)INT32_MAX, GNN_ERR_UNSUPPORTED,
              "gnn_graph_create: nnz = %lld does not fit 32-bit edge offsets", (long long)nnz);
  GNN_REQUIRE(indptr != nullptr, GNN_ERR_INVALID_ARG, "gnn_graph_create: indptr is null");
  GNN_REQUIRE(indices != nullptr || nnz == 0, GNN_ERR_INVALID_ARG,
              "gnn_graph_create: indices is null");
  gnn_graph* g = new gnn_graph();
  g->n = n;
  g->nnz = nnz;
  g->indptr = indptr;
  g->indices = indices;
  g->gcn_edge_balanced[0] = g->gcn_edge_balanced[1] = -1;
  g->gmm_edge_balanced = -1;
  g->gmm_bwd_edge_balanced[0] = g->gmm_bwd_edge_balanced[1] = -1;
  gnn_status_t s = build(g, static_cast<hipStream_t>(stream));
  if (s != GNN_OK) {
    free_all(g);
    return s;
  }
  *graph = g;
  return GNN_OK;
}

extern "C" gnn_status_t gnn_graph_destroy(gnn_graph_t* graph) {
  clear_error();
  free_all(graph);
  return GNN_OK;
}

// ---- static edge weights -----------------------------------------------------------------
__global__ void k_block_keys_only(int32_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ cols,
                                  int32_t block_cols, uint64_t* __restrict__ keys) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (row >= n) return;
  const int32_t beg = ptr[row], end = ptr[row + 1];
  for (int32_t i = beg + lane; i < end; i += 64)
    keys[i] = (uint64_t)(cols[i] / block_cols) * (uint64_t)n + (uint64_t)row;
}

__global__ void k_gather_f32(int64_t count, const int32_t* __restrict__ idx, const float* __restrict__ src,
                             float* __restrict__ dst) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src[idx[i]];
}

static void free_weights(gnn_edge_weights* w) {
  if (!w) return;
  (void)hipDeviceSynchronize();  // kernels that read the copies have finished
  for (int s = 0; s < 2; ++s) {
    pool_free(w->w_side[s]);
    pool_free(w->w_blk[s]);
  }
  delete w;
}

static gnn_status_t build_weights(gnn_edge_weights* w, const float* edge_w, hipStream_t st) {
  const gnn_graph* g = w->graph;
  const int64_t nnz = g->nnz;
  const int thr = 256;
  if (nnz == 0) return GNN_OK;
  for (int s = 0; s < 2; ++s) GNN_HIP(pool_alloc((void**)&w->w_side[s], sizeof(float) * (size_t)nnz));
  GNN_HIP(hipMemcpyAsync(w->w_side[0], edge_w, sizeof(float) * (size_t)nnz, hipMemcpyDeviceToDevice, st));
  k_gather_f32<<<(unsigned)cdiv(nnz, thr), thr, 0, st>>>(nnz, g->eid_t, edge_w, w->w_side[1]);
  GNN_LAUNCH_CHECK();
  if (g->nblk > 1) {
    // The blocked lists are a stable sort of each side's edges by (column block, row); sorting the
    // weights with the same keys and the same stable radix sort puts them in the same order.
    TempBuffers tmp(st);
    uint64_t *keys = nullptr, *keys_sorted = nullptr;
    GNN_HIP(tmp.alloc(&keys, (size_t)nnz));
    GNN_HIP(tmp.alloc(&keys_sorted, (size_t)nnz));
    const int64_t slots = (int64_t)g->nblk * g->n;
    int end_bit = 1;
    while (end_bit < 64 && ((uint64_t)(slots - 1) >> end_bit) != 0) ++end_bit;
    for (int s = 0; s < 2; ++s) {
      GNN_HIP(pool_alloc((void**)&w->w_blk[s], sizeof(float) * (size_t)nnz));
      const int32_t* ptr = s == 0 ? g->indptr : g->indptr_t;
      const int32_t* cols = s == 0 ? g->indices : g->indices_t;
      k_block_keys_only<<<(unsigned)cdiv((int64_t)g->n * 64, thr), thr, 0, st>>>(g->n, ptr, cols, g->block_cols, keys);
      GNN_LAUNCH_CHECK();
      size_t bytes = 0;
      GNN_HIP(rocprim::radix_sort_pairs(nullptr, bytes, keys, keys_sorted, w->w_side[s], w->w_blk[s],
                                        (size_t)nnz, 0, end_bit, st));
      void* scratch = nullptr;
      GNN_HIP(tmp.alloc((char**)&scratch, bytes));
      GNN_HIP(rocprim::radix_sort_pairs(scratch, bytes, keys, keys_sorted, w->w_side[s], w->w_blk[s],
                                        (size_t)nnz, 0, end_bit, st));
    }
  }
  GNN_HIP(hipStreamSynchronize(st));
  return GNN_OK;
}

extern "C" gnn_status_t gnn_edge_weights_create(const gnn_graph_t* g, const float* edge_w, void* stream,
                                                gnn_edge_weights_t** out) {
  clear_error();
  GNN_REQUIRE(g != nullptr && out != nullptr, GNN_ERR_INVALID_ARG, "gnn_edge_weights_create: null argument");
  GNN_REQUIRE(g->nnz == 0 || edge_w != nullptr, GNN_ERR_INVALID_ARG, "gnn_edge_weights_create: edge_w is null");
  *out = nullptr;
  gnn_edge_weights* w = new (std::nothrow) gnn_edge_weights();
  GNN_REQUIRE(w != nullptr, GNN_ERR_HIP, "gnn_edge_weights_create: out of host memory");
  w->graph = g;
  w->nnz = g->nnz;
  w->w_side[0] = w->w_side[1] = w->w_blk[0] = w->w_blk[1] = nullptr;
  gnn_status_t s = build_weights(w, edge_w, static_cast<hipStream_t>(stream));
  if (s != GNN_OK) {
    free_weights(w);
    return s;
  }
  *out = w;
  return GNN_OK;
}

extern "C" gnn_status_t gnn_edge_weights_destroy(gnn_edge_weights_t* w) {
  clear_error();
  free_weights(w);
  return GNN_OK;
}

extern "C" gnn_status_t gnn_graph_get_csc(const gnn_graph_t* g, int32_t* indptr_t, int32_t* indices_t,
                                          int32_t* eid_t, void* stream) {
  clear_error();
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "gnn_graph_get_csc: graph is null");
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (indptr_t)
    GNN_HIP(hipMemcpyAsync(indptr_t, g->indptr_t, sizeof(int32_t) * ((size_t)g->n + 1),
                           hipMemcpyDeviceToDevice, st));
  if (indices_t && g->nnz)
    GNN_HIP(hipMemcpyAsync(indices_t, g->indices_t, sizeof(int32_t) * (size_t)g->nnz,
                           hipMemcpyDeviceToDevice, st));
  if (eid_t && g->nnz)
    GNN_HIP(hipMemcpyAsync(eid_t, g->eid_t, sizeof(int32_t) * (size_t)g->nnz,
                           hipMemcpyDeviceToDevice, st));
  return GNN_OK;
}

extern "C" gnn_status_t gnn_graph_get_buckets(const gnn_graph_t* g, int side, int32_t* bucket_of_vertex,
                                              int32_t* order, int32_t* bucket_offsets, void* stream) {
  clear_error();
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "gnn_graph_get_buckets: graph is null");
  GNN_REQUIRE(side == 0 || side == 1, GNN_ERR_INVALID_ARG, "gnn_graph_get_buckets: side must be 0 or 1");
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (bucket_of_vertex && g->n)
    GNN_HIP(hipMemcpyAsync(bucket_of_vertex, g->bucket_of[side], sizeof(int32_t) * (size_t)g->n,
                           hipMemcpyDeviceToDevice, st));
  if (order && g->n)
    GNN_HIP(hipMemcpyAsync(order, g->order[side], sizeof(int32_t) * (size_t)g->n,
                           hipMemcpyDeviceToDevice, st));
  if (bucket_offsets)
    GNN_HIP(hipMemcpyAsync(bucket_offsets, g->bucket_offsets[side],
                           sizeof(int32_t) * (GNN_NUM_BUCKETS + 1), hipMemcpyDeviceToDevice, st));
  return GNN_OK;
}

extern "C" gnn_status_t gnn_graph_get_tiles(const gnn_graph_t* g, int32_t* n_tiles, int32_t* max_tile,
                                            int32_t* transposed_by_tile) {
  clear_error();
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "gnn_graph_get_tiles: graph is null");
  if (n_tiles) *n_tiles = g->n_tiles;
  if (max_tile) *max_tile = g->n_tiles != 0 ? g->max_tile : 0;
  if (transposed_by_tile) *transposed_by_tile = g->transposed_by_tile;
  return GNN_OK;
}

extern "C" gnn_status_t gnn_graph_get_blocked(const gnn_graph_t* g, int side, int32_t* num_blocks,
                                              int32_t* block_cols, int32_t* bptr, int32_t* bcol,
                                              void* stream) {
  clear_error();
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "gnn_graph_get_blocked: graph is null");
  GNN_REQUIRE(side == 0 || side == 1, GNN_ERR_INVALID_ARG, "gnn_graph_get_blocked: side must be 0 or 1");
  if (num_blocks) *num_blocks = g->nblk;
  if (block_cols) *block_cols = g->block_cols;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (g->nblk > 1) {
    if (bptr)
      GNN_HIP(hipMemcpyAsync(bptr, g->bptr[side], sizeof(int32_t) * ((size_t)g->nblk * g->n + 1),
                             hipMemcpyDeviceToDevice, st));
    if (bcol)
      GNN_HIP(hipMemcpyAsync(bcol, g->bcol[side], sizeof(int32_t) * (size_t)g->nnz,
                             hipMemcpyDeviceToDevice, st));
  }
  return GNN_OK;
}

extern "C" gnn_status_t gnn_graph_get_launch_groups(const gnn_graph_t* g, int side, int sums,
                                                    int32_t* groups, int32_t* count) {
  clear_error();
  GNN_REQUIRE(g != nullptr && count != nullptr, GNN_ERR_INVALID_ARG, "gnn_graph_get_launch_groups: null argument");
  GNN_REQUIRE(side == 0 || side == 1, GNN_ERR_INVALID_ARG, "gnn_graph_get_launch_groups: side must be 0 or 1");
  GNN_REQUIRE(sums == 1 || sums == 2, GNN_ERR_INVALID_ARG, "gnn_graph_get_launch_groups: sums must be 1 or 2");
  const std::vector<int32_t>& v = g->h_group[side][sums - 1];
  *count = v.empty() ? 0 : (int32_t)v.size() - 1;
  if (groups)
    for (size_t i = 0; i < v.size(); ++i) groups[i] = v[i];
  return GNN_OK;
}
