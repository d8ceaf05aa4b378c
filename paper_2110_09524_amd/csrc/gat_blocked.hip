// Column-blocked, XCD-sliced variants of the three GAT edge kernels, for graphs whose
// projected feature matrix does not fit the L2 caches.
//
// The single-launch kernels gather one full row (heads*f floats) per edge from
// anywhere in a matrix of hundreds of MB; on MI355X each of the 8 XCDs has its own
// 4 MB L2, so nearly every gather misses and the kernels run at the speed of the
// fabric behind the L2s.  Here the same sums are re-associated so that what a
// launch gathers is cache-resident:
//   * columns are cut into 8 slices, workgroup id mod 8 picks the slice; workgroups
//     are handed to the XCDs round-robin, so XCD k only ever touches slice k of a row;
//   * the gathered vertices are cut into blocks of `block_cols`; launch b walks only
//     the edges whose gathered vertex lies in block b (plan tables bptr/bcol), so one
//     launch touches block_cols * slice_bytes per XCD (2 MB by default);
//   * per-row partial sums live in an [n, heads*f] buffer that every launch after the
//     first reads, adds to and writes back (launches on one stream run in order, so
//     there is no race and the summation order is fixed).
// The edge-softmax of the forward pass runs online across the launches: every (row, slice)
// carries its running maximum and sums from block to block and the last block normalises,
// which also yields m and d (Sec. 6: exactly the O(|V|) state that is saved).
// All per-edge values are still recomputed on the fly; nothing per-edge is stored.
#include <atomic>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>

#include <hip/hip_fp16.h>

#include "common.h"
#include "gat_common.h"
#include "row_parts.h"
#include "rowgroup.h"

namespace gnn {

constexpr int kBlkThreads = 256;
constexpr int kSlices = 8;  // column slices of a wide row: one per XCD

// How a row of HF floats is cut: `ns` slices of SL float4 each.  Wide rows (>= 1 KB) give every
// XCD its own slice.  512-byte rows keep slices of a full 128-byte line (SL = 8) and have four of
// them: workgroup id mod 4 picks the slice, so XCD k and XCD k + 4 work on the same columns (for
// different rows) and each L2 still holds one slice of the column block.  A gather of a half line
// would cost the L1 the same fill as a full one.  Rows of 256 bytes and less are not for a launch per block: at
// Reddit scale the single-launch kernels were faster there (the whole matrix then fits the
// Infinity Cache, and a launch per block costs more than it saves).  The persistent kernels do take them, with one head
// whole and with heads of 8, 16 or 32 columns that share the slice.
struct Slicing {
  int SL, ns;
  int hs = 1;  // heads that share a slice
};
static bool pick_whole_slicing(int heads, int HF, Slicing& sl) {  // every slice inside one head
  // One head of at most 64 columns: the row is a single slice of up to 256 bytes, every XCD holds the
  // whole column block (12288 x 256 bytes = 3 MB).  Only the persistent kernels take it: a launch per
  // block measured slower than the single-launch kernels here (4.04 against 3.69 ms for the source
  // side of a 1 x 64 layer at Reddit scale), its read-add-write of the sums being as large as the
  // gathered block.
  if (heads == 1 && HF <= 64 && HF % 4 == 0 && config_get(kCfgResidentSums)) {
    sl = Slicing{16, 1};
    return true;
  }
  if (HF % 32 != 0) return false;
  const int q = HF / 32;  // 128-byte lines per row
  // Slices of 256 bytes (two lines, 16 lanes) where the row has 2, 4 or 8 of them and a slice
  // stays inside one head: an edge then costs one scalar gather per two row lines instead of
  // one per line, and a launch reads its index list and row metadata half as often.  With
  // fewer than 8 slices, workgroup id mod `ns` picks the slice, so XCD k and XCD k + ns work on
  // the same columns for different rows.  Measured at 1 KB rows (Reddit-scale GAT layer):
  // 23.6 -> 21.9 ms per step against 8 slices of 128 bytes; slices of 512 bytes lose
  // (the GCN sum: 17.8 -> 17.2 ms with 256-byte slices, 22.9 ms with 512-byte ones).
  if (q % 2 == 0 && (q / 2 == 2 || q / 2 == 4 || q / 2 == 8) && (q / 2) % heads == 0) {
    sl = Slicing{16, q / 2};
    return true;
  }
  if (q >= kSlices) {
    sl = Slicing{q, kSlices};
    return (q == 8 || q == 16 || q == 32) && kSlices % heads == 0;
  }
  if (q == 4 && q % heads == 0) {
    sl = Slicing{8, q};
    return true;
  }
  sl = Slicing{q, kSlices};  // 64-byte slices, every slice inside one head
  return q == 4 && kSlices % heads == 0;
}

// Heads narrower than a slice share it: the lanes of a group then make the scores of two, four or eight heads, each lane those of the
// head it has its columns in, and the persistent kernels keep the statistics of each.  A head to a slice of 128 bytes (4 x 32, 8 x 32) or
// 64 bytes (8 x 16) fetched the lists and scalars of an edge as often per byte of row as there were slices, in a launch per block, and
// had its hub rows wait in groups of 8 or 4 lanes.  Training pass, 232 965 vertices, 1.14 10^8 edges, power law | even, ms:
// 4 x 32 12.8 -> 9.7 | 12.0 -> 10.2, 8 x 16 25.8 -> 10.0 | 24.1 -> 10.5; 22 308, 10^7: 4 x 32 2.23 -> 0.77 | 0.86 -> 0.74.
// (All that with the source side's eight heads to a slice keeping 12 of a lane's registers in scratch memory, 24 and more with rows in
// parts: the vertex states of a chunk's edges alone are 32.)
static bool pick_slicing(int heads, int HF, Slicing& sl) {
  const int f = heads > 0 ? HF / heads : 0, ns = HF / 64;
  if (config_get(kCfgResidentSums) && heads > 1 && HF % 64 == 0 && (f == 8 || f == 16 || f == 32) &&
      (ns == 1 || ns == 2 || ns == 4 || ns == 8)) {
    sl = Slicing{16, ns, 64 / f};
    return true;
  }
  return pick_whole_slicing(heads, HF, sl);
}

// ---- one column block of a weighted row aggregation ---------------------------------
// MODE 0: forward        acc[v]  += sum_e alpha_e           z[u]      (acc = out)
// MODE 1: bwd, dst side  acc[v]  += sum_e alpha_e g_e       z[u]      (acc = T), sg += sum alpha g
// MODE 2: bwd, src side  acc[u]  += sum_e alpha_e           gout[v]   (acc = dz)
//                        scal[u, slice] += sum_e alpha_e g_e (<z[u], gout[v]>_slice - [leader] D[v])
//                        The dot product is taken lane by lane: a lane multiplies its four columns
//                        of the gathered row with its four columns of z[u] (kept in registers for
//                        the whole row) and adds alpha g times that to a per-lane sum; the lanes are
//                        added once per row.  The slices of a head add up to del[u, h].
// MODE 3: forward that also stashes the destination-side sums of the backward pass:
//                        acc = out as MODE 0, acc2[v] += sum_e alpha_e g_e z[u] (= t), sg += sum alpha g
// A group of SL lanes owns (row, slice); lane li owns the float4 at column slice*4*SL + 4*li.
//
// Each group walks kRowsPerGroup consecutive rows of the degree order, software-pipelined:
// while the edges of one row are processed, the segment bounds, the first index chunk,
// the per-row scalars and the running sums of the next row are already in flight, so the
// chain of dependent loads at the start of a row is paid once per group, not once per row.
constexpr int kRowsPerGroup = 4;
// LDS floats of one group: SL gathered indices, 2 * SL edge weights, the rows of its run and
// their (begin, end) in each of the launch's blocks; a multiple of 4 keeps the 16-byte reads aligned
template <int SL>
constexpr int kBlkGroupFloats = 3 * SL + kRowsPerGroup + 2 * kRowsPerGroup * kMaxMerge;
static_assert(kBlkGroupFloats<4> % 4 == 0 && kBlkGroupFloats<8> % 4 == 0 && kBlkGroupFloats<16> % 4 == 0 &&
              kBlkGroupFloats<32> % 4 == 0, "group scratch must stay 16-byte aligned");

template <int NA>
struct BlkRow {
  int32_t row, beg, end, c_first;
  float r_a, r_m, r_d, scal;
  float4 acc[NA], acc2[NA];
};

// HALF: the gathered matrix is an fp16 copy (the sums stay fp32).  A lane then owns 8 columns
// (16 bytes of the copy) instead of 4, and a 128-byte slice covers 64 columns.
__device__ __forceinline__ void fma8_half(float4 (&acc)[2], float w, const uint4& r) {
  const __half2* h = reinterpret_cast<const __half2*>(&r);
  const float2 a = __half22float2(h[0]), b = __half22float2(h[1]), c = __half22float2(h[2]),
               d = __half22float2(h[3]);
  acc[0].x = fmaf(w, a.x, acc[0].x); acc[0].y = fmaf(w, a.y, acc[0].y);
  acc[0].z = fmaf(w, b.x, acc[0].z); acc[0].w = fmaf(w, b.y, acc[0].w);
  acc[1].x = fmaf(w, c.x, acc[1].x); acc[1].y = fmaf(w, c.y, acc[1].y);
  acc[1].z = fmaf(w, d.x, acc[1].z); acc[1].w = fmaf(w, d.y, acc[1].w);
}

__device__ __forceinline__ float dot8_half(const float4 (&zr)[2], const uint4& r) {
  const __half2* h = reinterpret_cast<const __half2*>(&r);
  const float2 a = __half22float2(h[0]), b = __half22float2(h[1]), c = __half22float2(h[2]),
               d = __half22float2(h[3]);
  return dot4(zr[0], make_float4(a.x, a.y, b.x, b.y)) + dot4(zr[1], make_float4(c.x, c.y, d.x, d.y));
}

// STAGE: the per-edge scalar el[u] of the slice's head is read from an LDS copy of the block's
// part of the head-major table instead of being gathered from L2.  Such a scalar gather
// costs a CU one 128-byte line fill per edge, as much as the 128-byte row slice itself; with
// the table in LDS the row gathers have the L1 to themselves (15 -> 24 TB/s on the bare access
// pattern).  The table takes 4 * block_cols bytes (96 KB), so one 1024-thread workgroup per CU
// runs persistently and the groups draw their rows, four at a time in degree order, from a
// per-slice counter in device memory (zeroed before the launch).
constexpr int kStageThreads = 1024;

// NARROW: 32-bit byte offsets reach every gathered row, and lanes past a segment's end gather zeros from past the table.  Before, they
// gathered the block's first row, which with weight 0 made NaN of infinities.  47 029 vertices, 2.2 10^7 edges, training pass, before -> now, us:
// 4 x 64 4240 -> 3650, 4 x 32 3765 -> 3505, 4 x 256 14 130 -> 14 120, 1 x 128 2825 -> 2925, fp16 4 x 64 4130 -> 4180; forward, 4 x 64 1985 -> 1585.
template <int SL, int MODE, bool STAGE, bool HALF, bool SKIP, bool NARROW>
__global__ __launch_bounds__(STAGE ? kStageThreads : kBlkThreads) void k_gat_blk(
    int32_t n_rows, const int32_t* __restrict__ order, const int2* __restrict__ bseg_b,
    const int32_t* __restrict__ bcol, const float* __restrict__ feat /* gathered rows: z or gout */,
    const float* __restrict__ rowfeat /* MODE 2: z, whose row u meets every gathered gout[v] */,
    const float* __restrict__ el, const float* __restrict__ er, const float* __restrict__ m_in,
    const float* __restrict__ d_in, const float4* __restrict__ vstate, int32_t col_begin,
    GatDims dm, int sph, int first, int el_hm /* el is head-major [H][n] */,
    float* __restrict__ acc_buf, float* __restrict__ acc2_buf, float* __restrict__ scal_buf,
    int32_t* __restrict__ queue /* STAGE: one row counter per slice */, int32_t cols_here,
    int32_t quads_per_grab, int ns /* column slices: 8, 4, 2 or 1 */,
    int last /* forward modes: this is the last block */,
    float4* __restrict__ state /* forward modes: running (max, sum, sum2) per (row, slice) */,
    float* __restrict__ m_out, float* __restrict__ d_out,
    int nseg /* adjacent column blocks of this launch (1 .. kMaxMerge): segment j of the row at
                position r of the degree order is bseg_b[j * n_rows + r] */,
    const float* __restrict__ alpha_b /* MODE 2, nullable: stashed signed softmax values, [H][nnz] in the
                                         order of bcol (the "fusion with stashing" arm) */,
    int64_t nnz) {
  constexpr int THREADS = STAGE ? kStageThreads : kBlkThreads;
  constexpr int G = kWave / SL;
  constexpr int GPB = THREADS / SL;
  constexpr int R = kRowsPerGroup;
  constexpr int U = SL < 8 ? 4 : 8;   // gathered rows in flight per lane
  constexpr bool DUAL = MODE == 3;  // two vector accumulators per lane
  constexpr bool SRC = MODE == 2;   // one vector accumulator, the row's own z in registers, a per-lane dot sum
  constexpr int CPL = HALF ? 8 : 4;              // columns per lane
  constexpr int NA = CPL / 4;                    // float4 accumulators per lane and sum
  // The forward modes run the edge-softmax online across the block launches: every (row, slice)
  // carries its running maximum and sums from launch to launch, the running sums are rescaled
  // when the maximum grows, and the last block divides by the denominator.  No separate pass
  // over the edges is needed for the softmax statistics.
  constexpr bool ONLINE = MODE == 0 || MODE == 3;
  constexpr int GS = kBlkGroupFloats<SL>;  // LDS floats per group: idx | p | p2 | rows | (beg, end) per row and block
  static_assert(SL >= R, "one lane per pipelined row loads its metadata");
  static_assert(!STAGE || MODE != 2, "the source side needs 16 bytes per gathered vertex");
  extern __shared__ __align__(16) float lds[];  // GPB * GS floats, then (STAGE) the el table
  (void)G;

  const int lane = threadIdx.x & 63;
  const int li = lane & (SL - 1);
  const int grp = threadIdx.x / SL;
  const int slice = blockIdx.x % ns;
  const int H = dm.H, HF = dm.HF;
  const int h = slice / sph;
  const float* l_el = lds + GPB * GS;
  // [quad, quad_end): the group's current run of row quadruples (R consecutive rows of the
  // degree order each); a staged group draws the next run from the slice's counter
  int64_t quad = 0, quad_end = 0;
  if (STAGE) {
    float* dst = lds + GPB * GS;
    const float* src = el + (int64_t)h * n_rows + col_begin;
    for (int i = threadIdx.x; i < cols_here; i += THREADS) dst[i] = src[i];
    __syncthreads();
  } else {
    quad = (int64_t)(blockIdx.x / ns) * GPB + grp;
    quad_end = quad + 1;
  }

  int* l_idx = reinterpret_cast<int*>(lds + grp * GS);
  float* l_p = lds + grp * GS + SL;
  float* l_p2 = lds + grp * GS + 2 * SL;
  int* l_row = reinterpret_cast<int*>(lds + grp * GS + 3 * SL);
  int2* l_seg = reinterpret_cast<int2*>(l_row + R);  // [R][kMaxMerge]

  const int col = slice * CPL * SL + CPL * li;
  const bool leader = (slice % sph) == 0;  // one slice per head keeps the per-head scalars

  for (;;) {
    if (STAGE && quad == quad_end) {
      // One quadruple per draw: the rows come in degree order, so consecutive quadruples of the hub
      // rows are all heavy, and a group that took several at once would be the last to finish
      // (measured on the hub block of a Reddit-scale graph: 2.7 ms with one per draw, 6.9 ms with
      // four, 4.8 ms with a static round-robin assignment).
      int q = 0;
      if (li == 0) q = atomicAdd(queue + slice, quads_per_grab);
      quad = __shfl(q, lane & ~(SL - 1), 64);
      quad_end = quad + quads_per_grab;
    }
    const int64_t r0 = quad * R;
    if (r0 >= n_rows) break;  // the counter only grows: every group ends here
    wave_lds_fence();         // the previous rows' metadata reads are done
    // segment bounds of the group's R rows inside this column block, one lane each
    if (li < R) {
      const int64_t r = r0 + li;
      int32_t row = -1;
      bool any = false;
      if (r < n_rows) row = order[r];
      for (int j = 0; j < nseg; ++j) {
        int2 seg = make_int2(0, 0);
        if (r < n_rows) seg = bseg_b[(int64_t)j * n_rows + r];
        any = any || seg.x != seg.y;
        l_seg[li * kMaxMerge + j] = seg;
      }
      if (!first && !any && !(ONLINE && last)) row = -1;  // nothing to add to this row in these blocks
      l_row[li] = row;
    }
    wave_lds_fence();

    // issue every load a row needs before its edge loop
    auto fetch = [&](int k, BlkRow<NA>& s) {
      s.row = l_row[k];
      const int2 seg0 = l_seg[k * kMaxMerge];
      s.beg = seg0.x;
      s.end = seg0.y;
      s.c_first = col_begin;
      s.r_a = 0.f; s.r_m = 0.f; s.r_d = 1.f; s.scal = 0.f;
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        s.acc[a] = make_float4(0.f, 0.f, 0.f, 0.f);
        s.acc2[a] = s.acc[a];
      }
      if (s.row < 0) return;
      if (s.beg + li < s.end) s.c_first = bcol[s.beg + li];
      const int64_t rh = (int64_t)s.row * H + h;
      if (MODE == 2) {
        s.r_a = el[rh];  // row is a source: its el
      } else if (ONLINE) {
        s.r_a = er[rh];  // row is a destination; running max, denominator, second sum so far
        s.r_m = -INFINITY;
        s.r_d = 0.f;
        if (!first) {
          const float4 stt = state[(int64_t)s.row * kSlices + slice];
          s.r_m = stt.x; s.r_d = stt.y; s.scal = stt.z;
        }
      } else {
        s.r_a = er[rh];  // row is a destination: its er, max, denominator
        s.r_m = m_in[rh];
        s.r_d = d_in[rh];
      }
      if (!first) {
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          s.acc[a] = ld4_stream(acc_buf + (int64_t)s.row * HF + col + 4 * a);
          if (DUAL) s.acc2[a] = ld4_stream(acc2_buf + (int64_t)s.row * HF + col + 4 * a);
        }
        if (MODE == 1 && leader && li == 0) s.scal = scal_buf[rh];
        if (SRC && li == 0) s.scal = scal_buf[(int64_t)s.row * kSlices + slice];
      }
      if (SRC) {
#pragma unroll
        for (int a = 0; a < NA; ++a) s.acc2[a] = ld4_stream(rowfeat + (int64_t)s.row * HF + col + 4 * a);
      }
    };

    // Gathered rows are addressed with 32-bit byte offsets when the matrix is below 4 GB
    // (one 24-bit multiply-add per row instead of 64-bit arithmetic).
    constexpr uint32_t kElem = HALF ? 2u : 4u;  // bytes per stored element of the gathered matrix
    const uint32_t row_bytes = (uint32_t)HF * kElem, col_bytes = (uint32_t)col * kElem;
    const auto table = row_table(feat, NARROW ? (int64_t)n_rows * row_bytes : 0);

    BlkRow<NA> cur, nxt;
    fetch(0, cur);
    for (int k = 0; k < R; ++k) {
      if (k + 1 < R) fetch(k + 1, nxt);
      if (cur.row >= 0) {
        const float r_a = cur.r_a, r_m = cur.r_m, r_invd = ONLINE ? 0.f : 1.f / cur.r_d;
        float4 acc[NA], acc2[NA];
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          acc[a] = cur.acc[a];
          acc2[a] = cur.acc2[a];
        }
        float s_run = 0.f;  // chunk-phase lanes: sum of alpha g (MODE 1), of alpha g D[v] (MODE 2)
        float s_dot = 0.f;  // MODE 2, row-phase lanes: sum of alpha g <z[u], gout[v]> over the lane's columns
        // online state: the running maximum is uniform in the group, the sums are per lane
        // (lane 0 carries what earlier blocks left) and are added across lanes at the end
        float m_run = cur.r_m;
        float d_lane = li == 0 ? cur.r_d : 0.f, s2_lane = li == 0 ? cur.scal : 0.f;
        int32_t beg = cur.beg, end = cur.end, c_next = cur.c_first;
        for (int sgi = 0; sgi < nseg; ++sgi) {
        // the bounds and the first indices of the row's segment in the next block are in
        // flight while this one is processed
        int32_t beg_n = 0, end_n = 0, c_first_n = col_begin;
        if (sgi + 1 < nseg) {
          const int2 sn = l_seg[k * kMaxMerge + sgi + 1];
          beg_n = sn.x;
          end_n = sn.y;
          if (beg_n + li < end_n) c_first_n = bcol[beg_n + li];
        }
        for (int32_t c0 = beg; c0 < end; c0 += SL) {
          const bool e_ok = c0 + li < end;
          const int cnt = min(SL, end - c0);  // valid edges of this chunk (uniform in the group)
          // gathered vertex of edge c0 + li; lanes past the end gather zeros and get weight 0,
          // so the row phase below needs no per-edge conditionals
          const int32_t c = e_ok ? c_next : n_rows;
          if (c0 + SL + li < end) c_next = bcol[c0 + SL + li];
          l_idx[li] = c;
          // per-edge scalars: issue the loads now, use them after the row loads are in flight
          float e_a = 0.f, a_st = 0.f;
          float4 vs = make_float4(0.f, 0.f, 1.f, 0.f);
          if (MODE == 2 && alpha_b != nullptr && e_ok) a_st = alpha_b[(int64_t)h * nnz + c0 + li];
          if (e_ok) {
            if (MODE == 2) vs = vstate[(int64_t)h * n_rows + c];  // head-major (er, m, 1/d, D) of the destination
            else e_a = STAGE ? l_el[c - col_begin] : (el_hm ? el[(int64_t)h * n_rows + c] : el[(int64_t)c * H + h]);
          }
          wave_lds_fence();
          float4 part[NA], part2[NA];
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            part[a] = make_float4(0.f, 0.f, 0.f, 0.f);
            part2[a] = part[a];
          }
          float dpart = 0.f;
          float sc = 1.f;  // ONLINE: factor that brings the running sums to this chunk's maximum
#pragma unroll
          for (int t0 = 0; t0 < SL; t0 += U) {
            // the group's U gathered vertices in one go (broadcast LDS reads), then U row loads
            int idv[U];
#pragma unroll
            for (int q = 0; q < U / 4; ++q) {
              const int4 i4 = *reinterpret_cast<const int4*>(l_idx + t0 + 4 * q);
              idv[4 * q] = i4.x; idv[4 * q + 1] = i4.y; idv[4 * q + 2] = i4.z; idv[4 * q + 3] = i4.w;
            }
            // SKIP: quadruples of gathered rows that lie entirely past the end of the segment are skipped.
            // The branches keep the compiler from issuing the second half of a chunk's loads before the first half's
            // arithmetic, and a gather past the table costs little: only slices of 128 columns, with twice as many
            // such rows to a chunk, gain (4 x 256, see above, 14 260 without -> 14 120; 4 x 64 3650 -> 4180 with it),
            // and those of 16, whose chunks are one quadruple (8 x 16, recomputing, 5010 -> 4750).
            uint4 rowv[U];  // 16 bytes of the gathered row: 4 floats, or 8 halves
#pragma unroll
            for (int t4 = 0; t4 < U; t4 += 4) {
              if (!SKIP || t0 + t4 < cnt) {
#pragma unroll
                for (int t = t4; t < t4 + 4; ++t) {
                  if constexpr (NARROW) rowv[t] = table_load<uint4>(table, idv[t], row_bytes, col_bytes);
                  else rowv[t] = table_load_wide<uint4>(feat, n_rows, idv[t], row_bytes, col_bytes);
                }
              }
            }
            if (t0 == 0) {
              float p = 0.f, p2 = 0.f;
              if (e_ok) {
                if (MODE == 2) {
                  if (alpha_b != nullptr) {  // read back instead of recomputed; D[v] is still gathered
                    p = fabsf(a_st);
                    p2 = a_st > 0.f ? p : dm.slope * p;
                  } else {
                    const float raw = r_a + vs.x;
                    p = __expf(leaky(raw, dm.slope) - vs.y) * vs.z;
                    p2 = raw > 0.f ? p : dm.slope * p;
                  }
                  s_run = fmaf(p2, vs.w, s_run);
                } else if (!ONLINE) {
                  const float raw = e_a + r_a;
                  p = __expf(leaky(raw, dm.slope) - r_m) * r_invd;
                  p = raw > 0.f ? p : dm.slope * p;  // MODE 1
                  s_run += p;
                }
              }
              if (ONLINE) {
                const float raw = e_a + r_a;
                const float sc_e = e_ok ? leaky(raw, dm.slope) : -INFINITY;
                const float m_new = fmaxf(m_run, group_max_from<SL>(sc_e, 1));  // finite: lane 0 of a chunk is valid
                sc = (m_run == -INFINITY) ? 0.f : __expf(m_run - m_new);
                p = e_ok ? __expf(sc_e - m_new) : 0.f;
                p2 = raw > 0.f ? p : dm.slope * p;
                d_lane = fmaf(d_lane, sc, p);
                s2_lane = fmaf(s2_lane, sc, p2);
                m_run = m_new;
              }
              l_p[li] = p;
              if (DUAL || SRC) l_p2[li] = p2;
              wave_lds_fence();
            }
            float pv[U], pv2[U];
#pragma unroll
            for (int q = 0; q < U / 4; ++q) {
              const float4 p4 = *reinterpret_cast<const float4*>(l_p + t0 + 4 * q);
              pv[4 * q] = p4.x; pv[4 * q + 1] = p4.y; pv[4 * q + 2] = p4.z; pv[4 * q + 3] = p4.w;
              if (DUAL || SRC) {
                const float4 q4 = *reinterpret_cast<const float4*>(l_p2 + t0 + 4 * q);
                pv2[4 * q] = q4.x; pv2[4 * q + 1] = q4.y; pv2[4 * q + 2] = q4.z; pv2[4 * q + 3] = q4.w;
              }
            }
#pragma unroll
            for (int t4 = 0; t4 < U; t4 += 4) {
              if (!SKIP || t0 + t4 < cnt) {
#pragma unroll
                for (int t = t4; t < t4 + 4; ++t) {
                  if constexpr (HALF) {
                    fma8_half(part, pv[t], rowv[t]);
                    if (DUAL) fma8_half(part2, pv2[t], rowv[t]);
                    if constexpr (SRC && NA == 2) dpart = fmaf(pv2[t], dot8_half(acc2, rowv[t]), dpart);
                  } else {
                    const float4 rv = make_float4(__uint_as_float(rowv[t].x), __uint_as_float(rowv[t].y),
                                                  __uint_as_float(rowv[t].z), __uint_as_float(rowv[t].w));
                    fma4(part[0], pv[t], rv);
                    if (DUAL) fma4(part2[0], pv2[t], rv);
                    if (SRC) dpart = fmaf(pv2[t], dot4(acc2[0], rv), dpart);
                  }
                }
              }
            }
          }
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            if (ONLINE) {
              fold4(acc[a], sc, part[a]);
              if (DUAL) fold4(acc2[a], sc, part2[a]);
            } else {
              add4(acc[a], part[a]);
              if (DUAL) add4(acc2[a], part2[a]);
            }
          }
          if (SRC) s_dot += dpart;
          // nothing is in flight here, which the compiler does not see past the branches: it would wait for the next chunk's
          // scalars before its rows
          if (SRC && SKIP) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
          wave_lds_fence();
        }
        beg = beg_n;
        end = end_n;
        c_next = c_first_n;
        }
        if (ONLINE) {
          const float d_tot = group_sum_from<SL>(d_lane, 1);
          const float s2_tot = MODE == 3 ? group_sum_from<SL>(s2_lane, 1) : 0.f;
          if (last) {
            // the row is complete: normalise (a row without in-edges keeps out = 0, m = 0, d = 1)
            const float inv = d_tot > 0.f ? 1.f / d_tot : 0.f;
#pragma unroll
            for (int a = 0; a < NA; ++a) {
              scale4(acc[a], inv);
              if (DUAL) scale4(acc2[a], inv);
            }
            if (leader && li == 0) {
              const int64_t rh = (int64_t)cur.row * H + h;
              m_out[rh] = d_tot > 0.f ? m_run : 0.f;
              d_out[rh] = d_tot > 0.f ? d_tot : 1.f;
              if (MODE == 3) scal_buf[rh] = s2_tot * inv;
            }
          } else if (li == 0) {
            state[(int64_t)cur.row * kSlices + slice] = make_float4(m_run, d_tot, s2_tot, 0.f);
          }
        }
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          st4_stream(acc_buf + (int64_t)cur.row * HF + col + 4 * a, acc[a]);
          if (DUAL) st4_stream(acc2_buf + (int64_t)cur.row * HF + col + 4 * a, acc2[a]);
        }
        if (MODE == 1 && leader) {
          const float tot = group_sum_from<SL>(s_run, 1);
          if (li == 0) scal_buf[(int64_t)cur.row * H + h] = cur.scal + tot;
        }
        if (SRC) {
          // this slice's share of del[u, h]; the D term is counted by one slice per head
          const float tot = group_sum_from<SL>(s_dot - (leader ? s_run : 0.f), 1);
          if (li == 0) scal_buf[(int64_t)cur.row * kSlices + slice] = cur.scal + tot;
        }
      }
      cur = nxt;
    }
    if (!STAGE) break;
    ++quad;
  }
}

// ---- all column blocks in one persistent launch: the running sums stay in LDS -------------------
// The launches of k_gat_blk pay for cache residency with a read-add-write of the rows' running
// sums (and softmax statistics) per block.  Here one 1024-thread workgroup per CU runs for the
// whole pass and keeps the state of gat_res_slots (row, slice) pairs in LDS: the running sums, the
// softmax statistics, the row's own scalars.  It takes all of them through column block 0, then
// all of them through block 1, ... ("phases"), writes each row out in the last phase and then
// takes its next rows ("generation").  Every workgroup of the chip owns the same number of rows
// per generation, dealt from the degree order one position at a time in alternating direction,
// so the workgroups carry nearly equal loads in every phase and walk the blocks in step by
// themselves; the workgroups of an XCD meet once per generation (phase_step_done: a bounded wait
// that only serves cache residency), so an L2 serves one block at a time.  Inside a workgroup the
// groups draw (row, slice) slots from an LDS counter, longest rows first.  The chunks of a row, or of each of its parts, are summed in the
// order of the launch-per-block kernels (blocks ascending, edges in list order), so the results do not depend on who draws what.
// MODE as k_gat_blk; one segment per phase, per-edge scalars gathered from L2 or (TAB) read from LDS.
// sum += w d for an edge; a lane without one has weight 0, but its product with the row's own z may be 0 * Inf
__device__ __forceinline__ void add_dot(bool edge, float w, float d, float& sum) {
  const float s = fmaf(w, d, sum);
  sum = edge ? s : sum;
}

constexpr int kGatResThreads = 1024;
// Groups: SL / NA lanes, each with NA float4 of the slice.  NA = 2 is for rows of an fp16 copy, which a lane then reads in 16
// instead of 8 bytes and a wavefront eight at a time: half as many gather instructions, and twice as many (row, slice) pairs share
// what a pair costs whatever its length.  GAT layer, 232 965 vertices, 1.1 10^8 edges, fin = 602, forward, ms: 4 x 64 5.93 -> 4.77;
// fin = 64, with the backward pass, 4 x 64 13.1 -> 11.9, 1 x 128 6.87 -> 6.50.  (fp32 rows, two float4 a lane, four rows in flight:
// 7.18 -> 7.69 forward, 7.77 -> 8.02 source side.)
// TAB: the block's part of el in LDS, where it leaves room for fewer rows at a time; its next part travels in registers during
// a phase.  A gathered fp16 slice is one line, its score was another.  Forward of the layers above, NA = 2 without -> with it, us: 4 x 64
// 4765 -> 4450, 1 x 128 2416 -> 2320; 60 000 vertices, 250 even edges, 4 x 64 572 -> 488 (NA = 1: 712).  With two sums a row
// (MODE 3) the rows of a batch get too few: 11.9 -> 12.1 ms a training pass, and fp32 rows 16.8 -> 17.0.
constexpr int kGatTabPerThread = 12;
// idx, p of each head, (p2) of all groups
template <int SL, int MODE, int NA, int HS>
constexpr int kGatResGroupInts = (kGatResThreads * NA / SL) * (1 + HS + (HS == 1 && (MODE == 2 || MODE == 3) ? 1 : 0)) * SL;
// a (row, slice) pair: sums (two for MODE 3) | state float4 of each head | (beg, end) of two phases | row
template <int SL, int MODE, int HS>
constexpr int kGatResSlotInts = (MODE == 3 ? 2 : 1) * 4 * SL + 4 * HS + 4 + 1;
constexpr int kGatResLdsBytes = 160 * 1024;
// Pairs a workgroup holds beside `table` ints: what the LDS leaves, a multiple of 4 so that the arrays stay 16-byte aligned
template <int SL, int MODE, int NA, int HS>
constexpr int gat_res_slots(int table) {
  constexpr int most = MODE == 3 ? 256 : 512;
  const int fit = (kGatResLdsBytes / 4 - 4 - kGatResGroupInts<SL, MODE, NA, HS> - table) / kGatResSlotInts<SL, MODE, HS>;
  return (fit < most ? fit : most) / 4 * 4;
}

// PARTS: long rows are cut into parts (has_long_rows), which are added, with their statistics, after the last phase.
template <int SL, int MODE, int NA, bool TAB, bool SKIP, bool HALF, bool NARROW, int HS, bool PARTS>
__global__ __launch_bounds__(kGatResThreads) void k_gat_res(
    int32_t n_rows, const int32_t* __restrict__ order, const int2* __restrict__ bseg /* [nblk][n_rows] */,
    const int32_t* __restrict__ bcol, const float* __restrict__ feat /* gathered rows: z or gout */,
    const float* __restrict__ rowfeat /* MODE 2: z */, const float* __restrict__ el,
    const float* __restrict__ er, const float* __restrict__ m_in, const float* __restrict__ d_in,
    const float4* __restrict__ vstate, GatDims dm, int sph, int el_hm, int32_t block_cols,
    int nblk, int ns, float* __restrict__ acc_buf, float* __restrict__ acc2_buf, float* __restrict__ scal_buf,
    float* __restrict__ m_out, float* __restrict__ d_out, int32_t* __restrict__ clock, int spin_limit, int sync_every,
    const float* __restrict__ alpha_b /* MODE 2, nullable: stashed signed softmax values, [H][nnz] in the order of
                                         bcol (the "fusion with stashing" arm) */,
    int64_t nnz, int nslot /* (row, slice) pairs the LDS holds */, RowParts cut) {
  constexpr int L = SL / NA;   // lanes of a group
  constexpr int NE = NA * HS;  // edges of a chunk that a lane makes the score of, for the head it has its columns in
  static_assert(HS == 1 || (NA == 1 && !HALF && !TAB && MODE != 1 && L % HS == 0), "shared slices: fp32 rows, no table");
  constexpr int U = SL < 8 ? 4 : 8;
  static_assert(NA == 1 || HALF, "fp32 rows: one float4 a lane");
  static_assert(!TAB || MODE != 2, "the source side needs 16 bytes per gathered vertex");
  constexpr int GPB = kGatResThreads / L;
  constexpr int GS = kGatResGroupInts<SL, MODE, NA, HS> / GPB;  // LDS ints of a group
  constexpr bool DUAL = MODE == 3;
  constexpr bool SRC = MODE == 2;
  constexpr bool ONLINE = MODE == 0 || MODE == 3;
  extern __shared__ __align__(16) int lds_gr[];
  const int lane = threadIdx.x & 63;
  const int li = threadIdx.x & (L - 1);
  const int grp = threadIdx.x / L;
  const int slice = blockIdx.x % ns;
  const int64_t nwg = gridDim.x / ns, wg = blockIdx.x / ns;  // workgroups that serve this slice
  const int H = dm.H, HF = dm.HF;
  const int hd = li % HS;  // the lane's head among those of the slice
  const int h = HS > 1 ? slice * HS + hd : slice / sph;
  const bool leader = HS > 1 || (slice % sph) == 0;  // one slice per head keeps the per-head scalars
  const int piece = hd * (L / HS) + li / HS;          // the lane's columns: a piece of its head's
  auto edge_of = [&](int a) { return li / HS + (L / HS) * a; };  // a < NE: the chunk's edges that the lane makes the scores of
  // a row narrower than its slice (a single slice of fewer than 64 columns): the lanes past its end
  // gather the row's first columns again (same cache line) and keep zeros where it matters
  const bool col_ok = slice * 4 * SL + 4 * NA * piece < HF;
  const int col = col_ok ? slice * 4 * SL + 4 * NA * piece : 0;

  float4* l_acc = reinterpret_cast<float4*>(lds_gr);                                   // [nslot][SL]
  float4* l_acc2 = l_acc + (DUAL ? SL * nslot : 0);                                    // [nslot][SL] (MODE 3)
  float4* l_state = l_acc2 + SL * nslot;                                               // [nslot][HS]
  int2* l_seg = reinterpret_cast<int2*>(l_state + HS * nslot);                         // [2][nslot]
  int* l_row = reinterpret_cast<int*>(l_seg + 2 * nslot);                              // [nslot]
  int* l_idx = l_row + nslot + grp * GS;
  float* l_p = reinterpret_cast<float*>(l_idx + SL);
  float* l_p2 = l_p + SL;                                                              // HS = 1
  int* l_cnt = l_row + nslot + GPB * GS;                                               // [2]
  float* l_tab = reinterpret_cast<float*>(l_cnt + 4);                                  // [block_cols] (TAB)
  float tab[TAB ? kGatTabPerThread : 1] = {};
  auto fetch_table = [&](int p) {
#pragma unroll
    for (int i = 0; i < (TAB ? kGatTabPerThread : 0); ++i) {
      const int c = i * kGatResThreads + threadIdx.x;
      const int64_t u = (int64_t)p * block_cols + c;
      if (c < block_cols && u < n_rows) tab[i] = el_hm ? el[(int64_t)h * n_rows + u] : el[u * H + h];
    }
  };
  auto store_table = [&]() {
#pragma unroll
    for (int i = 0; i < (TAB ? kGatTabPerThread : 0); ++i) {
      const int c = i * kGatResThreads + threadIdx.x;
      if (c < block_cols) l_tab[c] = tab[i];
    }
  };
  if constexpr (TAB) {
    fetch_table(0);
    store_table();
  }

  const int rows_here = (int)((n_rows + nwg - 1) / nwg);
  auto slots_to = [&](int j) { return PARTS ? slots_before(cut, j) : j; };
  const int all_slots = slots_to(rows_here);
  // workgroups go to the XCDs round-robin: those with the same id mod 8 share an L2
  PhaseClock pc{clock ? clock + (blockIdx.x % kXcds) * kClockStride : nullptr, (int)(gridDim.x / kXcds), spin_limit,
                false, sync_every > 0 ? sync_every : nblk};

  const bool gathers_first = ns >= 4;
  constexpr uint32_t kElem = HALF ? 2u : 4u;  // bytes per stored element of the gathered matrix
  const uint32_t row_bytes = (uint32_t)HF * kElem, col_bytes = (uint32_t)col * kElem;
  const auto table = row_table(feat, NARROW ? (int64_t)n_rows * row_bytes : 0);
  using Halves = std::conditional_t<NA == 2, uint4, uint2>;
  using RowRaw = std::conditional_t<HALF, Halves, float4>;  // a lane's columns of a gathered row
  auto widen = [](const RowRaw& r, int a) {
    if constexpr (HALF) {
      const __half2* hh = reinterpret_cast<const __half2*>(&r) + 2 * a;
      const float2 lo = __half22float2(hh[0]), hi = __half22float2(hh[1]);
      return make_float4(lo.x, lo.y, hi.x, hi.y);
    } else {
      return r;
    }
  };

  struct Item {
    int32_t beg, end, c_first[NA];
    float4 zr[NA];  // MODE 2: the row's own z slice
  };

  // a finished row, normalised and written out
  auto finish = [&](int32_t row, float4 (&acc)[NA], float4 (&acc2)[NA], const float4& st) {
    if (ONLINE) {
      // normalise (a row without in-edges keeps out = 0, m = 0, d = 1)
      const float inv = st.y > 0.f ? 1.f / st.y : 0.f;
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        scale4(acc[a], inv);
        if (DUAL) scale4(acc2[a], inv);
      }
      if (leader && li < HS) {
        const int64_t rh = (int64_t)row * H + h;
        m_out[rh] = st.y > 0.f ? st.x : 0.f;
        d_out[rh] = st.y > 0.f ? st.y : 1.f;
        if (MODE == 3) scal_buf[rh] = st.z * inv;
      }
    } else if (MODE == 1) {
      if (leader && li == 0) scal_buf[(int64_t)row * H + h] = st.x;
    } else if (li < HS) {
      scal_buf[HS > 1 ? (int64_t)row * H + h : (int64_t)row * kSlices + slice] = st.x;
    }
    if (col_ok) {
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        st4_stream(acc_buf + (int64_t)row * HF + col + 4 * a, acc[a]);
        if (DUAL) st4_stream(acc2_buf + (int64_t)row * HF + col + 4 * a, acc2[a]);
      }
    }
  };

  int phase = 0;
  for (int j0 = 0, j1; j0 < rows_here; j0 = j1) {
    // rows j0 .. j1 - 1, an even share of the slots that are left, and at least one row (its parts fit: see the launch)
    const int s0 = slots_to(j0), left = all_slots - s0, gens = (left + nslot - 1) / nslot;
    const int room = min(nslot, max((left + gens - 1) / gens, PARTS ? 1 << log_parts(cut, j0) : 1));
    j1 = PARTS ? rows_that_fit(cut, j0, rows_here, room) : min(rows_here, j0 + room);
    const int nslots = slots_to(j1) - s0;
    // (the previous generation ended with a workgroup barrier: its tables are free)
    int64_t pos = -1;                         // thread q < nslots: position of slot q's row in the degree order
    int part = 0, logp = 0;                   // and which of the row's 2^logp parts
    auto bounds = [&](int p) {                // this thread's piece of its row's segment of block p, cut at whole chunks
      if (pos < 0) return make_int2(0, 0);
      const int2 sg = bseg[(int64_t)p * n_rows + pos];
      return PARTS ? part_of_segment(sg, part, logp, SL) : sg;
    };
    if ((int)threadIdx.x < nslots) {
      const int lo = PARTS ? row_of_slot(cut, j0, j1, threadIdx.x) : j0 + threadIdx.x;
      if (PARTS) {
        part = (int)threadIdx.x - (slots_before(cut, lo) - s0);
        logp = log_parts(cut, lo);
      }
      // consecutive positions of the degree order go to consecutive workgroups, in alternating
      // direction from one round to the next, so every workgroup gets the same mix of degrees
      const int64_t r = (int64_t)lo * nwg + ((lo & 1) ? nwg - 1 - wg : wg);
      int32_t row = -1;
      int2 seg = make_int2(0, 0);
      if (r < n_rows) {
        pos = r;
        row = order[r];
        seg = bounds(0);
      }
      l_row[threadIdx.x] = PARTS && row >= 0 && logp > 0 ? -2 - row : row;  // a row in parts: below -1
      l_seg[threadIdx.x] = seg;
      // state: forward (m_run, d, s2, er[row]); MODE 1 (sum alpha g, er, m, 1/d); MODE 2 (del share, el[row])
      for (int a = 0; a < HS; ++a) {
        float4 stt = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row >= 0) {
          const int64_t rh = (int64_t)row * H + (HS > 1 ? slice * HS + a : h);
          if (ONLINE) stt = make_float4(-INFINITY, 0.f, 0.f, er[rh]);
          else if (MODE == 1) stt = make_float4(0.f, er[rh], m_in[rh], 1.f / d_in[rh]);
          else stt = make_float4(0.f, el[rh], 0.f, 0.f);
        }
        l_state[threadIdx.x * HS + a] = stt;
      }
    }
    for (int i = threadIdx.x; i < nslots * SL; i += kGatResThreads) {
      l_acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (DUAL) l_acc2[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (threadIdx.x == 0) l_cnt[0] = 0;
    __syncthreads();  // the tables are in place

    // a group's next slot of phase p, from that phase's counter
    auto grab = [&](int p) {
      int q = 0;
      if (li == 0) q = atomicAdd(l_cnt + (p & 1), 1);
      return __shfl(q, lane & ~(L - 1), 64);
    };
    // what a slot needs before its edge loop in phase p: bounds, first indices, (MODE 2) the row's own z
    auto fetch = [&](int p, int q) {
      Item it{};
      if (q >= nslots) return it;
      const int2 sg = l_seg[(p & 1) * nslot + q];
      it.beg = sg.x;
      it.end = sg.y;
#pragma unroll
      for (int a = 0; a < NA; ++a)
        if (it.beg + li + L * a < it.end) it.c_first[a] = bcol[it.beg + li + L * a];
      if (SRC) {
        const int32_t tag = l_row[q], row = PARTS && tag < -1 ? -2 - tag : tag;
        if (row >= 0 && it.beg < it.end && col_ok) {
#pragma unroll
          for (int a = 0; a < NA; ++a) it.zr[a] = ld4_stream(rowfeat + (int64_t)row * HF + col + 4 * a);
        }
      }
      return it;
    };
    int q = grab(0);
    Item cur = fetch(0, q);

    for (int p = 0; p < nblk; ++p) {
      const int32_t col_begin = p * block_cols;
      const bool last = p + 1 == nblk;
      // the next phase's bounds travel while this one is worked on
      int2 seg_next = make_int2(0, 0);
      if (!last) seg_next = bounds(p + 1);
      if (threadIdx.x == 0) l_cnt[(p + 1) & 1] = 0;
      if constexpr (TAB) fetch_table(last ? 0 : p + 1);

      while (q < nslots) {
        const int qn = grab(p);
        const Item nxt = fetch(p, qn);
        const int32_t row = l_row[q];  // a row in parts is finished after the last phase
        const int32_t beg = cur.beg, end = cur.end;
        const bool ends = last && (!PARTS || row >= 0);
        if (row != -1 && (beg < end || ends)) {
          const float4 stt = l_state[q * HS + hd];
          float4 acc[NA], acc2[NA];
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            acc[a] = l_acc[q * SL + li + L * a];
            acc2[a] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (DUAL) acc2[a] = l_acc2[q * SL + li + L * a];
            if (SRC) acc2[a] = cur.zr[a];
          }
          const float r_a = ONLINE ? stt.w : stt.y;
          const float r_m = stt.z, r_invd = stt.w;  // MODE 1
          float s_run[NA], s_dot[NA], d_lane[NA], s2_lane[NA];
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            s_run[a] = 0.f;  // chunk-phase lanes: sum of alpha g (MODE 1), of alpha g D[v] (MODE 2)
            s_dot[a] = 0.f;  // MODE 2, row-phase lanes: sum of alpha g <z[u], gout[v]> over the lane's columns
            d_lane[a] = li < HS && a == 0 ? stt.y : 0.f;
            s2_lane[a] = li < HS && a == 0 ? stt.z : 0.f;
          }
          float m_run = stt.x;  // ONLINE
          int32_t c_next[NA];
#pragma unroll
          for (int a = 0; a < NA; ++a) c_next[a] = cur.c_first[a];
          for (int32_t c0 = beg; c0 < end; c0 += SL) {
            const int cnt = min(SL, end - c0);
            bool e_ok[NE];
            float e_a[NE], a_st[NE];
            float4 vs[NE];
            int32_t ce[NE];  // the vertices at the far end of the lane's edges
#pragma unroll
            for (int a = 0; a < NA; ++a) {
              const int32_t c = li + L * a < cnt ? c_next[a] : n_rows;  // no edge: zeros
              if (c0 + SL + li + L * a < end) c_next[a] = bcol[c0 + SL + li + L * a];
              l_idx[li + L * a] = c;
              ce[a] = c;
            }
            if constexpr (HS > 1) {
              wave_lds_fence();
#pragma unroll
              for (int a = 0; a < NE; ++a) ce[a] = l_idx[edge_of(a)];
            }
#pragma unroll
            for (int a = 0; a < NE; ++a) {
              e_ok[a] = edge_of(a) < cnt;
              e_a[a] = 0.f;
              a_st[a] = 0.f;
              vs[a] = make_float4(0.f, 0.f, 1.f, 0.f);
              if (SRC && alpha_b != nullptr && e_ok[a]) a_st[a] = alpha_b[(int64_t)h * nnz + c0 + edge_of(a)];
              if (e_ok[a]) {
                // (er, m, 1/d, D) of the destination: head-major, or the heads of a slice side by side
                if (SRC) vs[a] = vstate[HS > 1 ? (int64_t)ce[a] * H + h : (int64_t)h * n_rows + ce[a]];
                else if constexpr (TAB) e_a[a] = l_tab[ce[a] - col_begin];
                else e_a[a] = el_hm ? el[(int64_t)h * n_rows + ce[a]] : el[(int64_t)ce[a] * H + h];
              }
            }
            if constexpr (HS == 1) wave_lds_fence();
            float4 part[NA], part2[NA];
            float dpart[NA];
#pragma unroll
            for (int a = 0; a < NA; ++a) {
              part[a] = make_float4(0.f, 0.f, 0.f, 0.f);
              part2[a] = part[a];
              dpart[a] = 0.f;
            }
            float sc = 1.f;  // ONLINE: factor that brings the running sums to this chunk's maximum
#pragma unroll
            for (int t0 = 0; t0 < SL; t0 += U) {
              if (SKIP && t0 >= cnt) break;  // nothing of this chunk is left: no index or weight reads either
              int idv[U];
#pragma unroll
              for (int qq = 0; qq < U / 4; ++qq) {
                const int4 i4 = *reinterpret_cast<const int4*>(l_idx + t0 + 4 * qq);
                idv[4 * qq] = i4.x; idv[4 * qq + 1] = i4.y; idv[4 * qq + 2] = i4.z; idv[4 * qq + 3] = i4.w;
              }
              RowRaw rowv[U];
              // a wavefront that is about to issue its gathers goes first on its SIMD (measured on rows of
              // four slices: 7.29 -> 7.16 ms forward, 7.84 -> 7.77 ms source side; rows of one or two slices
              // lose 1-2 % with it)
              if (gathers_first) __builtin_amdgcn_s_setprio(3);
#pragma unroll
              for (int t4 = 0; t4 < U; t4 += 4) {
                if (!SKIP || t0 + t4 < cnt) {
#pragma unroll
                  for (int t = t4; t < t4 + 4; ++t) {
                    if constexpr (NARROW) rowv[t] = table_load<RowRaw>(table, idv[t], row_bytes, col_bytes);
                    else rowv[t] = table_load_wide<RowRaw>(feat, n_rows, idv[t], row_bytes, col_bytes);
                  }
                }
              }
              if (gathers_first) __builtin_amdgcn_s_setprio(0);
              if (t0 == 0) {
                float pe[NE], pe2[NE];
                if (ONLINE) {
                  float raw[NE], sc_e[NE], top = -INFINITY;
#pragma unroll
                  for (int a = 0; a < NE; ++a) {
                    raw[a] = e_a[a] + r_a;
                    sc_e[a] = e_ok[a] ? leaky(raw[a], dm.slope) : -INFINITY;
                    top = fmaxf(top, sc_e[a]);
                  }
                  const float m_new = fmaxf(m_run, group_max_from<L>(top, HS));  // finite: a chunk's first edge is valid
                  sc = (m_run == -INFINITY) ? 0.f : __expf(m_run - m_new);
#pragma unroll
                  for (int a = 0; a < NE; ++a) {
                    pe[a] = e_ok[a] ? __expf(sc_e[a] - m_new) : 0.f;
                    pe2[a] = raw[a] > 0.f ? pe[a] : dm.slope * pe[a];
                  }
#pragma unroll
                  for (int a = 0; a < NA; ++a) {
                    float dsum = pe[a], s2sum = pe2[a];
#pragma unroll
                    for (int j = 1; j < HS; ++j) {
                      dsum += pe[a + NA * j];
                      s2sum += pe2[a + NA * j];
                    }
                    d_lane[a] = fmaf(d_lane[a], sc, dsum);
                    s2_lane[a] = fmaf(s2_lane[a], sc, s2sum);
                  }
                  if constexpr (HS > 1 && DUAL) {  // which of the two weights: the sign
#pragma unroll
                    for (int a = 0; a < NE; ++a) pe[a] = raw[a] > 0.f ? pe[a] : -pe[a];
                  }
                  m_run = m_new;
                } else {
#pragma unroll
                  for (int a = 0; a < NE; ++a) {
                    pe[a] = pe2[a] = 0.f;
                    if (e_ok[a]) {
                      if (SRC) {
                        bool pass;  // the score's slope is 1
                        if (alpha_b != nullptr) {  // read back instead of recomputed; D[v] is still gathered
                          pe[a] = fabsf(a_st[a]);
                          pass = a_st[a] > 0.f;
                        } else {
                          const float raw = r_a + vs[a].x;
                          pe[a] = __expf(leaky(raw, dm.slope) - vs[a].y) * vs[a].z;
                          pass = raw > 0.f;
                        }
                        pe2[a] = pass ? pe[a] : dm.slope * pe[a];
                        if (HS > 1) pe[a] = pass ? pe[a] : -pe[a];
                        s_run[a % NA] = fmaf(pe2[a], vs[a].w, s_run[a % NA]);
                      } else {
                        const float raw = e_a[a] + r_a;
                        pe[a] = __expf(leaky(raw, dm.slope) - r_m) * r_invd;
                        pe[a] = raw > 0.f ? pe[a] : dm.slope * pe[a];  // MODE 1
                        s_run[a] += pe[a];
                      }
                    }
                  }
                }
#pragma unroll
                for (int a = 0; a < NE; ++a) {
                  l_p[hd * SL + edge_of(a)] = pe[a];
                  if (HS == 1 && (DUAL || SRC)) l_p2[edge_of(a)] = pe2[a];
                }
                wave_lds_fence();
              }
              float pv[U], pv2[U];
#pragma unroll
              for (int qq = 0; qq < U / 4; ++qq) {
                const float4 p4 = *reinterpret_cast<const float4*>(l_p + hd * SL + t0 + 4 * qq);
                pv[4 * qq] = p4.x; pv[4 * qq + 1] = p4.y; pv[4 * qq + 2] = p4.z; pv[4 * qq + 3] = p4.w;
                if (HS == 1 && (DUAL || SRC)) {
                  const float4 q4 = *reinterpret_cast<const float4*>(l_p2 + t0 + 4 * qq);
                  pv2[4 * qq] = q4.x; pv2[4 * qq + 1] = q4.y; pv2[4 * qq + 2] = q4.z; pv2[4 * qq + 3] = q4.w;
                }
              }
              if constexpr (HS > 1 && (DUAL || SRC)) {
#pragma unroll
                for (int t = 0; t < U; ++t) {
                  const float w = fabsf(pv[t]);
                  pv2[t] = pv[t] > 0.f ? w : dm.slope * w;
                  pv[t] = w;
                }
              }
#pragma unroll
              for (int t4 = 0; t4 < U; t4 += 4) {
                if (!SKIP || t0 + t4 < cnt) {
#pragma unroll
                  for (int t = t4; t < t4 + 4; ++t)
#pragma unroll
                    for (int a = 0; a < NA; ++a) {
                      const float4 rv = widen(rowv[t], a);
                      fma4(part[a], pv[t], rv);
                      if (DUAL) fma4(part2[a], pv2[t], rv);
                      if (SRC) add_dot(t0 + t < cnt, pv2[t], dot4(acc2[a], rv), dpart[a]);
                    }
                }
              }
            }
#pragma unroll
            for (int a = 0; a < NA; ++a) {
              if (ONLINE) {
                fold4(acc[a], sc, part[a]);
                if (DUAL) fold4(acc2[a], sc, part2[a]);
              } else {
                add4(acc[a], part[a]);
              }
              if (SRC) s_dot[a] += dpart[a];
            }
            wave_lds_fence();
          }
          // the sum over the lanes of all their values: that of SL lanes with one each, in the same order
          auto total = [&](const float (&v)[NA]) {
            float t = group_sum_from<L>(v[0], HS);
#pragma unroll
            for (int a = 1; a < NA; ++a) t += group_sum_from<L>(v[a], HS);
            return t;
          };
          // close the item: statistics and sums back to the slot, or (last phase) the finished row to memory
          float4 st_new = stt;
          if (ONLINE) {
            const float d_tot = total(d_lane);
            const float s2_tot = MODE == 3 ? total(s2_lane) : 0.f;
            st_new = make_float4(m_run, d_tot, s2_tot, stt.w);
          } else if (MODE == 1) {
            if (leader) st_new.x = stt.x + total(s_run);
          } else {
            // this slice's share of del[u, h]; the D term is counted by one slice per head
#pragma unroll
            for (int a = 0; a < NA; ++a) s_dot[a] -= leader ? s_run[a] : 0.f;
            st_new.x = stt.x + total(s_dot);
          }
          if (ends) {
            finish(row, acc, acc2, st_new);
          } else {
#pragma unroll
            for (int a = 0; a < NA; ++a) {
              l_acc[q * SL + li + L * a] = acc[a];
              if (DUAL) l_acc2[q * SL + li + L * a] = acc2[a];
            }
            if (li < HS) l_state[q * HS + hd] = st_new;
          }
        }
        q = qn;
        cur = nxt;
      }
      if ((int)threadIdx.x < nslots) l_seg[((p + 1) & 1) * nslot + threadIdx.x] = seg_next;
      __syncthreads();  // the workgroup is done with this block; the next phase's bounds are in LDS
      if constexpr (TAB) store_table();  // read after the second barrier
      if (!last) {      // first slot of the next phase: its loads travel during the wait below
        q = grab(p + 1);
        cur = fetch(p + 1, q);
      }
      phase_step_done(pc, phase++);
      __syncthreads();  // every workgroup of the XCD is done with this block (or the wait ran out)
    }

    if (PARTS && nslots != j1 - j0) {  // rows in parts: their sums, in order, by the group that has the first part
      for (int q0 = grp; q0 < nslots; q0 += GPB) {
        const int tag = l_row[q0];
        if (tag >= -1 || (q0 > 0 && l_row[q0 - 1] == tag)) continue;
        float4 st = make_float4(ONLINE ? -INFINITY : 0.f, 0.f, 0.f, 0.f), acc[NA], acc2[NA];
#pragma unroll
        for (int a = 0; a < NA; ++a) acc[a] = acc2[a] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ONLINE)
          for (int i = q0; i < nslots && l_row[i] == tag; ++i) st.x = fmaxf(st.x, l_state[i * HS + hd].x);
        for (int i = q0; i < nslots && l_row[i] == tag; ++i) {
          const float4 si = l_state[i * HS + hd];
          float sc = 1.f;  // to the maximum of all parts
          if (ONLINE) {
            sc = si.x == -INFINITY ? 0.f : __expf(si.x - st.x);
            st.y = fmaf(sc, si.y, st.y);
            st.z = fmaf(sc, si.z, st.z);
          } else {
            st.x += si.x;
          }
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            fma4(acc[a], sc, l_acc[i * SL + li + L * a]);
            if (DUAL) fma4(acc2[a], sc, l_acc2[i * SL + li + L * a]);
          }
        }
        finish(-2 - tag, acc, acc2, st);
      }
      __syncthreads();  // the next rows take the slots
    }
  }
}

__global__ void k_gat_zero_clock(int32_t* __restrict__ clock) { clock[threadIdx.x] = 0; }

// elT[h][v] = el[v][h]: a column block of gathered vertices then spans 4 B per vertex in
// the head a slice needs instead of 4*H (fewer L2 lines for the per-edge scalar gathers)
__global__ void k_gat_head_major(int64_t n, int H, const float* __restrict__ a, float* __restrict__ aT) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;  // index into aT
  if (i >= n * H) return;
  const int64_t h = i / n, v = i - h * n;
  aT[i] = a[v * H + h];
}

static gnn_status_t head_major(const gnn_graph_t* g, int H, const float* a, float* aT, hipStream_t st) {
  ProfScope p("gat_head_major", st);
  const int64_t cnt = (int64_t)g->n * H;
  k_gat_head_major<<<(unsigned)cdiv(cnt, 256), 256, 0, st>>>(g->n, H, a, aT);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

// ---- host side -------------------------------------------------------------------------
// fp16 copy of the gathered matrix (configuration key "gather_precision" = 1): rows of 2*HF bytes
// are cut into slices of 64 columns (one 128-byte line), each inside one head
bool gat_blocked_half(const gnn_graph_t* g, int heads, int f) {
  if (config_get(kCfgGatherPrecision) != 1 || !gat_blocked_whole(g, heads, f)) return false;
  const int HF = heads * f;
  if (HF % 64 != 0 || HF < 128) return false;
  const int q = HF / 64;
  return (q == 1 || q == 2 || q == 4 || q == 8) && q % heads == 0;
}

__global__ void k_to_half(int64_t quads, const float* __restrict__ src, __half* __restrict__ dst) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= quads) return;
  const float4 v = ld4(src + 4 * i);
  __half2* o = reinterpret_cast<__half2*>(dst + 4 * i);
  o[0] = __floats2half2_rn(v.x, v.y);
  o[1] = __floats2half2_rn(v.z, v.w);
}

static gnn_status_t to_half(const gnn_graph_t* g, int HF, const float* src, void* dst, hipStream_t st) {
  ProfScope p("gat_to_half", st);
  const int64_t quads = (int64_t)g->n * (HF / 4);
  k_to_half<<<(unsigned)cdiv(quads, 256), 256, 0, st>>>(quads, src, static_cast<__half*>(dst));
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

// Rows of 64 columns with several heads: the single-launch kernels up to here, whose gathers stay in the L2s, the persistent ones above.
// Training pass, single launch | persistent, us: 8 x 8 power law 15 523 rows, 8 10^5 edges 98 | 124, 2.1 10^6 151 | 161, 22 308, 3 10^6
// 212 | 193, 47 029, 1.2 10^7 728 | 530, 232 965, 1.14 10^8 8590 | 5190; 4 x 16 22 308, 10^7 409 | 424, 40 000, 4 10^6 233 | 270,
// 47 029, 1.2 10^7 567 | 544, 10^5, 2 10^7 1198 | 1030, 232 965, 1.14 10^8 8280 | 5150; even degrees favour the persistent kernels more.
// Wider rows: every size (15 523, 8 10^5, 16 x 8: 162 | 156; 8 x 16, 2.1 10^6 in slices of one head 1645, so 241).
constexpr int64_t kSharedEdgesOf8 = (int64_t)5 << 19;  // slices of eight heads
constexpr int64_t kSharedEdges = (int64_t)10 << 20;    // of two or four, and more rows than
constexpr int64_t kSharedRows = 32768;
bool gat_blocked_applies(const gnn_graph_t* g, int heads, int f) {
  if (!g->blocked_pays() || config_get(kCfgForceSimple)) return false;
  const int HF = heads * f;
  Slicing sl;
  if (!pick_slicing(heads, HF, sl)) return false;
  if (sl.hs == 1 || sl.ns > 1 || config_get(kCfgResidentSums) == 2) return true;
  return sl.hs == 8 ? g->nnz >= kSharedEdgesOf8 : g->nnz >= kSharedEdges && g->n > kSharedRows;
}

bool gat_blocked_whole(const gnn_graph_t* g, int heads, int f) {
  Slicing sl;
  return gat_blocked_applies(g, heads, f) && pick_whole_slicing(heads, heads * f, sl);
}
bool gat_blocked_shared(const gnn_graph_t* g, int heads, int f) {
  Slicing sl;
  return gat_blocked_applies(g, heads, f) && pick_slicing(heads, heads * f, sl) && sl.hs > 1;
}

__global__ void k_zero_i32(int n, int32_t* __restrict__ p) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// LDS bytes of the staged kernel: per-group scratch plus the block's table
template <int SL>
static size_t staged_lds_bytes(int64_t block_cols) {
  constexpr int GS = kBlkGroupFloats<SL>;
  return sizeof(float) * ((size_t)(kStageThreads / SL) * GS + (size_t)block_cols);
}
constexpr size_t kStageLdsLimit = 152 * 1024;  // of the 160 KB a CU has
constexpr int kStageMinEdgesPerRow = 48;        // mean edges per row of a block worth staging

// Name of a launch's timed bracket: the kernel's name, or "name#i" for the i-th launch of a pass
// when the environment variable GNN_PROF_PER_LAUNCH is set (for tuning the launch groups).
static const char* bracket_name(const char* name, size_t launch) {
  static const bool per_launch = std::getenv("GNN_PROF_PER_LAUNCH") != nullptr;
  if (!per_launch) return name;
  static std::mutex mu;
  static std::map<std::string, std::string> names;  // node addresses are stable
  std::lock_guard<std::mutex> lock(mu);
  std::string key = std::string(name) + "#" + std::to_string(launch);
  return names.emplace(key, key).first->second.c_str();
}

static constexpr bool skips_rows(int SL) { return SL == 4 || SL == 32; }  // see k_gat_blk

// 32-bit byte offsets (and 24-bit multiplies) reach every gathered row
static bool gat_narrow(const gnn_graph_t* g, GatDims dm) { return row_offsets_ok(g->n, 4 * dm.HF) && !config_get(kCfgWideOffsets); }

template <int SL, int MODE, bool HALF, bool SKIP, bool NARROW>
static gnn_status_t launch_blocks_impl(const gnn_graph_t* g, int side, const char* name, GatDims dm,
                                  int el_hm, const float* feat, const float* rowfeat,
                                  const float* el, const float* er, const float* m, const float* d,
                                  const float4* vstate, float* acc, float* acc2, float* scal,
                                  int32_t* queue, float4* state, float* m_out, float* d_out, hipStream_t st,
                                  const float* alpha_b = nullptr) {
  const int ns = dm.HF / ((HALF ? 8 : 4) * SL);
  const int sph = ns / dm.H;
  constexpr int GS = kBlkGroupFloats<SL>;
  const int rows_per_wg = (kBlkThreads / SL) * kRowsPerGroup;
  const unsigned grid = (unsigned)(cdiv(g->n, rows_per_wg) * ns);
  const size_t lds = sizeof(float) * (size_t)(kBlkThreads / SL) * GS;
  bool stage_ok = false;
  if constexpr (MODE != 2) {
    stage_ok = queue != nullptr && el_hm && (int)g->h_block_begin[side].size() == g->nblk + 1;
    if (stage_ok) {
      // more than 64 KB of dynamic LDS needs the attribute; once per instantiation (the call is
      // idempotent, so a race between two first callers is harmless)
      static std::atomic<bool> attr_set{false};
      if (!attr_set.load(std::memory_order_acquire)) {
        GNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gat_blk<SL, MODE, true, HALF, SKIP, NARROW>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStageLdsLimit));
        attr_set.store(true, std::memory_order_release);
      }
      ProfScope p("gat_blk_queue_reset", st);
      k_zero_i32<<<cdiv(g->nblk * kSlices, 64), 64, 0, st>>>(g->nblk * kSlices, queue);
      GNN_LAUNCH_CHECK();
    }
  }
  const std::vector<int32_t>& groups = g->h_group[side][(MODE == 2 || MODE == 3) ? 1 : 0];
  GNN_REQUIRE(groups.size() >= 2 && groups.front() == 0 && groups.back() == g->nblk, GNN_ERR_UNSUPPORTED,
              "gat blocked: the plan has no launch groups");
  for (size_t gi = 0; gi + 1 < groups.size(); ++gi) {
    const int b = groups[gi], b_end = groups[gi + 1], nseg = b_end - b;
    GNN_REQUIRE(nseg >= 1 && nseg <= kMaxMerge, GNN_ERR_UNSUPPORTED, "gat blocked: bad launch group");
    const int2* bseg_b = reinterpret_cast<const int2*>(g->bseg[side]) + (int64_t)b * g->n;
    const int32_t col_begin = b * g->block_cols;
    bool staged = false;
    if constexpr (MODE != 2) {
      // The LDS table pays on blocks whose rows are long (measured with 20480 columns: 2.7 ms
      // instead of 3.5 ms at 220 edges per row, 1.28 instead of 1.43 ms at 67, no difference at
      // 42); the persistent launch has a higher fixed cost, which sparser blocks do not repay.
      const int64_t edges = (int64_t)g->h_block_begin[side][b_end] - g->h_block_begin[side][b];
      const int64_t cols_wide = (int64_t)nseg * g->block_cols;
      const size_t stage_bytes = staged_lds_bytes<SL>(cols_wide);
      staged = stage_ok && stage_bytes <= kStageLdsLimit && edges >= (int64_t)kStageMinEdgesPerRow * g->n;
      if (staged) {
        const int32_t cols_here = (int32_t)(g->n - col_begin < cols_wide ? g->n - col_begin : cols_wide);
        // one persistent workgroup per CU, a multiple of 8 so that every XCD serves one slice
        const unsigned pgrid = (unsigned)(device_cu_count() / kSlices * kSlices);
        ProfScope p(bracket_name(name, gi), st);  // one timed bracket per launch
        k_gat_blk<SL, MODE, true, HALF, SKIP, NARROW><<<pgrid, kStageThreads, stage_bytes, st>>>(
            g->n, g->order[side], bseg_b, g->bcol[side], feat, rowfeat, el, er, m, d, vstate, col_begin, dm, sph,
            b == 0, el_hm, acc, acc2, scal, queue + b * kSlices, cols_here, 1, ns, b_end == g->nblk, state,
            m_out, d_out, nseg, alpha_b, g->nnz);
        GNN_LAUNCH_CHECK();
      }
    }
    if (!staged) {
      ProfScope p(bracket_name(name, gi), st);  // one timed bracket per launch
      k_gat_blk<SL, MODE, false, HALF, SKIP, NARROW><<<grid, kBlkThreads, lds, st>>>(
          g->n, g->order[side], bseg_b, g->bcol[side], feat, rowfeat, el, er, m, d, vstate, col_begin, dm, sph,
          b == 0, el_hm, acc, acc2, scal, nullptr, 0, 1, ns, b_end == g->nblk, state, m_out, d_out, nseg,
          alpha_b, g->nnz);
      GNN_LAUNCH_CHECK();
    }
  }
  return GNN_OK;
}

template <int SL, int MODE, bool HALF = false>
static gnn_status_t launch_blocks(const gnn_graph_t* g, int side, const char* name, GatDims dm,
                                  int el_hm, const float* feat, const float* rowfeat,
                                  const float* el, const float* er, const float* m, const float* d,
                                  const float4* vstate, float* acc, float* acc2, float* scal,
                                  int32_t* queue, float4* state, float* m_out, float* d_out, hipStream_t st,
                                  const float* alpha_b = nullptr) {
#define GNN_GAT_BLOCKS(NARROW_)                                                                                                \
  return launch_blocks_impl<SL, MODE, HALF, skips_rows(SL), NARROW_>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, \
                                                               acc2, scal, queue, state, m_out, d_out, st, alpha_b)
  if (gat_narrow(g, dm)) GNN_GAT_BLOCKS(true);
  GNN_GAT_BLOCKS(false);
#undef GNN_GAT_BLOCKS
}

// The persistent kernel applies to rows cut into slices of 64 columns (256 bytes of fp32, or one
// 128-byte line of an fp16 copy)
static bool gat_resident_applies(const gnn_graph_t* g, GatDims dm, bool whole = false /* slices inside one head */) {
  if (!config_get(kCfgResidentSums) || g->phase_clock == nullptr) return false;
  Slicing sl;
  return (whole ? pick_whole_slicing(dm.H, dm.HF, sl) : pick_slicing(dm.H, dm.HF, sl)) && sl.SL == 16;
}

// one workgroup per CU, a multiple of 8 so that every XCD serves one slice
static unsigned gat_resident_grid() { return (unsigned)(device_cu_count() / kXcds * kXcds); }

// fp16 rows, forward without a stash: the block's part of el in LDS as well; see kGatTabPerThread
static bool gat_resident_table(const gnn_graph_t* g) {
  return g->block_cols <= kGatTabPerThread * kGatResThreads;
}

static int64_t gat_resident_groups(int ns, int na) { return (int64_t)gat_resident_grid() / ns * (kGatResThreads * na / 16); }

template <int MODE, int NA, int HS, bool TAB, bool SKIP, bool HALF, bool NARROW, bool PARTS>
static gnn_status_t launch_resident_addr(const gnn_graph_t* g, int side, const char* name, GatDims dm, int el_hm,
                                         const float* feat, const float* rowfeat, const float* el, const float* er,
                                         const float* m, const float* d, const float4* vstate, float* acc,
                                         float* acc2, float* scal, float* m_out, float* d_out, hipStream_t st,
                                         const float* alpha_b) {
  constexpr int SL = 16;
  const int ns = dm.HF <= 4 * SL ? 1 : dm.HF / (4 * SL);
  const int sph = HS > 1 ? 1 : ns / dm.H;
  const int nslot = gat_res_slots<SL, MODE, NA, HS>(TAB ? g->block_cols : 0);
  static std::atomic<bool> attr_set{false};
  if (!attr_set.load(std::memory_order_acquire)) {
    GNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gat_res<SL, MODE, NA, TAB, SKIP, HALF, NARROW, HS, PARTS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kGatResLdsBytes));
    attr_set.store(true, std::memory_order_release);
  }
  const unsigned grid = gat_resident_grid();
  ProfScope p(name, st);
  k_gat_zero_clock<<<1, kXcds * kClockStride, 0, st>>>(g->phase_clock);
  GNN_LAUNCH_CHECK();
  k_gat_res<SL, MODE, NA, TAB, SKIP, HALF, NARROW, HS, PARTS><<<grid, kGatResThreads, kGatResLdsBytes, st>>>(
      g->n, g->order[side], reinterpret_cast<const int2*>(g->bseg[side]), g->bcol[side], feat, rowfeat, el, er, m, d,
      vstate, dm, sph, el_hm, g->block_cols, g->nblk, ns, acc, acc2, scal, m_out, d_out, g->phase_clock,
      (int)config_get(kCfgResidentSpin), (int)config_get(kCfgResidentSyncEvery), alpha_b, g->nnz, nslot,
      PARTS ? cut_long_rows(g, side, gat_resident_groups(ns, NA), grid / ns, nslot) : RowParts{});
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

template <int MODE, int NA, int HS, bool TAB, bool SKIP, bool HALF, bool NARROW>
static gnn_status_t launch_resident_parts(const gnn_graph_t* g, int side, const char* name, GatDims dm, int el_hm,
                                          const float* feat, const float* rowfeat, const float* el, const float* er,
                                          const float* m, const float* d, const float4* vstate, float* acc,
                                          float* acc2, float* scal, float* m_out, float* d_out, hipStream_t st,
                                          const float* alpha_b) {
  const int ns = dm.HF <= 64 ? 1 : dm.HF / 64;
  if (has_long_rows(g, side, gat_resident_groups(ns, NA)))
    return launch_resident_addr<MODE, NA, HS, TAB, SKIP, HALF, NARROW, true>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d,
                                                                           vstate, acc, acc2, scal, m_out, d_out, st, alpha_b);
  return launch_resident_addr<MODE, NA, HS, TAB, SKIP, HALF, NARROW, false>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d,
                                                                          vstate, acc, acc2, scal, m_out, d_out, st, alpha_b);
}

template <int MODE, int NA, int HS, bool TAB, bool SKIP, bool HALF>
static gnn_status_t launch_resident_impl(const gnn_graph_t* g, int side, const char* name, GatDims dm, int el_hm,
                                         const float* feat, const float* rowfeat, const float* el, const float* er,
                                         const float* m, const float* d, const float4* vstate, float* acc,
                                         float* acc2, float* scal, float* m_out, float* d_out, hipStream_t st,
                                         const float* alpha_b) {
  if (gat_narrow(g, dm))
    return launch_resident_parts<MODE, NA, HS, TAB, SKIP, HALF, true>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate,
                                                        acc, acc2, scal, m_out, d_out, st, alpha_b);
  return launch_resident_parts<MODE, NA, HS, TAB, SKIP, HALF, false>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate,
                                                       acc, acc2, scal, m_out, d_out, st, alpha_b);
}

template <int MODE>
static gnn_status_t launch_resident(const gnn_graph_t* g, int side, const char* name, GatDims dm, int el_hm,
                                    const float* feat, const float* rowfeat, const float* el, const float* er,
                                    const float* m, const float* d, const float4* vstate, float* acc, float* acc2,
                                    float* scal, float* m_out, float* d_out, hipStream_t st, const float* alpha_b,
                                    bool half_feat) {
  if (half_feat) {
    if constexpr (MODE != 1) {
#define GNN_GAT_HALF(NA_, TAB_)                                                                                             \
  return launch_resident_impl<MODE, NA_, 1, TAB_, true, true>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, \
                                                           acc2, scal, m_out, d_out, st, alpha_b)
      if constexpr (MODE == 0) {
        if (gat_resident_table(g)) GNN_GAT_HALF(2, true);
      }
      GNN_GAT_HALF(2, false);
#undef GNN_GAT_HALF
    }
  }
  Slicing sl;
  if constexpr (MODE != 1) {
    if (pick_slicing(dm.H, dm.HF, sl) && sl.hs > 1) {
#define GNN_GAT_SHARED(HS_)                                                                                              \
  case HS_:                                                                                                              \
    return launch_resident_impl<MODE, 1, HS_, false, true, false>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, \
                                                                  vstate, acc, acc2, scal, m_out, d_out, st, alpha_b)
      switch (sl.hs) {
        GNN_GAT_SHARED(2);
        GNN_GAT_SHARED(4);
        GNN_GAT_SHARED(8);
      }
#undef GNN_GAT_SHARED
    }
  }
  // gathers past a segment's end are skipped on rows of four and more slices; on narrower rows the
  // source side gains from it as well (6.48 -> 6.14 ms for the two layers of a 128 / 44-wide model at
  // Reddit scale), the forward modes lose a little (5.87 -> 5.96 ms)
  if (MODE == 2 || dm.HF / 64 >= 4)
    return launch_resident_impl<MODE, 1, 1, false, true, false>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc,
                                                                acc2, scal, m_out, d_out, st, alpha_b);
  if constexpr (MODE != 2)
    return launch_resident_impl<MODE, 1, 1, false, false, false>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc,
                                                                 acc2, scal, m_out, d_out, st, alpha_b);
  return GNN_ERR_UNSUPPORTED;  // not reached
}

template <int MODE>
static gnn_status_t run_blocks(const gnn_graph_t* g, int side, const char* name, GatDims dm,
                               int el_hm, const float* feat, const float* rowfeat, const float* el, const float* er, const float* m,
                               const float* d, const float4* vstate, float* acc, float* acc2,
                               float* scal, int32_t* queue, float4* state, float* m_out, float* d_out,
                               hipStream_t st, bool half_feat = false, const float* alpha_b = nullptr) {
  if (gat_resident_applies(g, dm, MODE == 1))
    return launch_resident<MODE>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, acc2, scal,
                                 m_out, d_out, st, alpha_b, half_feat);
  if (half_feat) {
    if constexpr (MODE != 1)
      return launch_blocks<8, MODE, true>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, acc2, scal,
                                          queue, state, m_out, d_out, st, alpha_b);
  }
  Slicing sl;
  if (!pick_whole_slicing(dm.H, dm.HF, sl)) sl.SL = 0;
  GNN_REQUIRE(sl.SL == 0 || dm.HF >= 128, GNN_ERR_UNSUPPORTED,
              "gat blocked: rows of one slice are served by the persistent kernels only");
  switch (sl.SL) {
    case 4: return launch_blocks<4, MODE>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, acc2, scal, queue, state, m_out, d_out, st, alpha_b);
    case 8: return launch_blocks<8, MODE>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, acc2, scal, queue, state, m_out, d_out, st, alpha_b);
    case 16: return launch_blocks<16, MODE>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, acc2, scal, queue, state, m_out, d_out, st, alpha_b);
    case 32: return launch_blocks<32, MODE>(g, side, name, dm, el_hm, feat, rowfeat, el, er, m, d, vstate, acc, acc2, scal, queue, state, m_out, d_out, st, alpha_b);
  }
  set_error("gat blocked: unsupported slice width");
  return GNN_ERR_UNSUPPORTED;
}

gnn_status_t gat_blocked_fwd(const gnn_graph_t* g, GatDims dm, const float* z, const float* el,
                             const float* er, float* m, float* d, float* out, float* t, float* sg,
                             float* el_t, int32_t* queue, float4* state, void* half_buf, hipStream_t st) {
  if (gat_blocked_shared(g, dm.H, dm.F)) el_t = nullptr;  // the heads of a slice stand side by side
  if (el_t) GNN_TRY(head_major(g, dm.H, el, el_t, st));
  if (!config_get(kCfgLdsScalarTable)) queue = nullptr;
  const float* el_use = el_t ? el_t : el;
  const int hm = el_t != nullptr;
  const bool half = half_buf != nullptr && gat_blocked_half(g, dm.H, dm.F);
  const float* feat = z;
  if (half) {  // the rows the edges gather come from an fp16 copy; el, er were made from the fp32 rows
    GNN_TRY(to_half(g, dm.HF, z, half_buf, st));
    feat = static_cast<const float*>(half_buf);
  }
  if (t)
    return run_blocks<3>(g, 0, "gat_fwd_fused", dm, hm, feat, nullptr, el_use, er, nullptr, nullptr, nullptr, out, t, sg,
                         queue, state, m, d, st, half);
  return run_blocks<0>(g, 0, "gat_fwd_fused", dm, hm, feat, nullptr, el_use, er, nullptr, nullptr, nullptr, out, nullptr,
                       nullptr, queue, state, m, d, st, half);
}

gnn_status_t gat_blocked_bwd_dst(const gnn_graph_t* g, GatDims dm, const float* z, const float* el,
                                 const float* er, const float* m, const float* d, const float* out,
                                 const float* gout, float* der, float4* vstate, float* t_buf,
                                 float* sg_buf, float* el_t, int32_t* queue, hipStream_t st) {
  if (el_t) GNN_TRY(head_major(g, dm.H, el, el_t, st));
  if (!config_get(kCfgLdsScalarTable)) queue = nullptr;
  GNN_TRY(run_blocks<1>(g, 0, "gat_bwd_dst", dm, el_t != nullptr, z, nullptr, el_t ? el_t : el, er, m, d, nullptr,
                        t_buf, nullptr, sg_buf, queue, nullptr, nullptr, nullptr, st));
  return gat_dst_finish(g, dm, gout, t_buf, out, sg_buf, er, m, d,
                        (gat_blocked_shared(g, dm.H, dm.F) ? 0 : kDstHeadMajor) |
                            (gat_blocked_half(g, dm.H, dm.F) ? kDstHalfGout : 0), der, vstate, st);
}

// dz[u,h,:] += a_l[h,:] del[u,h] + a_r[h,:] der[u,h], with del[u,h] = the sum of the shares its
// slices left in sd ([n][8], slice-major inside a vertex); one thread per float4 of dz
__global__ void k_gat_src_finish_blk(int64_t n, GatDims dm, int ns, const float* sd,
                                     const float* __restrict__ der, const float* __restrict__ a_l,
                                     const float* __restrict__ a_r, float* __restrict__ dz,
                                     float* del /* sd itself where ns is 0 */) {
  const int qpr = dm.HF / 4;  // float4 per row
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n * qpr) return;
  const int64_t u = i / qpr;
  const int col = 4 * (int)(i - u * qpr);
  const int h = col / dm.F, sph = ns / dm.H;
  float dl = 0.f;
  if (ns == 0) {  // del is there
    dl = sd[u * dm.H + h];
  } else {
    for (int s = 0; s < sph; ++s) dl += sd[u * kSlices + h * sph + s];  // fixed order
    if (col == h * dm.F) del[u * dm.H + h] = dl;
  }
  float4 o = ld4(dz + u * dm.HF + col);
  fma4(o, dl, ld4(a_l + col));
  fma4(o, der[u * dm.H + h], ld4(a_r + col));
  st4(dz + u * dm.HF + col, o);
}

// The per-edge stash of the "fusion with stashing" arm in the order the source-side kernel walks:
// alpha_b[h][q] for position q of the source side's blocked edge list = softmax value of that edge
// with the sign of its raw score.  One 16-lane group per source row, its segments block by block.
__global__ __launch_bounds__(256) void k_gat_stash_alpha_blk(
    int32_t n, int32_t nblk, int64_t nnz, int H, float slope, const int32_t* __restrict__ bptr,
    const int32_t* __restrict__ bcol, const float* __restrict__ el, const float* __restrict__ er,
    const float* __restrict__ m, const float* __restrict__ d, float* __restrict__ alpha_b) {
  const int li = threadIdx.x & 15;
  const int64_t u = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 4;
  if (u >= n) return;
  for (int b = 0; b < nblk; ++b) {
    const int32_t beg = bptr[(int64_t)b * n + u], end = bptr[(int64_t)b * n + u + 1];
    for (int32_t q = beg + li; q < end; q += 16) {
      const int64_t v = bcol[q];
      for (int h = 0; h < H; ++h) {
        const float raw = el[u * H + h] + er[v * H + h];
        const float a = __expf(leaky(raw, slope) - m[v * H + h]) / d[v * H + h];
        alpha_b[(int64_t)h * nnz + q] = raw > 0.f ? a : -a;
      }
    }
  }
}

gnn_status_t gat_blocked_stash_alpha(const gnn_graph_t* g, int H, float slope, const float* el, const float* er,
                                     const float* m, const float* d, float* alpha_b, hipStream_t st) {
  ProfScope p("gat_stash_alpha", st);
  k_gat_stash_alpha_blk<<<(unsigned)cdiv((int64_t)g->n * 16, 256), 256, 0, st>>>(
      g->n, g->nblk, g->nnz, H, slope, g->bptr[1], g->bcol[1], el, er, m, d, alpha_b);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

gnn_status_t gat_blocked_bwd_src(const gnn_graph_t* g, GatDims dm, const float* z, const float* el,
                                 const float4* vstate, const float* der, const float* gout,
                                 const float* a_l, const float* a_r, float* dz, float* del,
                                 float* sd_buf /* [n][8] scratch */, void* half_buf, hipStream_t st,
                                 const float* alpha_b) {
  const bool half = half_buf != nullptr && gat_blocked_half(g, dm.H, dm.F);
  const float* feat = gout;
  if (half) {
    GNN_TRY(to_half(g, dm.HF, gout, half_buf, st));
    feat = static_cast<const float*>(half_buf);
  }
  const bool shared = gat_blocked_shared(g, dm.H, dm.F);
  if (shared) sd_buf = del;  // a slice has all of its heads: no shares
  GNN_TRY(run_blocks<2>(g, 1, "gat_bwd_src", dm, 0, feat, z, el, nullptr, nullptr, nullptr, vstate, dz,
                        nullptr, sd_buf, nullptr, nullptr, nullptr, nullptr, st, half, alpha_b));
  Slicing sl;
  int ns = 0;
  if (half) ns = dm.HF / 64;
  else if (pick_slicing(dm.H, dm.HF, sl)) ns = sl.ns;
  GNN_REQUIRE(shared || (ns >= dm.H && ns % dm.H == 0 && ns <= kSlices), GNN_ERR_UNSUPPORTED, "gat blocked: bad slicing");
  ProfScope p("gat_bwd_src_finish", st);
  const int64_t quads = (int64_t)g->n * (dm.HF / 4);
  k_gat_src_finish_blk<<<(unsigned)cdiv(quads, 256), 256, 0, st>>>(g->n, dm, shared ? 0 : ns, sd_buf, der, a_l, a_r, dz, del);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

}  // namespace gnn

// Which instantiation of the column-blocked kernel a pass launches for this graph and shape
// (the persistent kernel, or the plain, not LDS-staged variant of the launch-per-block kernel),
// spelled as a profiler prints it; "" when the single-launch kernels run instead.  Lets a measurement script check that stored counter readings belong to
// the kernel it times.
extern "C" gnn_status_t gnn_gat_blocked_kernel_name(const gnn_graph_t* g, int heads, int f, int mode,
                                                    char* buf, size_t len) {
  using namespace gnn;
  clear_error();
  GNN_REQUIRE(g != nullptr && buf != nullptr && len > 0, GNN_ERR_INVALID_ARG,
              "gnn_gat_blocked_kernel_name: null argument");
  GNN_REQUIRE(mode >= 0 && mode <= 3, GNN_ERR_INVALID_ARG, "gnn_gat_blocked_kernel_name: mode must be 0..3");
  buf[0] = 0;
  if (heads <= 0 || f <= 0 || !gat_blocked_applies(g, heads, f)) return GNN_OK;
  const bool half = mode != 1 && gat_blocked_half(g, heads, f);
  Slicing sl;
  if (!pick_slicing(heads, heads * f, sl)) return GNN_OK;
  if (mode == 1 && !pick_whole_slicing(heads, heads * f, sl)) return GNN_OK;
  const GatDims dm = make_dims(heads, f, 0.2f);
  if (gat_resident_applies(g, dm, mode == 1)) {
    std::snprintf(buf, len, "k_gat_res<16, %d, %d, %s, %s, %s, %s, %d, %s>", mode,
                  half ? 2 : 1,
                  half && mode == 0 && gat_resident_table(g) ? "true" : "false",
                  (half || sl.hs > 1 || heads * f / 64 >= 4 || mode == 2) ? "true" : "false", half ? "true" : "false",
                  gat_narrow(g, dm) ? "true" : "false", sl.hs,
                  has_long_rows(g, mode == 2, gat_resident_groups(dm.HF <= 64 ? 1 : dm.HF / 64, half ? 2 : 1)) ? "true" : "false");
    return GNN_OK;
  }
  const int SL = half ? 8 : sl.SL;
  std::snprintf(buf, len, "k_gat_blk<%d, %d, false, %s, %s, %s>", SL, mode, half ? "true" : "false", skips_rows(SL) ? "true" : "false",
                gat_narrow(g, dm) ? "true" : "false");
  return GNN_OK;
}
