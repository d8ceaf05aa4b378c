// GCN layer with separable static edge weights e_uv = c_src[u] c_dst[v] (App. A.2 "GCN";
// the symmetric normalisation, mean and plain-sum aggregation are of this form).
//
// Reorganization (Sec. 4): multiplying by the edge weight is linear, so both factors move
// from the edges onto the vertices,
//     out[v] = c_dst[v] * sum over in-edges of  (c_src ⊙ (x w))[u],
// and the fused Scatter-ApplyEdge-Gather is an unweighted gather-sum of rows: no per-edge
// scalar is read at all.  Backward is the same sum over the CSC transpose (no atomics):
//     dz[u] = c_src[u] * sum over out-edges of (c_dst ⊙ gout)[v],  gw = x^T dz,  gx = dz w^T.
// Nothing per-edge is stored; the saved state is zs = c_src ⊙ (x w).
//
// Large graphs use the same column-blocked, XCD-sliced traversal as the GAT kernels: 8
// column slices (workgroup id mod 8, one per XCD), blocks of `block_cols` gathered vertices,
// one launch per block, running sums read-add-written between launches.
//
// Two thread mappings of the single-launch sum (Sec. 5, the vertex-balanced and the
// edge-balanced mapping of a fused Gather): k_rowsum gives a group one row, k_rowsum_eb gives
// a group a fixed run of consecutive edges and joins the pieces of a row that spans several
// runs with atomic adds.  gnn_gcn_tune times both on a graph and the layer calls then use the
// faster one per side (the profile-driven choice of the mapping).
#include <atomic>
#include <cstdio>
#include <type_traits>

#include "common.h"
#include "row_parts.h"
#include "rowgroup.h"

namespace gnn {

constexpr int kGcnBlock = 256;
constexpr int kGcnSlices = 8;
constexpr int kGcnRows = 4;  // consecutive rows of the degree order per group (software-pipelined)

// out[v,:] = c[v] * in[v,:]   (in == out allowed)
__global__ void k_scale_rows(int64_t quads, int q_per_row, const float* __restrict__ c,
                             const float* in, float* out) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= quads) return;
  const float s = c[i / q_per_row];
  const float4 v = ld4(in + 4 * i);
  st4(out + 4 * i, make_float4(s * v.x, s * v.y, s * v.z, s * v.w));
}

static bool gcn_narrow(const gnn_graph_t* g, int F) { return row_offsets_ok(g->n, 4 * F) && !config_get(kCfgWideOffsets); }

// ---- single launch: out[row,:] = scale[row] * sum over the row's gathered vertices of feat ----
// W: every edge carries a static weight (wgt, in the order of cols); scale may then be null
// Rows come with their bounds, and the next chunk's sources travel while a chunk is gathered: us, 30 000 vertices, 10^6 edges,
// 64 columns, layer 111 -> 99 unsliced.  NS slices of 4 L columns, see xcd_slice and gather_slices.
// U gathered rows in flight per lane, see launch_rowsum.
// NARROW: 32-bit byte offsets reach every gathered row (told at run time, the loads of one kind wait for those of the other: 64 columns
// with a weight per edge, 10^5 vertices, 2 10^6 edges, layer 145.9 -> 147.4 us).
template <int L, int NV, bool W, int NS, int U, bool NARROW>
__global__ __launch_bounds__(kGcnBlock) void k_rowsum(
    RowLaunch rl, const int4* __restrict__ rows, const int32_t* __restrict__ cols, const float* __restrict__ feat, int F,
    const float* __restrict__ scale, float* __restrict__ out, const float* __restrict__ wgt = nullptr) {
  constexpr int G = kWave / L;
  constexpr int GPB = G * (kGcnBlock / kWave);
  constexpr int NC = 4 * NV;
  constexpr int B = U < 4 ? U : 4;  // of which a chunk's end asks for this many at a time
  __shared__ int lds[GPB * L];
  __shared__ float lds_w[W ? GPB * L : 1];
  __shared__ float coop_buf[GPB * L * NC];
  const int lane = threadIdx.x & 63;
  const int li = lane & (L - 1);
  const int grp = threadIdx.x / L;
  int64_t r;
  int gi, ngrp;
  RowRange rr;
  unsigned block;
  const int col0 = xcd_slice<NS>(block) * 4 * L;
  if (!pick_row<GPB>(rl, grp, rr, r, gi, ngrp, block)) return;
  out += col0;
  const uint32_t row_bytes = 4u * F, lane_bytes = 4u * (col0 + 4 * li);
  const auto table = row_table(feat, NARROW ? (int64_t)rl.n_rows * row_bytes : 0);
  int* l_idx = lds + grp * L;
  float* l_w = lds_w + (W ? grp * L : 0);
  const int4 row = rows[r];
  const int32_t v = row.x;
  const uint32_t end = row.z;  // unsigned: positions past 2^31 - 1 are past every row's end

  bool slot_ok[NV];
  float4 acc[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    slot_ok[j] = NS > 1 || 4 * (li + j * L) < F;
    acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  uint32_t c0 = row.y + gi * L;
  // the next chunk's sources travel while this one is gathered; no edge: row n_rows, zeros
  int32_t c_next = c0 + li < end ? cols[c0 + li] : rl.n_rows;
  float w_next = W && c0 + li < end ? wgt[c0 + li] : 0.f;
  for (; c0 < end; c0 += ngrp * L) {
    l_idx[li] = c_next;
    if (W) l_w[li] = w_next;
    wave_lds_fence();
    const uint32_t e = c0 + ngrp * L + li;
    c_next = e < end ? cols[e] : rl.n_rows;
    if (W) w_next = e < end ? wgt[e] : 0.f;
    float4 part[NV];  // this chunk's share (two-level summation)
#pragma unroll
    for (int j = 0; j < NV; ++j) part[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    const int cnt = min((uint32_t)L, end - c0);
    for (int t0 = 0; t0 < cnt; t0 += U) {
      int uu[U];
      float ww[U];
#pragma unroll
      for (int t = 0; t < U; ++t) {
        uu[t] = l_idx[t0 + t];
        if (L == 64) uu[t] = __builtin_amdgcn_readfirstlane(uu[t]);
        if (W) ww[t] = l_w[t0 + t];
      }
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        if (!slot_ok[j]) continue;
        float4 rowv[U];
#pragma unroll
        for (int q = 0; q < U; q += B)
          if (t0 + q < cnt) {
            const uint32_t at = lane_bytes + 16u * (j * L);
#pragma unroll
            for (int t = q; t < q + B; ++t) {
              if constexpr (NARROW) rowv[t] = table_load<float4>(table, uu[t], row_bytes, at);
              else rowv[t] = table_load_wide<float4>(feat, rl.n_rows, uu[t], row_bytes, at);
            }
          }
#pragma unroll
        for (int q = 0; q < U; q += B)
          if (t0 + q < cnt) {
#pragma unroll
            for (int t = q; t < q + B; ++t) {
              if (W) fma4(part[j], ww[t], rowv[t]);
              else add4(part[j], rowv[t]);
            }
          }
      }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) add4(acc[j], part[j]);
    wave_lds_fence();
  }
  if (rr.coop) {
    float vv[NC];
#pragma unroll
    for (int j = 0; j < NV; ++j) pack4(vv + 4 * j, acc[j]);
    coop_sum<L, NC, GPB>(coop_buf, vv, grp, li);
    if (grp != 0) return;
#pragma unroll
    for (int j = 0; j < NV; ++j) acc[j] = unpack4(vv + 4 * j);
  }
  const float s = scale ? scale[v] : 1.f;
#pragma unroll
  for (int j = 0; j < NV; ++j)
    if (slot_ok[j])
      st4(out + (int64_t)v * F + 4 * (li + j * L), make_float4(s * acc[j].x, s * acc[j].y, s * acc[j].z, s * acc[j].w));
}

// ---- edge-balanced mapping of the same sum ------------------------------------------------
// A group owns kEbEdges consecutive positions of the edge array, whatever rows they belong to
// (every group does the same amount of gathering, however skewed the degrees are).  It finds
// the row of its first edge by bisection of ptr, then walks row by row.  A row that lies
// entirely inside the run is stored; a row that continues into other runs is added atomically
// onto an output that a fill kernel zeroed before (rows without edges stay zero).  Two pieces
// add up the same in either order; rows of more than two pieces (degree > kEbEdges) depend on
// the arrival order in the last bits.
constexpr int kEbEdges = 64;

__global__ void k_zero_f4(int64_t quads, float* __restrict__ p) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < quads) st4(p + 4 * i, make_float4(0.f, 0.f, 0.f, 0.f));
}

// W: every edge carries a static weight (wgt, in the order of cols); scale may then be null
template <int L, int NV, bool W = false>
__global__ __launch_bounds__(kGcnBlock) void k_rowsum_eb(
    int32_t n, int32_t nnz, const int32_t* __restrict__ ptr, const int32_t* __restrict__ cols,
    const float* __restrict__ feat, int F, const float* __restrict__ scale, float* __restrict__ out,
    const float* __restrict__ wgt = nullptr) {
  constexpr int GPB = kGcnBlock / L;
  constexpr int U = 4;
  constexpr int GS = (W ? 2 : 1) * (kEbEdges + U);  // the run's gathered vertices (and weights), each with U entries of padding
  __shared__ int lds[GPB * GS];
  const int lane = threadIdx.x & 63;
  const int li = lane & (L - 1);
  const int grp = threadIdx.x / L;
  const int64_t run = (int64_t)blockIdx.x * GPB + grp;
  if (run * kEbEdges >= nnz) return;
  const int32_t e0 = (int32_t)(run * kEbEdges);
  const int32_t e1 = min(e0 + kEbEdges, nnz);
  int* l_idx = lds + grp * GS;
  float* l_wt = reinterpret_cast<float*>(l_idx + kEbEdges + U);
  for (int i = li; i < kEbEdges + U; i += L) {
    l_idx[i] = e0 + i < e1 ? cols[e0 + i] : 0;  // padding gathers row 0, for nothing
    if (W) l_wt[i] = e0 + i < e1 ? wgt[e0 + i] : 0.f;
  }

  // row of the first edge: ptr[lo] <= e0 < ptr[hi] throughout (ptr[0] = 0, ptr[n] = nnz)
  int32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (ptr[mid] <= e0) lo = mid; else hi = mid;
  }
  int32_t v = lo, row_beg = ptr[v], row_end = ptr[v + 1];
  wave_lds_fence();

  bool slot_ok[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) slot_ok[j] = 4 * (li + j * L) < F;

  int32_t e = e0;
  while (e < e1) {
    const int32_t seg_end = min(row_end, e1);
    float4 acc[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int32_t t0 = e; t0 < seg_end; t0 += U) {
      int uu[U];
#pragma unroll
      for (int t = 0; t < U; ++t) {
        uu[t] = l_idx[t0 - e0 + t];
        if (L == 64) uu[t] = __builtin_amdgcn_readfirstlane(uu[t]);
      }
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        if (!slot_ok[j]) continue;
        float4 rowv[U];
#pragma unroll
        for (int t = 0; t < U; ++t) rowv[t] = ld4(feat + (int64_t)uu[t] * F + 4 * (li + j * L));
#pragma unroll
        for (int t = 0; t < U; ++t)
          if (t0 + t < seg_end) fma4(acc[j], W ? l_wt[t0 - e0 + t] : 1.f, rowv[t]);
      }
    }
    const float s = scale != nullptr ? scale[v] : 1.f;
    const bool whole = row_beg >= e0 && row_end <= e1;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      if (!slot_ok[j]) continue;
      float* o = out + (int64_t)v * F + 4 * (li + j * L);
      const float4 r = make_float4(s * acc[j].x, s * acc[j].y, s * acc[j].z, s * acc[j].w);
      if (whole) {
        st4(o, r);
      } else {
        unsafeAtomicAdd(o, r.x);
        unsafeAtomicAdd(o + 1, r.y);
        unsafeAtomicAdd(o + 2, r.z);
        unsafeAtomicAdd(o + 3, r.w);
      }
    }
    e = seg_end;
    if (e < e1) {  // the next row that has edges (it starts at e)
      do {
        ++v;
        row_beg = row_end;
        row_end = ptr[v + 1];
      } while (row_end == row_beg);
    }
  }
}

// ---- one column block of the same sum (running sums in acc_buf) -----------------------
// W: every edge carries a static weight, bw in the order of bcol (a second coalesced stream)
template <int SL, bool SKIP, bool W = false>
__global__ __launch_bounds__(kGcnBlock) void k_rowsum_blk(
    int32_t n_rows, const int32_t* __restrict__ order, const int2* __restrict__ bseg_b,
    const int32_t* __restrict__ bcol, const float* __restrict__ feat, int F,
    int first, int ns /* column slices: 8, 4, 2 or 1 */, float* __restrict__ acc_buf,
    int nseg /* adjacent column blocks of this launch (1 .. kMaxMerge): segment j of the row at
                position r of the degree order is bseg_b[j * n_rows + r] */,
    int narrow /* 32-bit byte offsets reach every gathered row */, const float* __restrict__ bw = nullptr) {
  constexpr int GPB = kGcnBlock / SL;
  constexpr int R = kGcnRows;
  constexpr int U = SL < 8 ? 4 : 8;
  constexpr int GS = SL + R + 2 * R * kMaxMerge + (W ? SL : 0);  // LDS ints per group: idx | rows | (beg, end) per row and block | weights
  static_assert(GS % 4 == 0, "group scratch must stay 16-byte aligned");
  static_assert(SL >= R, "one lane per pipelined row loads its metadata");
  __shared__ __align__(16) int lds[GPB * GS];
  const int lane = threadIdx.x & 63;
  const int li = lane & (SL - 1);
  const int grp = threadIdx.x / SL;
  const int slice = blockIdx.x % ns;
  const int64_t r0 = ((int64_t)(blockIdx.x / ns) * GPB + grp) * R;
  if (r0 >= n_rows) return;
  int* l_idx = lds + grp * GS;
  int* l_row = l_idx + SL;
  int2* l_seg = reinterpret_cast<int2*>(l_row + R);  // [R][kMaxMerge]
  float* l_w = reinterpret_cast<float*>(l_idx + SL + R + 2 * R * kMaxMerge);
  const int col = slice * 4 * SL + 4 * li;
  const uint32_t row_bytes = 4u * F, col_bytes = 4u * col;
  const auto table = row_table(feat, (int64_t)n_rows * row_bytes);  // used where `narrow`

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
    if (!first && !any) row = -1;  // nothing to add to this row in these blocks
    l_row[li] = row;
  }
  wave_lds_fence();

  struct Row {
    int32_t row, beg, end, c_first;
    float w_first;
    float4 acc;
  };
  auto fetch = [&](int k, Row& s) {
    s.row = l_row[k];
    const int2 seg0 = l_seg[k * kMaxMerge];
    s.beg = seg0.x;
    s.end = seg0.y;
    s.c_first = 0;
    s.w_first = 0.f;
    s.acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (s.row < 0) return;
    if (s.beg + li < s.end) {
      s.c_first = bcol[s.beg + li];
      if (W) s.w_first = bw[s.beg + li];
    }
    if (!first) s.acc = ld4_stream(acc_buf + (int64_t)s.row * F + col);
  };

  Row cur, nxt;
  fetch(0, cur);
  for (int k = 0; k < R; ++k) {
    if (k + 1 < R) fetch(k + 1, nxt);
    if (cur.row >= 0) {
      float4 acc = cur.acc;
      int32_t beg = cur.beg, end = cur.end, c_next = cur.c_first;
      float w_next = cur.w_first;
      for (int sgi = 0; sgi < nseg; ++sgi) {
      // the bounds and the first indices of the row's segment in the next block are in flight
      // while this one is processed
      int32_t beg_n = 0, end_n = 0, c_first_n = 0;
      float w_first_n = 0.f;
      if (sgi + 1 < nseg) {
        const int2 sn = l_seg[k * kMaxMerge + sgi + 1];
        beg_n = sn.x;
        end_n = sn.y;
        if (beg_n + li < end_n) {
          c_first_n = bcol[beg_n + li];
          if (W) w_first_n = bw[beg_n + li];
        }
      }
      for (int32_t c0 = beg; c0 < end; c0 += SL) {
        // lanes past the end gather zeros; with SKIP, quadruples of gathered rows that lie
        // entirely past the end are skipped.  The branches cost the overlap of the second half's loads with the first
        // half's sums: rows cut into four or more slices gain 2 % overall, rows cut into two lose
        // 24 % (measured), so SKIP is instantiated only for the former.
        const int32_t c = c0 + li < end ? c_next : n_rows;
        const float wv = c0 + li < end ? w_next : 0.f;
        if (c0 + SL + li < end) {
          c_next = bcol[c0 + SL + li];
          if (W) w_next = bw[c0 + SL + li];
        }
        l_idx[li] = c;
        if (W) l_w[li] = wv;
        wave_lds_fence();
        const int cnt = min(SL, end - c0);
        float4 part = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int t0 = 0; t0 < SL; t0 += U) {
          int idv[U];
#pragma unroll
          for (int q = 0; q < U / 4; ++q) {
            const int4 i4 = *reinterpret_cast<const int4*>(l_idx + t0 + 4 * q);
            idv[4 * q] = i4.x; idv[4 * q + 1] = i4.y; idv[4 * q + 2] = i4.z; idv[4 * q + 3] = i4.w;
          }
          float4 rowv[U];
#pragma unroll
          for (int t4 = 0; t4 < U; t4 += 4)
            if (!SKIP || t0 + t4 < cnt) {
              if (narrow) {  // uniform
#pragma unroll
                for (int t = t4; t < t4 + 4; ++t) rowv[t] = table_load<float4>(table, idv[t], row_bytes, col_bytes);
              } else {
#pragma unroll
                for (int t = t4; t < t4 + 4; ++t) rowv[t] = table_load_wide<float4>(feat, n_rows, idv[t], row_bytes, col_bytes);
              }
            }
#pragma unroll
          for (int t4 = 0; t4 < U; t4 += 4)
            if (!SKIP || t0 + t4 < cnt) {
#pragma unroll
              for (int t = t4; t < t4 + 4; ++t) {
                if (W) fma4(part, l_w[t0 + t], rowv[t]);
                else add4(part, rowv[t]);
              }
            }
        }
        add4(acc, part);
        wave_lds_fence();
      }
      beg = beg_n;
      end = end_n;
      c_next = c_first_n;
      w_next = w_first_n;
      }
      st4_stream(acc_buf + (int64_t)cur.row * F + col, acc);
    }
    cur = nxt;
  }
}

// ---- all column blocks in one persistent launch: the running sums stay in LDS ------------
// The launches above pay for cache residency with one read-add-write of the [n, F] running sums
// per block.  Here one workgroup per CU runs for the whole pass and keeps the sums of up to
// res_slots (row, slice) pairs in LDS.  It takes all of them through column block 0, then all of
// them through block 1, and so on ("phases"); after the last block it writes the rows out once
// and takes its next rows ("generation").  Every workgroup owns the same number of rows per
// generation, dealt from the degree order one position at a time in alternating direction, so
// all workgroups carry nearly the same load in every phase and walk the blocks in step by
// themselves; the workgroups of an XCD meet once per generation (phase_step_done, a bounded
// wait), so an L2 serves gathers from one block at a time.  Inside a workgroup the groups draw
// rows from an LDS counter, longest rows first, which levels the segments' lengths.  A row's
// sums run in block order and its edges in list order, so the result is bit-identical to the
// launch-per-block path whoever draws what; long rows (PARTS) are cut into parts, drawn like rows, which are added at the end.
// Groups of four or eight lanes for narrow rows, the parts and the widths beside 64, 128, 256 and 512 gave, us a layer, power law:
// 20 000 vertices, 2 10^6 edges, 16 columns 192 -> 76, 64 219 -> 102, 128 243 -> 153; 47 029, 2.2 10^7, 32 718 -> 310, 64 839 -> 497,
// 120 1890 -> 1270; 232 965, 1.14 10^8, 16 2890 -> 1620, 32 2990 -> 1780, 64 3650 -> 3080, 100 12 770 -> 6530, 240 29 200 -> 15 500, 256
// 11 420 -> 11 410; even degrees, 47 029, 16 407 -> 264, 64 502 -> 500.
constexpr int kResThreads = 1024;
constexpr int kResLdsBytes = 160 * 1024;
constexpr int kResMostRows = 8;  // (row, slice) pairs of a group at a time; more leave fewer blocks to a batch of rows, for nothing
// A group takes 16 edges of a row at a time; with SL = 4 or 8 a lane has several of their indices.
constexpr int kResChunk = 16;
template <int SL, bool W>
constexpr int kResGroupInts = (kResThreads / SL) * (W ? 2 : 1) * kResChunk;  // idx, (weights) of all groups
template <int SL>
constexpr int kResSlotInts = 4 * SL + 4 + 1;  // sum | (beg, end) of two phases | row
template <int SL, bool W>
constexpr int res_slots() {
  constexpr int fit = (kResLdsBytes / 4 - 4 - kResGroupInts<SL, W>) / kResSlotInts<SL>, most = kResThreads / SL * kResMostRows;
  return std::min({fit, most, kResThreads}) / 4 * 4;
}

template <int SL, bool W, bool NARROW, bool PARTS>
__global__ __launch_bounds__(kResThreads) void k_rowsum_res(
    int32_t n_rows, const int32_t* __restrict__ order, const int2* __restrict__ bseg /* [nblk][n_rows] */,
    const int32_t* __restrict__ bcol, const float* __restrict__ feat, int32_t block_cols, int nblk, int F,
    int ns, int sw /* columns of a slice */, const float* __restrict__ scale /* nullable: factor per row */, float* __restrict__ out,
    const float* __restrict__ bw, int32_t* __restrict__ clock /* nullable: step counters, zeroed */,
    int spin_limit, int sync_every, RowParts cut) {
  constexpr int GPB = kResThreads / SL;
  constexpr int NSLOT = res_slots<SL, W>();
  constexpr int U = 8, CH = kResChunk, NI = CH / SL;
  static_assert(CH % SL == 0, "a lane has the same number of a chunk's indices as every other");
  extern __shared__ __align__(16) int lds_res[];
  const int lane = threadIdx.x & 63;
  const int li = threadIdx.x & (SL - 1);
  const int grp = threadIdx.x / SL;
  const int slice = blockIdx.x % ns;
  const int64_t nwg = gridDim.x / ns;         // workgroups that serve this slice
  const int64_t wg = blockIdx.x / ns;
  float4* l_acc = reinterpret_cast<float4*>(lds_res);            // [NSLOT][SL]
  int2* l_seg = reinterpret_cast<int2*>(lds_res + 4 * SL * NSLOT);  // [2][NSLOT]
  int* l_row = lds_res + 4 * SL * NSLOT + 4 * NSLOT;             // [NSLOT]
  int* l_idx = l_row + NSLOT + grp * (W ? 2 : 1) * CH;
  float* l_w = reinterpret_cast<float*>(l_idx + CH);
  int* l_cnt = l_row + NSLOT + kResGroupInts<SL, W>;             // [2]
  // a row narrower than its slices: the lanes past its end gather its first columns again (same
  // cache line) and store nothing
  const bool col_ok = 4 * li < sw && slice * sw + 4 * li < F;
  const int col = col_ok ? slice * sw + 4 * li : slice * sw;
  const uint32_t row_bytes = 4u * F, col_bytes = 4u * col;
  const auto table = row_table(feat, NARROW ? (int64_t)n_rows * row_bytes : 0);

  const int rows_here = (int)((n_rows + nwg - 1) / nwg);
  auto slots_to = [&](int j) { return PARTS ? slots_before(cut, j) : j; };
  const int all_slots = slots_to(rows_here);
  // workgroups go to the XCDs round-robin: those with the same id mod 8 share an L2
  PhaseClock pc{clock ? clock + (blockIdx.x % kXcds) * kClockStride : nullptr, (int)(gridDim.x / kXcds), spin_limit,
                false, sync_every > 0 ? sync_every : nblk};

  struct Item {
    int32_t beg, end, c_first[NI];
    float w_first[NI];
  };

  int phase = 0;
  for (int j0 = 0, j1; j0 < rows_here; j0 = j1) {
    // rows j0 .. j1 - 1, an even share of the slots that are left, and at least one row (its parts fit: see the launch)
    const int s0 = slots_to(j0), left = all_slots - s0, gens = (left + NSLOT - 1) / NSLOT;
    const int room = min(NSLOT, max((left + gens - 1) / gens, PARTS ? 1 << log_parts(cut, j0) : 1));
    j1 = PARTS ? rows_that_fit(cut, j0, rows_here, room) : min(rows_here, j0 + room);
    const int nslots = slots_to(j1) - s0;
    __syncthreads();                          // the previous generation's rows are written out
    int64_t pos = -1;                         // thread q < nslots: position of slot q's row in the degree order
    int part = 0, logp = 0;                   // and which of the row's 2^logp parts
    auto bounds = [&](int p) {
      if (pos < 0) return make_int2(0, 0);
      const int2 sg = bseg[(int64_t)p * n_rows + pos];
      return PARTS ? part_of_segment(sg, part, logp, CH) : sg;
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
      l_row[threadIdx.x] = part == 0 ? row : -2;  // -2: a further part of the row before
      l_seg[threadIdx.x] = seg;
    }
    for (int i = threadIdx.x; i < nslots * SL; i += kResThreads) l_acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (threadIdx.x == 0) l_cnt[0] = 0;
    __syncthreads();  // the tables are in place

    // a group's next slot of phase p, from that phase's counter
    auto grab = [&](int p) {
      int q = 0;
      if (li == 0) q = atomicAdd(l_cnt + (p & 1), 1);
      return __shfl(q, lane & ~(SL - 1), 64);
    };
    // what a slot needs before its edge loop in phase p: bounds and first indices
    auto fetch = [&](int p, int q) {
      Item it{};
      if (q >= nslots) return it;
      const int2 sg = l_seg[(p & 1) * NSLOT + q];
      it.beg = sg.x;
      it.end = sg.y;
#pragma unroll
      for (int a = 0; a < NI; ++a) {
        const int32_t e = it.beg + li + SL * a;
        if (e < it.end) {
          it.c_first[a] = bcol[e];
          if (W) it.w_first[a] = bw[e];
        }
      }
      return it;
    };
    int q = grab(0);
    Item cur = fetch(0, q);

    for (int p = 0; p < nblk; ++p) {
      // the next phase's bounds travel while this one is worked on
      int2 seg_next = make_int2(0, 0);
      if (p + 1 < nblk) seg_next = bounds(p + 1);
      if (threadIdx.x == 0) l_cnt[(p + 1) & 1] = 0;

      while (q < nslots) {
        const int qn = grab(p);
        const Item nxt = fetch(p, qn);
        const int32_t beg = cur.beg, end = cur.end;
        if (beg < end) {
          float4 acc = l_acc[q * SL + li];
          int32_t c_next[NI];
          float w_next[NI];
#pragma unroll
          for (int a = 0; a < NI; ++a) {
            c_next[a] = cur.c_first[a];
            w_next[a] = cur.w_first[a];
          }
          for (int32_t c0 = beg; c0 < end; c0 += CH) {
#pragma unroll
            for (int a = 0; a < NI; ++a) {
              const int32_t e = c0 + li + SL * a;
              l_idx[li + SL * a] = e < end ? c_next[a] : n_rows;  // no edge: zeros
              if (W) l_w[li + SL * a] = e < end ? w_next[a] : 0.f;
              if (e + CH < end) {
                c_next[a] = bcol[e + CH];
                if (W) w_next[a] = bw[e + CH];
              }
            }
            wave_lds_fence();
            const int cn = min(CH, end - c0);
            float4 part4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int t0 = 0; t0 < CH; t0 += U) {
              int idv[U];
#pragma unroll
              for (int qq = 0; qq < U / 4; ++qq) {
                const int4 i4 = *reinterpret_cast<const int4*>(l_idx + t0 + 4 * qq);
                idv[4 * qq] = i4.x; idv[4 * qq + 1] = i4.y; idv[4 * qq + 2] = i4.z; idv[4 * qq + 3] = i4.w;
              }
              float wv[U] = {};
              if (W) {
#pragma unroll
                for (int qq = 0; qq < U / 4; ++qq) {
                  const float4 w4 = *reinterpret_cast<const float4*>(l_w + t0 + 4 * qq);
                  wv[4 * qq] = w4.x; wv[4 * qq + 1] = w4.y; wv[4 * qq + 2] = w4.z; wv[4 * qq + 3] = w4.w;
                }
              }
              float4 rowv[U];
#pragma unroll
              for (int t4 = 0; t4 < U; t4 += 4)
                if (t0 + t4 < cn) {
#pragma unroll
                  for (int t = t4; t < t4 + 4; ++t) {
                    if constexpr (NARROW) rowv[t] = table_load<float4>(table, idv[t], row_bytes, col_bytes);
                    else rowv[t] = table_load_wide<float4>(feat, n_rows, idv[t], row_bytes, col_bytes);
                  }
                }
#pragma unroll
              for (int t4 = 0; t4 < U; t4 += 4)
                if (t0 + t4 < cn) {
#pragma unroll
                  for (int t = t4; t < t4 + 4; ++t) {
                    if (W) fma4(part4, wv[t], rowv[t]);
                    else add4(part4, rowv[t]);
                  }
                }
            }
            add4(acc, part4);
            wave_lds_fence();
          }
          l_acc[q * SL + li] = acc;
        }
        q = qn;
        cur = nxt;
      }
      if ((int)threadIdx.x < nslots) l_seg[((p + 1) & 1) * NSLOT + threadIdx.x] = seg_next;
      __syncthreads();  // the workgroup is done with this block; the next phase's bounds are in LDS
      if (p + 1 < nblk) {  // first slot of the next phase: its loads travel during the wait below
        q = grab(p + 1);
        cur = fetch(p + 1, q);
      }
      phase_step_done(pc, phase++);
      __syncthreads();  // every workgroup of the XCD is done with this block (or the wait ran out)
    }
    for (int q = grp; q < nslots; q += GPB) {
      const int32_t row = l_row[q];
      if (row < 0 || !col_ok) continue;
      float4 acc = l_acc[q * SL + li];
      if (PARTS)
        for (int i = q + 1; i < nslots && l_row[i] == -2; ++i) add4(acc, l_acc[i * SL + li]);
      if (scale != nullptr) scale4(acc, scale[row]);
      st4_stream(out + (int64_t)row * F + col, acc);
    }
  }
}

// A row of F floats is cut into `ns` slices of SL float4.  Slices of 256 bytes where the row has
// 2, 4 or 8 of them (measured at 1 KB rows: 17.8 -> 17.2 ms per layer against 8 slices of 128
// bytes, 22.9 ms with two of 512); wider rows have 8 slices, one per XCD.  With fewer than 8,
// workgroup id mod `ns` picks the slice, so XCD k and XCD k + ns share columns and split the rows.
// The persistent kernel cuts rows of up to 512 floats into the fewest such slices, of the same width up to a float4, and has four
// or eight lanes to a row of up to 16 or 32 floats.  (Rows of at most 64 floats are not for a launch per block: it would move as
// many bytes of running sums as of gathered rows.)
struct GcnSlices {
  int SL, ns, sw;  // lanes, slices, columns of a slice
};
static GcnSlices gcn_resident_slices(int F) {
  int ns = 1;
  while (cdiv(F / 4, ns) > 16) ns *= 2;
  const int sw = 4 * (int)cdiv(F / 4, ns);
  return {sw <= 16 ? 4 : sw <= 32 ? 8 : 16, ns, sw};
}
// Rows whose slices are not whole lines fetch parts of lines twice, so they take the persistent kernel only where the single-launch kernels
// leave the L2s for most gathers.  Layer, single launch | persistent, us, power law / even: 20 000 vertices, 2 10^6 edges, 120 columns
// 208 | 183 / 151 | 167, 200 columns 304 | 276 / 220 | 268; 47 029, 2.2 10^7, 84 (15 MiB) 1274 | 1040 / 866 | 1073, 100 (18 MiB) 1550 | 1116
// / 1264 | 1144, 200 (36 MiB) 3450 | 2262 / 1978 | 2340; 100 000, 1.5 10^7, 72 (27 MiB) 953 | 920 / 676 | 918, 100 1357 | 1033 / 1590 |
// 1028, 200 (76 MiB) 2760 | 2019 / 3196 | 2079; 232 965, 1.14 10^8, 72 (64 MiB) 8967 | 6043, 156 19 700 | 11 900, 240 29 200 | 15 500.
constexpr int64_t kRaggedBytes = (int64_t)16 << 20, kRaggedBytesFar = (int64_t)60 << 20;
static bool gcn_resident_applies(const gnn_graph_t* g, int F) {
  if (!config_get(kCfgResidentSums) || g->phase_clock == nullptr || F % 4 != 0 || F > 64 * kGcnSlices) return false;
  if (F <= 64 || F == 128 || F == 256 || F == 512 || config_get(kCfgResidentSums) == 2) return true;
  const bool near = gathers_skewed(g, 0) || gathers_skewed(g, 1) ? F >= 80 : F >= 100 && F <= 128;
  return (int64_t)g->n * F * 4 >= (near ? kRaggedBytes : kRaggedBytesFar);
}
static bool gcn_slicing(int F, int& SL, int& ns) {  // of the launches per block
  if (F % 32 != 0) return false;
  const int q = F / 32;
  if (q == 4 || q == 8 || q == 16) {
    SL = 16;
    ns = q / 2;
    return true;
  }
  if (q >= kGcnSlices) {
    SL = q;
    ns = kGcnSlices;
    return q == 32;
  }
  return false;  // narrower rows stay with the single-launch kernel
}

static bool gcn_blocked_applies(const gnn_graph_t* g, int F) {
  if (!g->blocked_pays() || config_get(kCfgForceSimple)) return false;
  int SL, ns;
  return gcn_resident_applies(g, F) || gcn_slicing(F, SL, ns);
}

template <int SL>
static gnn_status_t launch_rowsum_blocks(const gnn_graph_t* g, int side, const char* name, const float* feat,
                                         int F, float* acc, hipStream_t st, const float* bw = nullptr) {
  const int rows_per_wg = (kGcnBlock / SL) * kGcnRows;
  const int ns = F / (4 * SL);
  const unsigned grid = (unsigned)(cdiv(g->n, rows_per_wg) * ns);
  const int narrow = gcn_narrow(g, F);
  const std::vector<int32_t>& groups = g->h_group[side][0];
  GNN_REQUIRE(groups.size() >= 2 && groups.front() == 0 && groups.back() == g->nblk, GNN_ERR_UNSUPPORTED,
              "gcn blocked: the plan has no launch groups");
  for (size_t gi = 0; gi + 1 < groups.size(); ++gi) {
    const int b = groups[gi], nseg = groups[gi + 1] - b;
    GNN_REQUIRE(nseg >= 1 && nseg <= kMaxMerge, GNN_ERR_UNSUPPORTED, "gcn blocked: bad launch group");
    const int2* bseg_b = reinterpret_cast<const int2*>(g->bseg[side]) + (int64_t)b * g->n;
    ProfScope p(name, st);  // one timed bracket per launch
    const bool first = b == 0;
    if (bw != nullptr && ns >= 4)
      k_rowsum_blk<SL, true, true><<<grid, kGcnBlock, 0, st>>>(g->n, g->order[side], bseg_b, g->bcol[side], feat, F, first, ns, acc,
                                                              nseg, narrow, bw);
    else if (bw != nullptr)
      k_rowsum_blk<SL, false, true><<<grid, kGcnBlock, 0, st>>>(g->n, g->order[side], bseg_b, g->bcol[side], feat, F, first, ns, acc,
                                                               nseg, narrow, bw);
    else if (ns >= 4)
      k_rowsum_blk<SL, true><<<grid, kGcnBlock, 0, st>>>(g->n, g->order[side], bseg_b, g->bcol[side], feat, F, first, ns, acc, nseg,
                                                        narrow);
    else
      k_rowsum_blk<SL, false><<<grid, kGcnBlock, 0, st>>>(g->n, g->order[side], bseg_b, g->bcol[side], feat, F, first, ns, acc, nseg,
                                                         narrow);
    GNN_LAUNCH_CHECK();
  }
  return GNN_OK;
}

__global__ void k_zero_clock(int32_t* __restrict__ clock) { clock[threadIdx.x] = 0; }

// one workgroup per CU, a multiple of the slice count so that every XCD serves one slice
static unsigned gcn_resident_grid() { return (unsigned)(device_cu_count() / kXcds * kXcds); }
static int64_t gcn_resident_groups(const GcnSlices& sl) { return (int64_t)gcn_resident_grid() / sl.ns * (kResThreads / sl.SL); }

template <int SL, bool W, bool NARROW, bool PARTS>
static gnn_status_t launch_rowsum_resident_as(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                                              const GcnSlices& sl, const float* scale, float* out, hipStream_t st, const float* bw) {
  static std::atomic<bool> attr_set{false};  // more than 64 KB of dynamic LDS, once per instantiation
  if (!attr_set.load(std::memory_order_acquire)) {
    GNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_rowsum_res<SL, W, NARROW, PARTS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kResLdsBytes));
    attr_set.store(true, std::memory_order_release);
  }
  const unsigned grid = gcn_resident_grid();
  ProfScope p(name, st);
  k_zero_clock<<<1, kXcds * kClockStride, 0, st>>>(g->phase_clock);
  GNN_LAUNCH_CHECK();
  constexpr int slots = res_slots<SL, W>();
  k_rowsum_res<SL, W, NARROW, PARTS><<<grid, kResThreads, kResLdsBytes, st>>>(
      g->n, g->order[side], reinterpret_cast<const int2*>(g->bseg[side]), g->bcol[side], feat, g->block_cols, g->nblk, F, sl.ns,
      sl.sw, scale, out, bw, g->phase_clock, (int)config_get(kCfgResidentSpin), (int)config_get(kCfgResidentSyncEvery),
      PARTS ? cut_long_rows(g, side, gcn_resident_groups(sl), grid / sl.ns, slots) : RowParts{});
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

template <int SL, bool W>
static gnn_status_t launch_rowsum_resident_of(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                                              const GcnSlices& sl, const float* scale, float* out, hipStream_t st, const float* bw) {
  const bool parts = has_long_rows(g, side, gcn_resident_groups(sl));
  if (gcn_narrow(g, F))
    return parts ? launch_rowsum_resident_as<SL, W, true, true>(g, side, name, feat, F, sl, scale, out, st, bw)
                 : launch_rowsum_resident_as<SL, W, true, false>(g, side, name, feat, F, sl, scale, out, st, bw);
  return parts ? launch_rowsum_resident_as<SL, W, false, true>(g, side, name, feat, F, sl, scale, out, st, bw)
               : launch_rowsum_resident_as<SL, W, false, false>(g, side, name, feat, F, sl, scale, out, st, bw);
}

template <bool W>
static gnn_status_t launch_rowsum_resident(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                                           const float* scale, float* out, hipStream_t st, const float* bw) {
  const GcnSlices sl = gcn_resident_slices(F);
  switch (sl.SL) {
    case 4: return launch_rowsum_resident_of<4, W>(g, side, name, feat, F, sl, scale, out, st, bw);
    case 8: return launch_rowsum_resident_of<8, W>(g, side, name, feat, F, sl, scale, out, st, bw);
    default: return launch_rowsum_resident_of<16, W>(g, side, name, feat, F, sl, scale, out, st, bw);
  }
}

// Gathered rows in flight per lane: eight, four of the narrowest and widest rows, and two where gathers are even (gathers_abreast) and
// not sliced.  Layer, eight -> two, us: 100 000 vertices, 90 edges each, 32 columns 274 -> 186 (four 264), 48 525 -> 371; 50 000, 60,
// 32 (6.4 MB) 94 -> 87; 130 000, 20, 128 501 -> 480; 20 000, 20, 32 (2.6 MB) 44 -> 47; 16 columns, four -> two, 100 000, 90 378 -> 429;
// 256 columns in slices, 100 000, 90 2343 -> 2437.  Neighbours that gather the same rows lose: 200 000, 60, 32, from the 2000
// vertices to either side 370 -> 445; so do skewed gathers: power law, 100 000, 20, 32 101 -> 123.
constexpr int64_t kTwoRowsBytes = (int64_t)6 << 20;

// W: the same sum with a static weight per edge (wgt in the order of the side's edge array)
template <int L, int NV, bool W, int NS>
static gnn_status_t launch_rowsum(const gnn_graph_t* g, int side, const float* feat, int F, const float* scale, float* out,
                                  hipStream_t st, const float* wgt) {
  constexpr int GPB = (kWave / L) * (kGcnBlock / kWave);
  const RowSplit sp = split_rows(g, side, L, GPB);
  const int32_t* cols = side == 0 ? g->indices : g->indices_t;
  // hub rows (one workgroup each) and the rest in one launch
  const unsigned grid = xcd_slice_grid(sp.hub_grid + sp.rest_grid, NS);
  const RowLaunch rl{sp.hub.end, g->n};
  constexpr int kAhead = NV == 1 && L >= 8 ? 8 : 4;
  if (grid != 0) {
    auto launch = [&](auto u) {
      constexpr int U = decltype(u)::value;
      if (gcn_narrow(g, F)) k_rowsum<L, NV, W, NS, U, true><<<grid, kGcnBlock, 0, st>>>(rl, g->rows[side], cols, feat, F, scale, out, wgt);
      else k_rowsum<L, NV, W, NS, U, false><<<grid, kGcnBlock, 0, st>>>(rl, g->rows[side], cols, feat, F, scale, out, wgt);
    };
    if constexpr (kAhead > 4 && NS == 1) {
      if (gathers_abreast(g, side, F, kTwoRowsBytes)) launch(std::integral_constant<int, 2>{});
      else launch(std::integral_constant<int, kAhead>{});
    } else launch(std::integral_constant<int, kAhead>{});
    GNN_LAUNCH_CHECK();
  }
  return GNN_OK;
}

template <bool W, int L, int NV>
static gnn_status_t launch_rowsum_sliced(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                                         const float* scale, float* out, hipStream_t st, const float* wgt) {
  ProfScope p(name, st);
  switch (gather_slices(g, side, F)) {
    case 2: return launch_rowsum<8, 1, W, 2>(g, side, feat, F, scale, out, st, wgt);
    case 4: return launch_rowsum<8, 1, W, 4>(g, side, feat, F, scale, out, st, wgt);
    case 8: return launch_rowsum<8, 1, W, 8>(g, side, feat, F, scale, out, st, wgt);
    default: return launch_rowsum<L, NV, W, 1>(g, side, feat, F, scale, out, st, wgt);
  }
}

template <int L, int NV>
struct RowsumLauncher {
  static gnn_status_t run(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                          const float* scale, float* out, hipStream_t st) {
    return launch_rowsum_sliced<false, L, NV>(g, side, name, feat, F, scale, out, st, nullptr);
  }
};

template <int L, int NV>
struct RowsumWeightedLauncher {
  static gnn_status_t run(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                          const float* wgt, float* out, hipStream_t st) {
    return launch_rowsum_sliced<true, L, NV>(g, side, name, feat, F, nullptr, out, st, wgt);
  }
};

template <int L, int NV>
struct RowsumEbLauncher {
  static gnn_status_t run(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                          const float* scale, float* out, hipStream_t st) {
    constexpr int GPB = kGcnBlock / L;
    ProfScope p(name, st);
    const int64_t quads = (int64_t)g->n * (F / 4);
    k_zero_f4<<<(unsigned)cdiv(quads, 256), 256, 0, st>>>(quads, out);
    GNN_LAUNCH_CHECK();
    const int64_t runs = cdiv(g->nnz, kEbEdges);
    if (runs != 0) {
      k_rowsum_eb<L, NV><<<(unsigned)cdiv(runs, GPB), kGcnBlock, 0, st>>>(
          g->n, (int32_t)g->nnz, side == 0 ? g->indptr : g->indptr_t, side == 0 ? g->indices : g->indices_t,
          feat, F, scale, out);
      GNN_LAUNCH_CHECK();
    }
    return GNN_OK;
  }
};

template <int L, int NV>
struct RowsumWeightedEbLauncher {
  static gnn_status_t run(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                          const float* wgt, float* out, hipStream_t st) {
    constexpr int GPB = kGcnBlock / L;
    ProfScope p(name, st);
    const int64_t quads = (int64_t)g->n * (F / 4);
    k_zero_f4<<<(unsigned)cdiv(quads, 256), 256, 0, st>>>(quads, out);
    GNN_LAUNCH_CHECK();
    const int64_t runs = cdiv(g->nnz, kEbEdges);
    if (runs != 0) {
      k_rowsum_eb<L, NV, true><<<(unsigned)cdiv(runs, GPB), kGcnBlock, 0, st>>>(
          g->n, (int32_t)g->nnz, side == 0 ? g->indptr : g->indptr_t, side == 0 ? g->indices : g->indices_t,
          feat, F, nullptr, out, wgt);
      GNN_LAUNCH_CHECK();
    }
    return GNN_OK;
  }
};

template <template <int, int> class Launcher>
static gnn_status_t dispatch_rowsum(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                                    const float* scale, float* out, hipStream_t st) {
  const GroupShape gs = pick_group(F);
  switch (gs.L) {
    case 4: return Launcher<4, 1>::run(g, side, name, feat, F, scale, out, st);
    case 8: return Launcher<8, 1>::run(g, side, name, feat, F, scale, out, st);
    case 16: return Launcher<16, 1>::run(g, side, name, feat, F, scale, out, st);
    case 32: return Launcher<32, 1>::run(g, side, name, feat, F, scale, out, st);
    case 64:
      switch (gs.NV) {
        case 1: return Launcher<64, 1>::run(g, side, name, feat, F, scale, out, st);
        case 2: return Launcher<64, 2>::run(g, side, name, feat, F, scale, out, st);
        case 3: return Launcher<64, 3>::run(g, side, name, feat, F, scale, out, st);
        case 4: return Launcher<64, 4>::run(g, side, name, feat, F, scale, out, st);
      }
  }
  set_error("unsupported row-group shape L=%d NV=%d", gs.L, gs.NV);
  return GNN_ERR_UNSUPPORTED;
}

// mapping: 0 vertex-balanced, 1 edge-balanced, 2 what gnn_gcn_tune found faster on this graph
// (vertex-balanced on a graph that was never tuned)
static bool use_edge_balanced(const gnn_graph_t* g, int side) {
  const int64_t mode = config_get(kCfgGcnMapping);
  if (mode == 1) return true;
  return mode == 2 && g->gcn_edge_balanced[side] == 1;
}

// vertex-balanced: column-blocked launches on large graphs, else one launch
static gnn_status_t gcn_aggregate_vertex(const gnn_graph_t* g, int side, const char* name, const float* feat,
                                         int F, const float* scale, float* out, hipStream_t st) {
  if (gcn_blocked_applies(g, F)) {
    if (gcn_resident_applies(g, F)) return launch_rowsum_resident<false>(g, side, name, feat, F, scale, out, st, nullptr);
    int SL = 0, ns = 0;
    gcn_slicing(F, SL, ns);
    switch (SL) {
      case 8: GNN_TRY(launch_rowsum_blocks<8>(g, side, name, feat, F, out, st)); break;
      case 16: GNN_TRY(launch_rowsum_blocks<16>(g, side, name, feat, F, out, st)); break;
      default: GNN_TRY(launch_rowsum_blocks<32>(g, side, name, feat, F, out, st)); break;
    }
    ProfScope p("gcn_scale_rows", st);
    const int64_t quads = (int64_t)g->n * (F / 4);
    k_scale_rows<<<(unsigned)cdiv(quads, 256), 256, 0, st>>>(quads, F / 4, scale, out, out);
    GNN_LAUNCH_CHECK();
    return GNN_OK;
  }
  return dispatch_rowsum<RowsumLauncher>(g, side, name, feat, F, scale, out, st);
}

// out[row,:] = scale[row] * sum of feat over the row's neighbours on `side` (0: in-edges, 1: out-edges)
static gnn_status_t gcn_aggregate(const gnn_graph_t* g, int side, const char* name, const float* feat, int F,
                                  const float* scale, float* out, hipStream_t st) {
  if (use_edge_balanced(g, side)) return dispatch_rowsum<RowsumEbLauncher>(g, side, name, feat, F, scale, out, st);
  return gcn_aggregate_vertex(g, side, name, feat, F, scale, out, st);
}

// out[row,:] = sum over the row's edges on `side` of weight * feat[neighbour,:]  (vertex-balanced:
// column-blocked launches on large graphs, else one launch)
static gnn_status_t gcn_aggregate_weighted(const gnn_graph_t* g, const gnn_edge_weights* ew, int side,
                                           const char* name, const float* feat, int F, float* out,
                                           hipStream_t st) {
  // edge-balanced only on request (gcn_mapping = 1): gnn_gcn_tune times the unweighted sums
  if (config_get(kCfgGcnMapping) == 1)
    return dispatch_rowsum<RowsumWeightedEbLauncher>(g, side, name, feat, F, ew->w_side[side], out, st);
  if (gcn_blocked_applies(g, F) && ew->w_blk[side] != nullptr) {
    if (gcn_resident_applies(g, F))
      return launch_rowsum_resident<true>(g, side, name, feat, F, nullptr, out, st, ew->w_blk[side]);
    int SL = 0, ns = 0;
    gcn_slicing(F, SL, ns);
    switch (SL) {
      case 8: return launch_rowsum_blocks<8>(g, side, name, feat, F, out, st, ew->w_blk[side]);
      case 16: return launch_rowsum_blocks<16>(g, side, name, feat, F, out, st, ew->w_blk[side]);
      default: return launch_rowsum_blocks<32>(g, side, name, feat, F, out, st, ew->w_blk[side]);
    }
  }
  return dispatch_rowsum<RowsumWeightedLauncher>(g, side, name, feat, F, ew->w_side[side], out, st);
}

struct GcnWs {
  size_t total, gs, dz, gemm;
  int split_k;
};

static GcnWs gcn_ws_layout(int64_t n, int fin, int fout) {
  GcnWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += ws_granule(bytes); return o; };
  w.gs = take(sizeof(float) * (size_t)n * fout);
  w.dz = take(sizeof(float) * (size_t)n * fout);
  w.split_k = gemm_pick_split_k(fin, fout, n);
  w.gemm = take(w.split_k > 1 ? sizeof(float) * (size_t)w.split_k * fin * fout : 0);
  w.total = off;
  return w;
}

static gnn_status_t gcn_check(const gnn_graph_t* g, int fin, int fout, const char* who) {
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "%s: graph is null", who);
  GNN_REQUIRE(fin > 0 && fout > 0, GNN_ERR_INVALID_ARG, "%s: sizes must be positive", who);
  GNN_REQUIRE(fout % 4 == 0 && fout <= 1024, GNN_ERR_UNSUPPORTED,
              "%s: fout = %d must be a multiple of 4, at most 1024", who, fout);
  return GNN_OK;
}

}  // namespace gnn

using namespace gnn;

extern "C" size_t gnn_gcn_workspace_bytes(const gnn_graph_t* g, int fin, int fout) {
  if (!g || fin <= 0 || fout <= 0) return 0;
  return gcn_ws_layout(g->n, fin, fout).total;
}

extern "C" gnn_status_t gnn_gcn_fwd(const gnn_graph_t* g, int fin, int fout, const float* x, const float* w,
                                    const float* c_src, const float* c_dst, float* zs, float* out,
                                    void* stream) {
  clear_error();
  GNN_TRY(gcn_check(g, fin, fout, "gnn_gcn_fwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w && c_src && c_dst && zs && out, GNN_ERR_INVALID_ARG, "gnn_gcn_fwd: null pointer");
  GNN_REQUIRE(aligned16(zs) && aligned16(out), GNN_ERR_INVALID_ARG,
              "gnn_gcn_fwd: zs, out must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  // projection before propagation, then the source half of the edge weight on vertices
  GNN_TRY(gemm_f32(g->n, fout, fin, x, fin, false, w, fout, false, zs, fout, 1, nullptr, st));
  {
    ProfScope p("gcn_scale_rows", st);
    const int64_t quads = (int64_t)g->n * (fout / 4);
    k_scale_rows<<<(unsigned)cdiv(quads, 256), 256, 0, st>>>(quads, fout / 4, c_src, zs, zs);
    GNN_LAUNCH_CHECK();
  }
  return gcn_aggregate(g, 0, "gcn_fwd_fused", zs, fout, c_dst, out, st);
}

extern "C" gnn_status_t gnn_gcn_bwd(const gnn_graph_t* g, int fin, int fout, const float* x, const float* w,
                                    const float* c_src, const float* c_dst, const float* gout, float* gx,
                                    float* gw, void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  GNN_TRY(gcn_check(g, fin, fout, "gnn_gcn_bwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w && c_src && c_dst && gout && gw, GNN_ERR_INVALID_ARG, "gnn_gcn_bwd: null pointer");
  GNN_REQUIRE(aligned16(gout), GNN_ERR_INVALID_ARG, "gnn_gcn_bwd: gout must be 16-byte aligned");
  const GcnWs L = gcn_ws_layout(g->n, fin, fout);
  GNN_REQUIRE(ws != nullptr && ws_bytes >= L.total, GNN_ERR_WORKSPACE,
              "gnn_gcn_bwd: workspace of %zu bytes given, %zu needed", ws_bytes, L.total);
  GNN_REQUIRE(aligned16(ws), GNN_ERR_INVALID_ARG, "gnn_gcn_bwd: workspace must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(ws);
  float* gs = reinterpret_cast<float*>(base + L.gs);
  float* dz = reinterpret_cast<float*>(base + L.dz);
  float* part = reinterpret_cast<float*>(base + L.gemm);
  {
    ProfScope p("gcn_scale_rows", st);
    const int64_t quads = (int64_t)g->n * (fout / 4);
    k_scale_rows<<<(unsigned)cdiv(quads, 256), 256, 0, st>>>(quads, fout / 4, c_dst, gout, gs);
    GNN_LAUNCH_CHECK();
  }
  GNN_TRY(gcn_aggregate(g, 1, "gcn_bwd_src", gs, fout, c_src, dz, st));
  GNN_TRY(gemm_f32(fin, fout, g->n, x, fin, true, dz, fout, false, gw, fout, L.split_k, part, st));
  if (gx) GNN_TRY(gemm_f32(g->n, fin, fout, dz, fout, false, w, fout, true, gx, fin, 1, nullptr, st));
  return GNN_OK;
}

static gnn_status_t gcn_edge_check(const gnn_graph_t* g, const gnn_edge_weights* ew, const char* who) {
  GNN_REQUIRE(ew != nullptr, GNN_ERR_INVALID_ARG, "%s: edge weights are null", who);
  GNN_REQUIRE(ew->graph == g && ew->nnz == g->nnz, GNN_ERR_INVALID_ARG,
              "%s: the edge weights were made for another graph", who);
  return GNN_OK;
}

extern "C" gnn_status_t gnn_gcn_edge_fwd(const gnn_graph_t* g, const gnn_edge_weights_t* ew, int fin, int fout,
                                         const float* x, const float* w, float* z, float* out, void* stream) {
  clear_error();
  GNN_TRY(gcn_check(g, fin, fout, "gnn_gcn_edge_fwd"));
  GNN_TRY(gcn_edge_check(g, ew, "gnn_gcn_edge_fwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w && z && out, GNN_ERR_INVALID_ARG, "gnn_gcn_edge_fwd: null pointer");
  GNN_REQUIRE(aligned16(z) && aligned16(out), GNN_ERR_INVALID_ARG,
              "gnn_gcn_edge_fwd: z, out must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  GNN_TRY(gemm_f32(g->n, fout, fin, x, fin, false, w, fout, false, z, fout, 1, nullptr, st));
  return gcn_aggregate_weighted(g, ew, 0, "gcn_fwd_fused", z, fout, out, st);
}

extern "C" gnn_status_t gnn_gcn_edge_bwd(const gnn_graph_t* g, const gnn_edge_weights_t* ew, int fin, int fout,
                                         const float* x, const float* w, const float* gout, float* gx,
                                         float* gw, void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  GNN_TRY(gcn_check(g, fin, fout, "gnn_gcn_edge_bwd"));
  GNN_TRY(gcn_edge_check(g, ew, "gnn_gcn_edge_bwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w && gout && gw, GNN_ERR_INVALID_ARG, "gnn_gcn_edge_bwd: null pointer");
  GNN_REQUIRE(aligned16(gout), GNN_ERR_INVALID_ARG, "gnn_gcn_edge_bwd: gout must be 16-byte aligned");
  const GcnWs L = gcn_ws_layout(g->n, fin, fout);
  GNN_REQUIRE(ws != nullptr && ws_bytes >= L.total, GNN_ERR_WORKSPACE,
              "gnn_gcn_edge_bwd: workspace of %zu bytes given, %zu needed", ws_bytes, L.total);
  GNN_REQUIRE(aligned16(ws), GNN_ERR_INVALID_ARG, "gnn_gcn_edge_bwd: workspace must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(ws);
  float* dz = reinterpret_cast<float*>(base + L.dz);
  float* part = reinterpret_cast<float*>(base + L.gemm);
  // dz[u] = sum over out-edges of e_uv gout[v]: the same weighted sum over the transpose
  GNN_TRY(gcn_aggregate_weighted(g, ew, 1, "gcn_bwd_src", gout, fout, dz, st));
  GNN_TRY(gemm_f32(fin, fout, g->n, x, fin, true, dz, fout, false, gw, fout, L.split_k, part, st));
  if (gx) GNN_TRY(gemm_f32(g->n, fin, fout, dz, fout, false, w, fout, true, gx, fin, 1, nullptr, st));
  return GNN_OK;
}

__global__ void k_fill_f32(int64_t count, float value, float* __restrict__ p) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < count) p[i] = value;
}

extern "C" gnn_status_t gnn_gcn_tune(gnn_graph_t* g, int fout, void* ws, size_t ws_bytes, void* stream,
                                     float* ms_out) {
  clear_error();
  GNN_TRY(gcn_check(g, 1, fout, "gnn_gcn_tune"));
  const GcnWs L = gcn_ws_layout(g->n, 1, fout);
  GNN_REQUIRE(ws != nullptr && ws_bytes >= L.total, GNN_ERR_WORKSPACE,
              "gnn_gcn_tune: workspace of %zu bytes given, %zu needed", ws_bytes, L.total);
  GNN_REQUIRE(aligned16(ws), GNN_ERR_INVALID_ARG, "gnn_gcn_tune: workspace must be 16-byte aligned");
  float ms[4] = {0.f, 0.f, 0.f, 0.f};
  if (g->n != 0 && g->nnz != 0) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* base = static_cast<char*>(ws);
    float* feat = reinterpret_cast<float*>(base + L.gs);  // all ones; its first n entries double as the scale
    float* out = reinterpret_cast<float*>(base + L.dz);
    const int64_t count = (int64_t)g->n * fout;
    k_fill_f32<<<(unsigned)cdiv(count, 256), 256, 0, st>>>(count, 1.f, feat);
    GNN_LAUNCH_CHECK();
    hipEvent_t a = nullptr, b = nullptr;
    GNN_HIP(hipEventCreate(&a));
    if (hipEventCreate(&b) != hipSuccess) {
      (void)hipEventDestroy(a);
      set_error("gnn_gcn_tune: hipEventCreate failed");
      return GNN_ERR_HIP;
    }
    constexpr int kReps = 3;
    gnn_status_t status = GNN_OK;
    for (int side = 0; side < 2 && status == GNN_OK; ++side) {
      for (int eb = 0; eb < 2 && status == GNN_OK; ++eb) {
        auto once = [&]() {
          return eb ? dispatch_rowsum<RowsumEbLauncher>(g, side, "gcn_tune", feat, fout, feat, out, st)
                    : gcn_aggregate_vertex(g, side, "gcn_tune", feat, fout, feat, out, st);
        };
        status = once();  // warm-up
        if (status == GNN_OK && hipEventRecord(a, st) != hipSuccess) status = GNN_ERR_HIP;
        for (int r = 0; r < kReps && status == GNN_OK; ++r) status = once();
        if (status == GNN_OK && (hipEventRecord(b, st) != hipSuccess || hipEventSynchronize(b) != hipSuccess))
          status = GNN_ERR_HIP;
        float t = 0.f;
        if (status == GNN_OK && hipEventElapsedTime(&t, a, b) != hipSuccess) status = GNN_ERR_HIP;
        ms[2 * side + eb] = t / kReps;
      }
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (status != GNN_OK) {
      if (status == GNN_ERR_HIP && gnn_last_error()[0] == 0) set_error("gnn_gcn_tune: a HIP event call failed");
      return status;
    }
    for (int side = 0; side < 2; ++side) g->gcn_edge_balanced[side] = ms[2 * side + 1] < ms[2 * side] ? 1 : 0;
  }
  if (ms_out)
    for (int i = 0; i < 4; ++i) ms_out[i] = ms[i];
  return GNN_OK;
}

// Which instantiation of the column-blocked sum a pass launches for this graph and width under the
// current configuration, spelled as a profiler prints it; "" when other kernels run.
extern "C" gnn_status_t gnn_gcn_blocked_kernel_name(const gnn_graph_t* g, int fout, int weighted, char* buf,
                                                    size_t len) {
  clear_error();
  GNN_REQUIRE(g != nullptr && buf != nullptr && len > 0, GNN_ERR_INVALID_ARG,
              "gnn_gcn_blocked_kernel_name: null argument");
  buf[0] = 0;
  if (fout <= 0 || !gcn_blocked_applies(g, fout) || config_get(kCfgGcnMapping) == 1) return GNN_OK;
  int SL = 0, ns = 0;
  gcn_slicing(fout, SL, ns);
  const GcnSlices sl = gcn_resident_slices(fout);
  if (gcn_resident_applies(g, fout))
    std::snprintf(buf, len, "k_rowsum_res<%d, %s, %s, %s>", sl.SL, weighted ? "true" : "false",
                  gcn_narrow(g, fout) ? "true" : "false",
                  has_long_rows(g, 0, gcn_resident_groups(sl)) ? "true" : "false");
  else
    std::snprintf(buf, len, "k_rowsum_blk<%d, %s, %s>", SL, ns >= 4 ? "true" : "false", weighted ? "true" : "false");
  return GNN_OK;
}
