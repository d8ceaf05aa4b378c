// MoNet / GMMConv layer with general pseudo-coordinates (App. A.2 "GMMConv": w_k(m) for an
// r-dimensional m_uv; Sec. 7.2 uses r = 1, 2, 3), and the learnable projection of the degree
// pair that produces them.
//
//   w_k(e)  = exp(-1/2 sum_d ((m[e,d] - mu[k,d]) inv_sigma[k,d])^2)            (ApplyEdge)
//   out[v]  = (1/K) sum_in-edges sum_k w_k(e) hk[u,k,:]                         (Aggregate)
//
// m is a per-edge input [E, r] in CSR order (an input like the graph itself, not an
// intermediate: nothing else per-edge is stored).  Forward fuses the Gaussian weights with the
// aggregation as in the degree-pair layer.  Backward recomputes the weights:
//   destination side (CSR walk): dw_k(e) = <gout[v], hk[u,k,:]> / K needs one dot product per edge
//     and kernel here (the pseudo-coordinates vary freely along a row, so the dot product cannot
//     be postponed past the neighbourhood sum as in the degree-pair layer); from it
//     gmu, ginv_sigma (summed over all edges in a fixed two-stage order) and gm[e,:];
//   source side (CSC walk, no atomics): dhk[u,k,:] = (1/K) sum_out-edges w_k(e) gout[v,:],
//     with m read through the plan's CSC position -> CSR edge id table.
// These are two kernels where a row of hk is wider than 64 floats.  Narrower rows (K fout <= 64) have both sides in one walk over the
// out-edges, which owns hk[u]: gmu, ginv_sigma, dhk and, where the coordinates are made on the spot, the
// projection's gradients.  gm[e,:] comes from that walk too while the array stays in the caches, otherwise from a walk
// over the in-edges of its own.
// At most 4 kernels and 4 pseudo-coordinate dimensions; fout <= 256.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "common.h"
#include "partial_sums.h"
#include "row_parts.h"
#include "rowgroup.h"

namespace gnn {

constexpr int kPsBlock = 256;
constexpr int kPsK = 4;   // kernels
constexpr int kPsR = 4;   // pseudo-coordinate dimensions
constexpr int kPsVals = 2 * kPsK * kPsR;  // gmu and ginv_sigma entries per partial slot

struct PsParams {
  int K, R, F;
  int wide;  // 64-bit row offsets also where 32 bits reach every row ("wide_offsets")
};

// the K x R means and inverse widths, zero-padded to KT x RT, in registers (uniform)
template <int KT = kPsK, int RT = kPsR>
struct PsKernels {
  float mu[KT][RT], is[KT][RT];
};
template <int KT = kPsK, int RT = kPsR>
__device__ __forceinline__ PsKernels<KT, RT> load_kernels(const float* __restrict__ mu, const float* __restrict__ is,
                                                          int K, int R) {
  PsKernels<KT, RT> p;
#pragma unroll
  for (int k = 0; k < KT; ++k)
#pragma unroll
    for (int d = 0; d < RT; ++d) {
      const bool ok = k < K && d < R;
      p.mu[k][d] = ok ? mu[k * R + d] : 0.f;
      p.is[k][d] = ok ? is[k * R + d] : 0.f;
    }
  return p;
}
template <int RT>
__device__ __forceinline__ void load_pseudo(const float* __restrict__ m, int64_t e, int R, float (&out)[RT]) {
#pragma unroll
  for (int d = 0; d < RT; ++d) out[d] = d < R ? m[e * R + d] : 0.f;
}
template <int KT, int RT>
__device__ __forceinline__ float gauss_k(const PsKernels<KT, RT>& p, int k, const float (&m)[RT]) {
  float q = 0.f;
#pragma unroll
  for (int d = 0; d < RT; ++d) {  // padded dimensions have inv_sigma 0
    const float t = (m[d] - p.mu[k][d]) * p.is[k][d];
    q = fmaf(t, t, q);
  }
  return __expf(-0.5f * q);
}

// ---- forward: one row group per destination (hub rows: one workgroup), one edge at a time ----
template <int L>
__global__ __launch_bounds__(kPsBlock) void k_gmmp_fwd(
    RowLaunch rl, const int32_t* __restrict__ order, const int32_t* __restrict__ indptr,
    const int32_t* __restrict__ indices, const float* __restrict__ hk, const float* __restrict__ pseudo,
    const float* __restrict__ mu, const float* __restrict__ inv_sigma, PsParams pm, float* __restrict__ out) {
  constexpr int GPB = kPsBlock / L;
  __shared__ float coop_buf[GPB * L * 4];
  const int li = threadIdx.x & (L - 1);
  const int grp = threadIdx.x / L;
  int64_t r;
  int gi, ngrp;
  RowRange rr;
  if (!pick_row<GPB>(rl, grp, rr, r, gi, ngrp)) return;
  const int K = pm.K, R = pm.R, F = pm.F, KF = K * F;
  const float inv_k = 1.f / (float)K;
  const PsKernels<> pk = load_kernels(mu, inv_sigma, K, R);
  const int32_t v = order[r];
  const int32_t beg = indptr[v], end = indptr[v + 1];
  const bool col_ok = 4 * li < F;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), part = acc;
  int folded = 0;
  for (int32_t e = beg + gi; e < end; e += ngrp) {
    const int32_t u = indices[e];
    float m[kPsR];
    load_pseudo(pseudo, e, R, m);
    if (col_ok) {
      float4 rowv[kPsK];
#pragma unroll
      for (int k = 0; k < kPsK; ++k)
        if (k < K) rowv[k] = ld4(hk + (int64_t)u * KF + k * F + 4 * li);
#pragma unroll
      for (int k = 0; k < kPsK; ++k)
        if (k < K) fma4(part, gauss_k(pk, k, m) * inv_k, rowv[k]);
    }
    if (++folded == 32) {  // two-level summation keeps long rows accurate
      add4(acc, part);
      part = make_float4(0.f, 0.f, 0.f, 0.f);
      folded = 0;
    }
  }
  add4(acc, part);
  if (rr.coop) {
    float vv[4];
    pack4(vv, acc);
    coop_sum<L, 4, GPB>(coop_buf, vv, grp, li);
    if (grp != 0) return;
    acc = unpack4(vv);
  }
  if (col_ok) st4(out + (int64_t)v * F + 4 * li, acc);
}

// ---- backward, destination side: gmu, ginv_sigma partials and gm[e,:] -------------------------
// partial[block][kPsVals]: entries k*R+d of gmu, then of ginv_sigma, summed over the block's edges
// in a fixed order (group slots, then groups in order).
template <int L>
__global__ __launch_bounds__(kPsBlock) void k_gmmp_bwd_dst(
    RowLaunch rl, const int32_t* __restrict__ order, const int32_t* __restrict__ indptr,
    const int32_t* __restrict__ indices, const float* __restrict__ hk, const float* __restrict__ pseudo,
    const float* __restrict__ mu, const float* __restrict__ inv_sigma, const float* __restrict__ gout,
    PsParams pm, float* __restrict__ partial, float* __restrict__ gpseudo /* nullable */) {
  constexpr int GPB = kPsBlock / L;
  __shared__ float blk[GPB][kPsVals];
  const int li = threadIdx.x & (L - 1);
  const int grp = threadIdx.x / L;
  int64_t r;
  int gi, ngrp;
  RowRange rr;
  const bool active = pick_row<GPB>(rl, grp, rr, r, gi, ngrp);
  const int K = pm.K, R = pm.R, F = pm.F, KF = K * F;
  const float inv_k = 1.f / (float)K;
  float gm_acc[kPsK][kPsR], gs_acc[kPsK][kPsR];  // every lane of the group keeps the same sums
#pragma unroll
  for (int k = 0; k < kPsK; ++k)
#pragma unroll
    for (int d = 0; d < kPsR; ++d) {
      gm_acc[k][d] = 0.f;
      gs_acc[k][d] = 0.f;
    }
  if (active) {
    const PsKernels<> pk = load_kernels(mu, inv_sigma, K, R);
    const int32_t v = order[r];
    const int32_t beg = indptr[v], end = indptr[v + 1];
    const bool col_ok = 4 * li < F;
    const float4 g4 = col_ok ? ld4(gout + (int64_t)v * F + 4 * li) : make_float4(0.f, 0.f, 0.f, 0.f);
    for (int32_t e = beg + gi; e < end; e += ngrp) {
      const int32_t u = indices[e];
      float m[kPsR];
      load_pseudo(pseudo, e, R, m);
      float dots[kPsK];
#pragma unroll
      for (int k = 0; k < kPsK; ++k) {
        dots[k] = 0.f;
        if (k < K && col_ok) dots[k] = dot4(g4, ld4(hk + (int64_t)u * KF + k * F + 4 * li));
      }
      float gm[kPsR];
#pragma unroll
      for (int d = 0; d < kPsR; ++d) gm[d] = 0.f;
#pragma unroll
      for (int k = 0; k < kPsK; ++k) {
        if (k >= K) continue;
        const float dw = group_sum_from<L>(dots[k], 1) * inv_k;  // <gout[v], hk[u,k,:]> / K, in every lane
        const float dlog = dw * gauss_k(pk, k, m);
#pragma unroll
        for (int d = 0; d < kPsR; ++d) {
          const float diff = m[d] - pk.mu[k][d];
          const float is = pk.is[k][d];
          const float t = dlog * diff * is;  // padded dimensions: is = 0
          gm_acc[k][d] = fmaf(t, is, gm_acc[k][d]);
          gs_acc[k][d] = fmaf(-t, diff, gs_acc[k][d]);
          gm[d] = fmaf(-t, is, gm[d]);
        }
      }
      if (gpseudo != nullptr && li == 0) {
#pragma unroll
        for (int d = 0; d < kPsR; ++d)
          if (d < R) gpseudo[(int64_t)e * R + d] = gm[d];
      }
    }
  }
  // lane 0 of every group parks its sums; then one thread per entry adds the groups in order
  if (li == 0) {
#pragma unroll
    for (int k = 0; k < kPsK; ++k)
#pragma unroll
      for (int d = 0; d < kPsR; ++d) {
        blk[grp][k * kPsR + d] = gm_acc[k][d];
        blk[grp][kPsK * kPsR + k * kPsR + d] = gs_acc[k][d];
      }
  }
  __syncthreads();
  if (threadIdx.x < kPsVals) {
    float s = 0.f;
    for (int g2 = 0; g2 < GPB; ++g2) s += blk[g2][threadIdx.x];
    partial[(int64_t)blockIdx.x * kPsVals + threadIdx.x] = s;
  }
}

// totals [kPsVals] (padded K x R layout) -> gmu, ginv_sigma [K, R]
__global__ void k_gmmp_param_split(int K, int R, const float* __restrict__ totals, float* __restrict__ gmu,
                                   float* __restrict__ gis) {
  const int i = threadIdx.x;
  if (i >= K * R) return;
  const int k = i / R, d = i - k * R;
  gmu[i] = totals[k * kPsR + d];
  gis[i] = totals[kPsK * kPsR + k * kPsR + d];
}

// ---- backward, source side: dhk[u,k,:] = (1/K) sum over out-edges w_k(e) gout[v,:] ------------
template <int L>
__global__ __launch_bounds__(kPsBlock) void k_gmmp_bwd_src(
    RowLaunch rl, const int32_t* __restrict__ order_t, const int32_t* __restrict__ indptr_t,
    const int32_t* __restrict__ indices_t, const int32_t* __restrict__ eid_t,
    const float* __restrict__ pseudo, const float* __restrict__ pseudo_t /* nullable: pseudo in this walk's order */,
    const float* __restrict__ mu, const float* __restrict__ inv_sigma,
    const float* __restrict__ gout, PsParams pm, float* __restrict__ dhk) {
  constexpr int GPB = kPsBlock / L;
  __shared__ float coop_buf[GPB * L * 4 * kPsK];
  const int li = threadIdx.x & (L - 1);
  const int grp = threadIdx.x / L;
  int64_t r;
  int gi, ngrp;
  RowRange rr;
  if (!pick_row<GPB>(rl, grp, rr, r, gi, ngrp)) return;
  const int K = pm.K, R = pm.R, F = pm.F, KF = K * F;
  const float inv_k = 1.f / (float)K;
  const PsKernels<> pk = load_kernels(mu, inv_sigma, K, R);
  const int32_t u = order_t[r];
  const int32_t beg = indptr_t[u], end = indptr_t[u + 1];
  const bool col_ok = 4 * li < F;
  float4 acc[kPsK];
#pragma unroll
  for (int k = 0; k < kPsK; ++k) acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int32_t p = beg + gi; p < end; p += ngrp) {
    const int32_t v = indices_t[p];
    float m[kPsR];
    if (pseudo_t != nullptr) load_pseudo(pseudo_t, p, R, m);
    else load_pseudo(pseudo, eid_t[p], R, m);
    if (col_ok) {
      const float4 g4 = ld4(gout + (int64_t)v * F + 4 * li);
#pragma unroll
      for (int k = 0; k < kPsK; ++k)
        if (k < K) fma4(acc[k], gauss_k(pk, k, m) * inv_k, g4);
    }
  }
  if (rr.coop) {
    float vv[4 * kPsK];
#pragma unroll
    for (int k = 0; k < kPsK; ++k) pack4(vv + 4 * k, acc[k]);
    coop_sum<L, 4 * kPsK, GPB>(coop_buf, vv, grp, li);
    if (grp != 0) return;
#pragma unroll
    for (int k = 0; k < kPsK; ++k) acc[k] = unpack4(vv + 4 * k);
  }
  if (col_ok) {
#pragma unroll
    for (int k = 0; k < kPsK; ++k)
      if (k < K) st4(dhk + (int64_t)u * KF + k * F + 4 * li, acc[k]);
  }
}

// ---- narrow rows (K * fout <= 64 floats): chunks of edges, gathered rows in flight ------------
// With 16 hidden features (the paper's MoNet settings) a projected row hk[u] is 128-192 bytes.  The
// kernels above then spend their time on the per-edge chain index -> row -> arithmetic, taken one
// edge at a time (measured at Reddit scale with every gather served by the L2: forward 1.4 of 1.6 ms,
// so the fabric behind the L2s is not what bounds them).  Here a group of G lanes owns the row and
// one float4 of hk[u, :, :] per lane (lane li: kernel li / (F/4), columns 4 (li % (F/4))), and an edge
// set is walked in chunks of G edges in two phases, as in the attention kernels:
//   chunk phase: lane li takes edge li of the chunk: index, pseudo-coordinates, the K Gaussian
//                weights; index and weights are parked in LDS;
//   row phase:   every lane reads them back (broadcast reads) and has 8 row loads in flight.
// LDS traffic of a group stays inside its wavefront.
constexpr int kNrU = 8;  // gathered rows in flight per lane

// PROJ variants: the pseudo-coordinates are not read from an [E, r] array but made on the spot from the
// per-vertex scalar at the two ends of the edge, m[d] = tanh(P[d,0] c[u] + P[d,1] c[v] + pb[d]) (the
// paper's MoNet models project the degree pair this way): one more scalar gather per edge, no
// per-edge tensor at all.
struct ProjArgs {
  const float* c;   // [n]
  const float* P;   // [r, 2]
  const float* pb;  // [r]
};
template <int RT>
struct ProjRegs {
  float p0[RT], p1[RT], b[RT];
};
template <int RT>
__device__ __forceinline__ ProjRegs<RT> load_proj(const ProjArgs& a, int R) {
  ProjRegs<RT> q;
#pragma unroll
  for (int d = 0; d < RT; ++d) {
    const bool ok = d < R;
    q.p0[d] = ok ? a.P[2 * d] : 0.f;
    q.p1[d] = ok ? a.P[2 * d + 1] : 0.f;
    q.b[d] = ok ? a.pb[d] : 0.f;
  }
  return q;
}
template <int RT>
__device__ __forceinline__ void project(const ProjRegs<RT>& q, int R, float cu, float cv, float (&m)[RT]) {
#pragma unroll
  for (int d = 0; d < RT; ++d) m[d] = d < R ? tanhf(fmaf(q.p0[d], cu, fmaf(q.p1[d], cv, q.b[d]))) : 0.f;
}
constexpr int kPsValsProj = kPsVals + 3 * kPsR;  // + (gP[d,0], gP[d,1], gpb[d]) per dimension

// U values side by side in LDS, up to four at a time
template <int U, typename T>
struct alignas(sizeof(T) * (U < 4 ? U : 4)) LdsRun {
  T x[U < 4 ? U : 4];
};
template <int U, typename T>
__device__ __forceinline__ void read_run(const T* p, T (&v)[U]) {
  constexpr int B = U < 4 ? U : 4;
#pragma unroll
  for (int q = 0; q < U; q += B) {
    const auto run = *reinterpret_cast<const LdsRun<U, T>*>(p + q);
#pragma unroll
    for (int t = 0; t < B; ++t) v[q + t] = run.x[t];
  }
}
template <int U, typename T>
__device__ __forceinline__ void write_run(T* p, const T (&v)[U]) {
  constexpr int B = U < 4 ? U : 4;
#pragma unroll
  for (int q = 0; q < U; q += B) {
    LdsRun<U, T> run;
#pragma unroll
    for (int t = 0; t < B; ++t) run.x[t] = v[q + t];
    *reinterpret_cast<LdsRun<U, T>*>(p + q) = run;
  }
}

// Gathered rows of a table of n rows.  Up to 2 GB they come through a buffer resource, which reads zeros and no memory past its end:
// that is where edges past the row's end point (kPastTable), so a chunk's loads are issued four at a time without a branch to each.
// A branch to each -> this, us: forward, 200 000 vertices, 4 10^6 edges, K = 2, 16 columns, power law 86 -> 76, 13 000 x 200, even 40 -> 32,
// 230 000 x 9, K = 3, 12 columns 81 -> 79, 230 000 x 10, K = 2, 8 columns, even 55 -> 55; backward 113 -> 96 (the first of these), 75 -> 72 (the third), 60 000
// vertices, 1.5 10^7 edges, K = R = 3 277 -> 231.  By twos: 79, 36, 88, 55; 103, 73, 245.
constexpr uint32_t kPastTable = 0x80000000u;
__host__ __device__ __forceinline__ bool narrow_table(int64_t n, int row_floats) {
  return n < (1 << 24) && n * row_floats * 4 <= (int64_t)kPastTable;
}
__device__ __forceinline__ uint32_t row_offset(bool narrow, int32_t v, bool ok, int row_floats) {
  return !ok ? kPastTable : narrow ? __umul24((uint32_t)v, 4u * row_floats) : (uint32_t)v;
}
template <int U, typename Resource>
__device__ __forceinline__ void gather_rows(bool narrow, Resource table, const float* base, int row_floats,
                                            const uint32_t (&off)[U], uint32_t lane_off, int cnt, float4 (&rowv)[U]) {
#pragma unroll
  for (int t4 = 0; t4 < U; t4 += 4) {
    if (t4 != 0 && t4 >= cnt) break;
    if (narrow) {  // uniform
#pragma unroll
      for (int t = t4; t < t4 + 4 && t < U; ++t)
        rowv[t] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(table, off[t] + lane_off, 0, 0));
    } else {
#pragma unroll
      for (int t = t4; t < t4 + 4 && t < U; ++t) {
        rowv[t] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (off[t] != kPastTable) rowv[t] = ld4(base + (int64_t)off[t] * row_floats + lane_off / 4);
      }
    }
  }
}
// the gathered rows of a chunk's edges from t0 on, `cnt` of them at most: what is asked for by fours is used by fours
template <int U, typename Fn>
__device__ __forceinline__ void each_row(int cnt, Fn fn) {
#pragma unroll
  for (int t4 = 0; t4 < U; t4 += 4) {
    if (t4 != 0 && t4 >= cnt) break;
#pragma unroll
    for (int t = t4; t < t4 + 4 && t < U; ++t) fn(t);
  }
}
__device__ __forceinline__ auto table_resource(const float* p, int64_t n, int row_floats) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (uint32_t)(n * row_floats * 4), 0x00020000);
}

// forward: out[v, f] = (1/K) sum_e sum_k w_k(e) hk[u, k, f]; the sum over k is taken last, across lanes
// W: wavefronts per SIMD that it leaves room for, see launch_fwd_nr
template <int G, bool PROJ, int KT, int RT, int U, int W>
__global__ __launch_bounds__(kPsBlock, W) void k_gmmp_fwd_nr(
    RowLaunch rl, const int4* __restrict__ rows, const int32_t* __restrict__ indices, const float* __restrict__ hk, const float* __restrict__ pseudo,
    ProjArgs pa, const float* __restrict__ mu, const float* __restrict__ inv_sigma, PsParams pm,
    float* __restrict__ out) {
  constexpr int GPB = kPsBlock / G;
  constexpr int GS = G + KT * G;  // indices | weights [KT][G]
  __shared__ __align__(16) float lds[GPB * GS];
  __shared__ float coop_buf[GPB * G * 4];
  const int lane = threadIdx.x & 63;
  const int li = threadIdx.x & (G - 1);
  const int grp = threadIdx.x / G;
  int64_t r;
  int gi, ngrp;
  RowRange rr;
  if (!pick_row<GPB>(rl, grp, rr, r, gi, ngrp)) return;
  const int K = pm.K, R = pm.R, F = pm.F, KF = K * F, F4 = F / 4;
  const float inv_k = 1.f / (float)K;
  const PsKernels<KT, RT> pk = load_kernels<KT, RT>(mu, inv_sigma, K, R);
  const int4 row = rows[r];
  const int32_t v = row.x;
  const uint32_t beg = row.y, end = row.z;  // unsigned: positions past 2^31 - 1 are past every row's end
  ProjRegs<RT> pq;
  float cv = 0.f;
  if (PROJ) {
    pq = load_proj<RT>(pa, R);
    cv = pa.c[v];
  }
  const bool col_ok = li < K * F4;
  const int myk = col_ok ? li / F4 : 0;
  uint32_t* l_off = reinterpret_cast<uint32_t*>(lds + grp * GS);
  float* l_w = lds + grp * GS + G;
  // four kernels of four coordinates are bound by the vector units, where a branch to each row between two kinds of loads shows: forward,
  // 100 000 vertices, 60 even edges, 8 columns 102 -> 91, 12 156 -> 143 (one row in flight)
  constexpr bool kPlain = PROJ && U < kNrU && KT * RT >= 16;
  const bool narrow = !kPlain && pm.wide == 0 && narrow_table(rl.n_rows, KF);
  const auto table = table_resource(hk, rl.n_rows, KF);
  const uint32_t lane_off = 16u * li;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), part = acc;
  int folded = 0;
  // The sources travel two chunks ahead, their scalars one; the rows of a chunk are asked for before its weights are made.
  const uint32_t step = ngrp * G;
  auto source = [&](uint32_t e) { return e < end ? indices[e] : 0; };
  uint32_t e0 = beg + gi * G;
  int32_t u = source(e0 + li), u1 = source(e0 + step + li);
  float cu = PROJ ? pa.c[u] : 0.f;
  for (; e0 < end; e0 += step) {
    const bool e_ok = e0 + li < end;
    const int cnt = min((uint32_t)G, end - e0);
    wave_lds_fence();  // the previous chunk's reads are done
    l_off[li] = row_offset(narrow, u, e_ok, KF);
    wave_lds_fence();
    float m[RT];
    if (!PROJ) {
#pragma unroll
      for (int d = 0; d < RT; ++d) m[d] = 0.f;
      if (e_ok) load_pseudo(pseudo, e0 + li, R, m);
    }
    const float c_here = cu;
    u = u1;
    u1 = source(e0 + 2 * step + li);
    if (PROJ) cu = pa.c[u];
    float4 rowv[U];
    auto fetch = [&](int t0) {
      uint32_t off[U];
      read_run(l_off + t0, off);
      if (col_ok) gather_rows(narrow, table, hk, KF, off, lane_off, cnt - t0, rowv);
    };
    fetch(0);
    if (PROJ) project(pq, R, c_here, cv, m);
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      const float w = gauss_k(pk, k, m) * inv_k;
      l_w[k * G + li] = e_ok ? w : 0.f;
    }
    wave_lds_fence();
#pragma unroll
    for (int t0 = 0; t0 < G; t0 += U) {
      if (t0 < cnt) {
        if (t0 > 0) fetch(t0);
        float wv[U];
        read_run(l_w + myk * G + t0, wv);
        if (col_ok) each_row<U>(cnt - t0, [&](int t) { fma4(part, wv[t], rowv[t]); });
      }
    }
    folded += G;
    if (folded >= 32) {  // two-level summation keeps long rows accurate
      add4(acc, part);
      part = make_float4(0.f, 0.f, 0.f, 0.f);
      folded = 0;
    }
  }
  add4(acc, part);
  // kernels 1 .. K-1 sit F/4 lanes further on: add them in order
  float4 tot = acc;
  const int base = lane & ~(G - 1);
  for (int k = 1; k < K; ++k) {
    const int srcl = base + ((li + k * F4) & (G - 1));
    tot.x += __shfl(acc.x, srcl, 64);
    tot.y += __shfl(acc.y, srcl, 64);
    tot.z += __shfl(acc.z, srcl, 64);
    tot.w += __shfl(acc.w, srcl, 64);
  }
  if (rr.coop) {
    float vv[4];
    pack4(vv, tot);
    coop_sum<G, 4, GPB>(coop_buf, vv, grp, li);
    if (grp != 0) return;
    tot = unpack4(vv);
  }
  if (li < F4) st4(out + (int64_t)v * F + 4 * li, tot);
}

__global__ void k_monet_zero_clock(int32_t* __restrict__ p) { p[threadIdx.x] = 0; }

// ---- forward past the L2s: all column blocks in one persistent launch, the sums in LDS ----------------
// k_gmmp_fwd_nr gathers a row of hk and a scalar per edge from anywhere, and the rows that miss the L2s come at the rate of the fabric
// behind them.  Here one 1024-thread workgroup to a CU keeps the sums of its rows in LDS, F floats each, and takes all of them through
// the plan's column blocks one after the other; the block's rows of hk are in the L2 then, and its scalars in LDS: one line to an edge.
// Rows are dealt to the workgroups one position of the degree order at a time, in alternating direction, and inside a workgroup
// the groups draw them from a counter, longest first.  A row with more than its share of edges would be what a workgroup waits for
// in every block, so it is cut into 2, 4, ... parts, drawn like rows; the parts' sums are added in order at the end.
// Bound by the instructions of the vector units, some 150 to a wavefront's 64 edges with tanhf a third of them, and by segments that
// are shorter than a chunk.  MoNet forward, us, k_gmmp_fwd_nr -> here: 232 965 vertices, 1.12 10^8 edges, K = 2, 16 columns
// 1410 -> 970 (a branch to each gather instead of the buffer loads: 1000; workgroups that meet after every block 1015, every
// fourth 975); 2 x 32, R = 2 2380 -> 1200; 100 000 vertices, 3 10^7 edges, K = 3 410 -> 250; uniform, 230 000 x 320, K = 2 973 -> 639,
// 100 000 x 200, K = 3 360 -> 290.
constexpr int kMonetThreads = 1024;
constexpr int kMonetTabPerThread = 12;
template <int G, int KT>
constexpr int kMonetGroupInts = (kMonetThreads / G) * (1 + KT) * G;  // idx, weights of all groups
// a slot: sum, (beg, end) of two blocks, row, c of the row
constexpr int monet_slot_ints(int F) { return F + 4 + 1 + 1; }

template <int G, bool PROJ, int KT, int RT>
__global__ __launch_bounds__(kMonetThreads) void k_monet_res(
    int32_t n_rows, const int32_t* __restrict__ order, const int2* __restrict__ bseg /* [nblk][n_rows] */,
    const int32_t* __restrict__ indptr, const int32_t* __restrict__ cols /* PROJ: block by block, else row by row */,
    const float* __restrict__ hk, const float* __restrict__ pseudo, ProjArgs pa, const float* __restrict__ mu, const float* __restrict__ inv_sigma, PsParams pm,
    int32_t block_cols, int nblk, int cap /* slots the LDS holds */, RowParts cut, int32_t* __restrict__ clock, int spin_limit,
    int sync_every, float* __restrict__ out) {
  constexpr int GPB = kMonetThreads / G, U = 8;
  extern __shared__ __align__(16) int lds_mr[];
  const int lane = threadIdx.x & 63, li = threadIdx.x & (G - 1), grp = threadIdx.x / G;
  const int64_t nwg = gridDim.x, wg = blockIdx.x;
  const int K = pm.K, R = pm.R, F = pm.F, KF = K * F, F4 = F / 4;
  const float inv_k = 1.f / (float)K;
  const PsKernels<KT, RT> pk = load_kernels<KT, RT>(mu, inv_sigma, K, R);
  const ProjRegs<RT> pq = PROJ ? load_proj<RT>(pa, R) : ProjRegs<RT>{};
  const bool col_ok = li < K * F4;
  const int myk = col_ok ? li / F4 : 0;
  const uint32_t lane_off = 16u * li;
  const auto table = table_resource(hk, n_rows, KF);
  float4* l_sum = reinterpret_cast<float4*>(lds_mr);        // [cap][F4]
  uint32_t* l_off = reinterpret_cast<uint32_t*>(lds_mr + cap * F + grp * (1 + KT) * G);  // [G], weights [KT][G]
  float* l_w = reinterpret_cast<float*>(l_off + G);
  int2* l_seg = reinterpret_cast<int2*>(lds_mr + cap * F + kMonetGroupInts<G, KT>);  // [2][cap]
  int* l_row = reinterpret_cast<int*>(l_seg + 2 * cap);     // [cap]
  float* l_cv = reinterpret_cast<float*>(l_row + cap);      // [cap]
  int* l_cnt = reinterpret_cast<int*>(l_cv + cap);          // [2]
  float* l_tab = reinterpret_cast<float*>(l_cnt + 2);       // [block_cols]

  float tab[kMonetTabPerThread] = {};
  auto fetch_table = [&](int p) {
#pragma unroll
    for (int i = 0; i < (PROJ ? kMonetTabPerThread : 0); ++i) {
      const int c = i * kMonetThreads + threadIdx.x;
      const int64_t u = (int64_t)p * block_cols + c;
      if (c < block_cols && u < n_rows) tab[i] = pa.c[u];
    }
  };
  auto store_table = [&]() {
#pragma unroll
    for (int i = 0; i < (PROJ ? kMonetTabPerThread : 0); ++i) {
      const int c = i * kMonetThreads + threadIdx.x;
      if (c < block_cols) l_tab[c] = tab[i];
    }
  };
  fetch_table(0);
  store_table();

  const int rows_here = (int)((n_rows + nwg - 1) / nwg);
  // workgroups go to the XCDs round-robin: those with the same id mod 8 share an L2
  PhaseClock pc{clock ? clock + (blockIdx.x % kXcds) * kClockStride : nullptr, (int)(gridDim.x / kXcds), spin_limit,
                false, sync_every > 0 ? sync_every : nblk};
  struct Item {
    int32_t beg, end, c_first;
  };

  int phase = 0;
  for (int j0 = 0, j1; j0 < rows_here; j0 = j1) {
    // rows j0 .. j1 - 1: as many as there are slots for (a row's parts fit: see the launch)
    const int s0 = slots_before(cut, j0);
    j1 = rows_that_fit(cut, j0, rows_here, cap);
    const int nslots = slots_before(cut, j1) - s0;
    // thread q: slot q
    int64_t pos = -1;
    int part = 0, logp = 0;
    int32_t row = -1, next = 0;  // the row, and where its edges of the next block begin
    if ((int)threadIdx.x < nslots) {
      const int lo = row_of_slot(cut, j0, j1, threadIdx.x);
      part = (int)threadIdx.x - (slots_before(cut, lo) - s0);
      logp = log_parts(cut, lo);
      const int64_t r = (int64_t)lo * nwg + ((lo & 1) ? nwg - 1 - wg : wg);
      if (r < n_rows) {
        pos = r;
        row = order[r];
        if (!PROJ) next = indptr[row];
      }
    }
    // This thread's piece of its row's segment of block p, asked for block by block.  Coordinates of edges are in the order of the rows, which
    // is walked then; the rows' edges are in the order of the blocks.  (With projected ones, too, 2750 us a training pass, see above, not 2695.)
    auto bounds = [&](int p) {
      if (pos < 0) return make_int2(0, 0);
      const int2 sg = bseg[(int64_t)p * n_rows + pos];
      const int64_t len = sg.y - sg.x;
      const int beg = PROJ ? sg.x : next;
      next += (int)len;
      return make_int2(beg + (int)(len * part >> logp), beg + (int)(len * (part + 1) >> logp));
    };
    if ((int)threadIdx.x < nslots) {
      l_row[threadIdx.x] = part == 0 ? row : -2;  // -2: a further part of the row before
      if (PROJ) l_cv[threadIdx.x] = row >= 0 ? pa.c[row] : 0.f;
      l_seg[threadIdx.x] = bounds(0);
    }
    for (int i = threadIdx.x; i < nslots * F4; i += kMonetThreads) l_sum[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (threadIdx.x == 0) l_cnt[0] = 0;
    __syncthreads();  // the tables are in place

    auto grab = [&](int p) {  // a group's next slot of block p, from that block's counter
      int q = 0;
      if (li == 0) q = atomicAdd(l_cnt + (p & 1), 1);
      return __shfl(q, lane & ~(G - 1), 64);
    };
    auto fetch = [&](int p, int q) {
      Item it{0, 0, p * block_cols};
      if (q >= nslots) return it;
      const int2 sg = l_seg[(p & 1) * cap + q];
      it.beg = sg.x;
      it.end = sg.y;
      if (it.beg + li < it.end) it.c_first = cols[it.beg + li];
      return it;
    };
    int q = grab(0);
    Item cur = fetch(0, q);
    for (int p = 0; p < nblk; ++p) {
      const int32_t col_begin = p * block_cols;
      const bool last = p + 1 == nblk;
      // the next block's bounds and scalars travel while this one is worked on
      int2 seg_next = make_int2(0, 0);
      if (!last) seg_next = bounds(p + 1);
      if (threadIdx.x == 0) l_cnt[(p + 1) & 1] = 0;
      fetch_table(last ? 0 : p + 1);

      while (q < nslots) {
        const int qn = grab(p);
        const Item nxt = fetch(p, qn);
        if (cur.beg < cur.end) {
          const float cv = PROJ ? l_cv[q] : 0.f;
          float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), part4 = acc;
          int folded = 0;
          int32_t c_next = cur.c_first;
          for (int32_t e0 = cur.beg; e0 < cur.end; e0 += G) {
            const bool e_ok = e0 + li < cur.end;
            const int32_t c = e_ok ? c_next : col_begin;
            if (e0 + G + li < cur.end) c_next = cols[e0 + G + li];
            wave_lds_fence();  // the previous chunk's reads are done
            l_off[li] = e_ok ? __umul24((uint32_t)c, 4u * KF) : kPastTable;
            wave_lds_fence();
            float m[RT];
            if (!PROJ) {
#pragma unroll
              for (int d = 0; d < RT; ++d) m[d] = 0.f;
              if (e_ok) load_pseudo(pseudo, e0 + li, R, m);
            }
            float4 rowv[U];
            const int cnt = cur.end - e0;
            auto rows_of = [&](int t0) {
              uint32_t off[U];
              read_run(l_off + t0, off);
              if (col_ok) gather_rows(true, table, hk, KF, off, lane_off, cnt - t0, rowv);
            };
            rows_of(0);
            if (PROJ) project(pq, R, l_tab[c - col_begin], cv, m);
#pragma unroll
            for (int k = 0; k < KT; ++k) {
              const float w = gauss_k(pk, k, m) * inv_k;
              l_w[k * G + li] = e_ok ? w : 0.f;
            }
            wave_lds_fence();
#pragma unroll
            for (int t0 = 0; t0 < G; t0 += U) {
              if (t0 < cnt) {
                if (t0 > 0) rows_of(t0);
                float wv[U];
                read_run(l_w + myk * G + t0, wv);
                if (col_ok) each_row<U>(cnt - t0, [&](int t) { fma4(part4, wv[t], rowv[t]); });
              }
            }
            folded += G;
            if (folded >= 32) {  // two-level summation, as in k_gmmp_fwd_nr
              add4(acc, part4);
              part4 = make_float4(0.f, 0.f, 0.f, 0.f);
              folded = 0;
            }
          }
          add4(acc, part4);
          // kernels 1 .. K-1 sit F/4 lanes further on: add them in order
          float4 tot = acc;
          const int base = lane & ~(G - 1);
          for (int k = 1; k < K; ++k) {
            const int srcl = base + ((li + k * F4) & (G - 1));
            tot.x += __shfl(acc.x, srcl, 64);
            tot.y += __shfl(acc.y, srcl, 64);
            tot.z += __shfl(acc.z, srcl, 64);
            tot.w += __shfl(acc.w, srcl, 64);
          }
          if (li < F4) {
            add4(tot, l_sum[q * F4 + li]);
            l_sum[q * F4 + li] = tot;
          }
        }
        q = qn;
        cur = nxt;
      }
      if ((int)threadIdx.x < nslots) l_seg[((p + 1) & 1) * cap + threadIdx.x] = seg_next;
      __syncthreads();  // the workgroup is done with this block; the next one's bounds are in LDS
      store_table();
      if (!last) {      // first slot of the next block: its loads travel during the wait below
        q = grab(p + 1);
        cur = fetch(p + 1, q);
      }
      phase_step_done(pc, phase++);
      __syncthreads();  // every workgroup of the XCD is done with this block (or the wait ran out)
    }
    // the rows' sums, parts added in order
    for (int s = grp; s < nslots; s += GPB) {
      const int32_t row = l_row[s];
      if (row < 0 || li >= F4) continue;
      float4 acc = l_sum[s * F4 + li];
      for (int t = s + 1; t < nslots && l_row[t] == -2; ++t) add4(acc, l_sum[t * F4 + li]);
      st4_stream(out + (int64_t)row * F + 4 * li, acc);
    }
    __syncthreads();  // the tables are free for the next rows
  }
}


// destination side of backward, the coordinates' gradient alone (the walk below has the rest): the row phase leaves every
// lane's part of <gout[v], hk[u, k, :]> in LDS, and the lane that owns the edge adds the F/4 parts of each kernel in
// lane order; loads ahead as in k_gmmp_fwd_nr.
template <int G, int KT, int RT, int U>
__global__ __launch_bounds__(kPsBlock) void k_gmmp_bwd_dst_nr(
    RowLaunch rl, const int4* __restrict__ rows, const int32_t* __restrict__ indices, const float* __restrict__ hk,
    const float* __restrict__ pseudo, const float* __restrict__ mu, const float* __restrict__ inv_sigma,
    const float* __restrict__ gout, PsParams pm, float* __restrict__ gpseudo) {
  constexpr int GPB = kPsBlock / G;
  constexpr int GS = G + G * G;  // indices | partial dot products [column lane][edge]
  __shared__ __align__(16) float lds[GPB * GS];
  const int li = threadIdx.x & (G - 1);
  const int grp = threadIdx.x / G;
  int64_t r;
  int gi, ngrp;
  RowRange rr;
  if (!pick_row<GPB>(rl, grp, rr, r, gi, ngrp)) return;
  const int K = pm.K, R = pm.R, F = pm.F, KF = K * F, F4 = F / 4;
  const float inv_k = 1.f / (float)K;
  const PsKernels<KT, RT> pk = load_kernels<KT, RT>(mu, inv_sigma, K, R);
  const int4 row = rows[r];
  const int32_t v = row.x;
  const uint32_t beg = row.y, end = row.z;  // unsigned, as in k_gmmp_fwd_nr
  const bool col_ok = li < K * F4;
  const int f4 = col_ok ? li % F4 : 0;
  const float4 g4 = col_ok ? ld4(gout + (int64_t)v * F + 4 * f4) : make_float4(0.f, 0.f, 0.f, 0.f);
  uint32_t* l_off = reinterpret_cast<uint32_t*>(lds + grp * GS);
  float* l_d = lds + grp * GS + G;
  const bool narrow = pm.wide == 0 && narrow_table(rl.n_rows, KF);
  const auto table = table_resource(hk, rl.n_rows, KF);
  const uint32_t lane_off = 16u * li;
  const uint32_t step = ngrp * G;
  auto source = [&](uint32_t e) { return e < end ? indices[e] : 0; };
  uint32_t e0 = beg + gi * G;
  int32_t u = source(e0 + li), u1 = source(e0 + step + li);
  for (; e0 < end; e0 += step) {
    const bool e_ok = e0 + li < end;
    const int cnt = min((uint32_t)G, end - e0);
    wave_lds_fence();  // the previous chunk's reads are done
    l_off[li] = row_offset(narrow, u, e_ok, KF);
    wave_lds_fence();
    float m[RT];
#pragma unroll
    for (int d = 0; d < RT; ++d) m[d] = 0.f;
    if (e_ok) load_pseudo(pseudo, e0 + li, R, m);
    u = u1;
    u1 = source(e0 + 2 * step + li);
    float4 rowv[U];
    auto fetch = [&](int t0) {
      uint32_t off[U];
      read_run(l_off + t0, off);
      if (col_ok) gather_rows(narrow, table, hk, KF, off, lane_off, cnt - t0, rowv);
    };
    fetch(0);
#pragma unroll
    for (int t0 = 0; t0 < G; t0 += U) {
      if (t0 < cnt) {
        if (t0 > 0) fetch(t0);
        float dv[U] = {};
        if (col_ok) each_row<U>(cnt - t0, [&](int t) { dv[t] = dot4(g4, rowv[t]); });  // past the row's end: not looked at
        write_run(l_d + li * G + t0, dv);
      }
    }
    wave_lds_fence();
    if (e_ok) {
      float gm[RT];
#pragma unroll
      for (int d = 0; d < RT; ++d) gm[d] = 0.f;
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        if (k >= K) continue;
        float dot = 0.f;
        for (int j = 0; j < F4; ++j) dot += l_d[(k * F4 + j) * G + li];
        const float dlog = dot * inv_k * gauss_k(pk, k, m);  // dw_k(e) w_k(e)
#pragma unroll
        for (int d = 0; d < RT; ++d) {
          const float is = pk.is[k][d];
          const float t = dlog * (m[d] - pk.mu[k][d]) * is;  // padded dimensions: is = 0
          gm[d] = fmaf(-t, is, gm[d]);
        }
      }
#pragma unroll
      for (int d = 0; d < RT; ++d)
        if (d < R) gpseudo[(int64_t)(e0 + li) * R + d] = gm[d];
    }
  }
}

// Backward, both sides in one walk over the out-edges.  A row owns hk[u] and dhk[u] and gathers gout[v], with which
// a lane adds w_k(e) gout[v] to dhk and, through LDS, hands its part of <gout[v], hk[u, k, :]> to the lane that
// owns the edge; that lane has the pseudo-coordinates and weights already and sums the parameters' gradients.
// Apart, the destination side gathered the K times wider hk[u] and both sides evaluated every tanh and exp.
// 232 965 vertices, 1.12 10^8 edges, K = 2, R = 1, 16 columns, us: 1470 + 1240 -> 1320 (1860 compiled for the most kernels and
// dimensions, as the forward kernel is, which the gathers of hk[u] bound: 1425, and 1478 compiled for K = 2, R = 1).
// Wavefronts per SIMD that k_gmmp_bwd_nr leaves room for: a few registers less than it would take (100 000 vertices, 2 10^6 edges, K = 3,
// R = 2 73 us with what it would take, 60 so).  Three where four would keep up to 36 registers of the sums in scratch memory: 100 000, 2 10^6,
// 8 columns, power law | even, unbounded, room for four, three: K = R = 4 268, 440, 233 | 91, 126, 86; K = 4, R = 3 256, 266, 216 |
// 79, 83, 81; K = 3, R = 4 250, 253, 213 | 86, 83, 81.
template <int KT, int RT>
constexpr int kNrMinWaves = KT <= 3 && RT == 1 ? 5 : KT * RT < 12 ? 4 : 3;
template <int G, bool PROJ, int KT, int RT>
__global__ __launch_bounds__(kPsBlock, (kNrMinWaves<KT, RT>)) void k_gmmp_bwd_nr(
    RowLaunch rl, const int4* __restrict__ rows_t, const int32_t* __restrict__ indices_t, const int32_t* __restrict__ eid_t, const float* __restrict__ hk,
    const float* __restrict__ pseudo, const float* __restrict__ pseudo_t /* nullable: pseudo in this walk's order */,
    ProjArgs pa, const float* __restrict__ mu, const float* __restrict__ inv_sigma, const float* __restrict__ gout,
    PsParams pm, float* __restrict__ dhk, double* __restrict__ partial, float* __restrict__ gpseudo /* nullable */) {
  constexpr int NVALS = 2 * KT * RT + (PROJ ? 3 * RT : 0);
  constexpr int GPB = kPsBlock / G;
  constexpr int GS = G + KT * G + G * G;  // indices | weights [KT][G] | partial dot products [column lane][edge]
  __shared__ __align__(16) float lds[GPB * GS];
  __shared__ float coop_buf[GPB * G * 4];
  __shared__ double blk[GPB][NVALS];
  const int li = threadIdx.x & (G - 1);
  const int grp = threadIdx.x / G;
  int64_t r;
  int gi, ngrp;
  RowRange rr;
  const bool active = pick_row<GPB>(rl, grp, rr, r, gi, ngrp);
  const int K = pm.K, R = pm.R, F = pm.F, KF = K * F, F4 = F / 4;
  const float inv_k = 1.f / (float)K;
  float sums[NVALS];  // over the edges this lane owned
#pragma unroll
  for (int i = 0; i < NVALS; ++i) sums[i] = 0.f;
  if (active) {
    const PsKernels<KT, RT> pk = load_kernels<KT, RT>(mu, inv_sigma, K, R);
    const int4 row = rows_t[r];
    const int32_t u = row.x;
    const uint32_t beg = row.y, end = row.z;  // unsigned, as in k_gmmp_fwd_nr
    ProjRegs<RT> pq;
    float cu = 0.f;
    if (PROJ) {
      pq = load_proj<RT>(pa, R);
      cu = pa.c[u];
    }
    const bool col_ok = li < K * F4;
    const int myk = col_ok ? li / F4 : 0, f4 = col_ok ? li % F4 : 0;
    const float4 h4 = col_ok ? ld4(hk + (int64_t)u * KF + 4 * li) : make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t* l_off = reinterpret_cast<uint32_t*>(lds + grp * GS);
    float* l_w = lds + grp * GS + G;
    float* l_d = l_w + KT * G;
    const bool narrow = pm.wide == 0 && narrow_table(rl.n_rows, F);
    const auto table = table_resource(gout, rl.n_rows, F);
    const uint32_t lane_off = 16u * f4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), part = acc;
    int folded = 0;
    // loads ahead as in k_gmmp_fwd_nr
    const uint32_t step = ngrp * G;
    auto target = [&](uint32_t p) { return p < end ? indices_t[p] : 0; };
    uint32_t p0 = beg + gi * G;
    int32_t v = target(p0 + li), v1 = target(p0 + step + li);
    float cv_next = PROJ ? pa.c[v] : 0.f;
    for (; p0 < end; p0 += step) {
      const bool e_ok = p0 + li < end;
      const int cnt = min((uint32_t)G, end - p0);
      wave_lds_fence();  // the previous chunk's reads are done
      l_off[li] = row_offset(narrow, v, e_ok, F);
      wave_lds_fence();
      int32_t e = 0;
      float m[RT], w[KT];
      if (!PROJ) {
#pragma unroll
        for (int d = 0; d < RT; ++d) m[d] = 0.f;
        if (e_ok) {
          if (pseudo_t == nullptr || gpseudo != nullptr) e = eid_t[p0 + li];
          if (pseudo_t != nullptr) load_pseudo(pseudo_t, p0 + li, R, m);
          else load_pseudo(pseudo, e, R, m);
        }
      }
      const float cv = cv_next;
      v = v1;
      v1 = target(p0 + 2 * step + li);
      if (PROJ) cv_next = pa.c[v];
      float4 rowv[kNrU];
      auto fetch = [&](int t0) {
        uint32_t off[kNrU];
        read_run(l_off + t0, off);
        if (col_ok) gather_rows(narrow, table, gout, F, off, lane_off, cnt - t0, rowv);
      };
      fetch(0);
      if (PROJ) project(pq, R, cu, cv, m);
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        w[k] = gauss_k(pk, k, m) * inv_k;
        l_w[k * G + li] = w[k] = e_ok ? w[k] : 0.f;
      }
      wave_lds_fence();
#pragma unroll
      for (int t0 = 0; t0 < G; t0 += kNrU) {
        if (t0 < cnt) {
          if (t0 > 0) fetch(t0);
          float wv[kNrU], dv[kNrU] = {};
          read_run(l_w + myk * G + t0, wv);
          if (col_ok)
            each_row<kNrU>(cnt - t0, [&](int t) {
              fma4(part, wv[t], rowv[t]);
              dv[t] = dot4(h4, rowv[t]);  // past the row's end: not looked at
            });
          *reinterpret_cast<float4*>(l_d + li * G + t0) = make_float4(dv[0], dv[1], dv[2], dv[3]);
          *reinterpret_cast<float4*>(l_d + li * G + t0 + 4) = make_float4(dv[4], dv[5], dv[6], dv[7]);
        }
      }
      wave_lds_fence();
      if (e_ok) {
        float gm[RT];
#pragma unroll
        for (int d = 0; d < RT; ++d) gm[d] = 0.f;
#pragma unroll
        for (int k = 0; k < KT; ++k) {
          if (k >= K) continue;
          float dot = 0.f;
          for (int j = 0; j < F4; ++j) dot += l_d[(k * F4 + j) * G + li];
          const float dlog = dot * w[k];  // dw_k(e) w_k(e), 1 / K in the weight
#pragma unroll
          for (int d = 0; d < RT; ++d) {
            const float diff = m[d] - pk.mu[k][d];
            const float is = pk.is[k][d];
            const float t = dlog * diff * is;  // padded dimensions: is = 0
            sums[k * RT + d] = fmaf(t, is, sums[k * RT + d]);
            sums[KT * RT + k * RT + d] = fmaf(-t, diff, sums[KT * RT + k * RT + d]);
            gm[d] = fmaf(-t, is, gm[d]);
          }
        }
        if (PROJ) {
#pragma unroll
          for (int d = 0; d < RT; ++d) {
            const float dpre = gm[d] * (1.f - m[d] * m[d]);  // through the tanh; padded dimensions: gm = 0
            float* gp = sums + 2 * KT * RT + 3 * d;
            gp[0] = fmaf(dpre, cu, gp[0]);
            gp[1] = fmaf(dpre, cv, gp[1]);
            gp[2] += dpre;
          }
        } else if (gpseudo != nullptr) {
#pragma unroll
          for (int d = 0; d < RT; ++d)
            if (d < R) gpseudo[(int64_t)e * R + d] = gm[d];
        }
      }
      folded += G;
      if (folded >= 32) {  // two-level summation keeps long rows accurate
        add4(acc, part);
        part = make_float4(0.f, 0.f, 0.f, 0.f);
        folded = 0;
      }
    }
    add4(acc, part);
    if (rr.coop) {
      float vv[4];
      pack4(vv, acc);
      coop_sum<G, 4, GPB>(coop_buf, vv, grp, li);
      acc = unpack4(vv);
    }
    if (col_ok && (!rr.coop || grp == 0)) st4(dhk + (int64_t)u * KF + 4 * li, acc);
  }
  // The group's lanes are added in a fixed (butterfly) order, then the groups in order; what K and R leave out is 0.  From
  // here on in 64 bits: the sums over all edges cancel, the bias' gradient most (1.12 10^8 edges, four inputs, its worst
  // error 2.6e-5, with two kernels for the two sides 6.0e-6, now 1.6e-6; the time is unchanged).
#pragma unroll
  for (int i = 0; i < NVALS; ++i) {
    const double s = group_sum_wide<G>((double)sums[i]);
    if (li == 0) blk[grp][i] = s;
  }
  __syncthreads();
  if (threadIdx.x < NVALS) {
    double s = 0.;
    for (int g2 = 0; g2 < GPB; ++g2) s += blk[g2][threadIdx.x];
    partial[(int64_t)blockIdx.x * NVALS + threadIdx.x] = s;
  }
}

// The sums over the workgroups' partials [parts][nvals], nvals <= kPsValsProj, in two launches: ranges of kParamChunk parts,
// one workgroup each, then those ranges, by the one workgroup that also stores the gradients.  The order is fixed.
constexpr int kParamChunk = 256;

// thread c < nvals returns the sum of column c; the order does not depend on the columns there are
constexpr int kParamThreads = 1024;
__device__ __forceinline__ double sum_columns(int nvals, int parts, const double* __restrict__ partial) {
  constexpr int W = 64, SLOTS = kParamThreads / W;
  static_assert(kPsValsProj <= W, "one thread per column");
  __shared__ double sub[SLOTS][W];
  const int c = threadIdx.x % W, slot = threadIdx.x / W;
  double s = 0.;
  if (c < nvals) {
#pragma unroll 8
    for (int z = slot; z < parts; z += SLOTS) s += partial[(int64_t)z * nvals + c];
  }
  sub[slot][c] = s;
  __syncthreads();
  if (slot == 0) {
#pragma unroll
    for (int q = 1; q < SLOTS; ++q) s += sub[q][c];
  }
  return s;
}
__global__ __launch_bounds__(kParamThreads) void k_gmmp_param_rows(int nvals, int parts, const double* __restrict__ partial,
                                                                   double* __restrict__ rows) {
  const int z0 = blockIdx.x * kParamChunk;
  const double s = sum_columns(nvals, min(kParamChunk, parts - z0), partial + (int64_t)z0 * nvals);
  if (threadIdx.x < nvals) rows[(int64_t)blockIdx.x * nvals + threadIdx.x] = s;
}
// columns: gmu [kt][rt], ginv_sigma [kt][rt], then, where gP is not null, (gP[d,0], gP[d,1], gpb[d]) [rt]
__device__ __forceinline__ void store_param_total(int K, int R, int kt, int rt, int i, float s, float* gmu, float* gis, float* gP, float* gpb) {
  const int krt = kt * rt;
  if (i < 2 * krt) {
    float* g = i < krt ? gmu : gis;
    i = i < krt ? i : i - krt;
    const int k = i / rt, d = i - k * rt;
    if (k < K && d < R) g[k * R + d] = s;
  } else {
    i -= 2 * krt;
    const int d = i / 3, j = i - 3 * d;
    if (d >= R) return;
    if (j < 2) gP[2 * d + j] = s;
    else gpb[d] = s;
  }
}
// The workgroups but the first sum the parts of the product beside (count = 0: none), 256 threads to each of its blocks: a launch of its own
// is some 5 us, of memory latency like this one.
__global__ __launch_bounds__(kParamThreads) void k_gmmp_param_totals(int K, int R, int kt, int rt, int nrows,
                                                                const double* __restrict__ rows, float* __restrict__ gmu,
                                                                float* __restrict__ gis, float* __restrict__ gP /* nullable */,
                                                                float* __restrict__ gpb, PartialSum product, bool wide) {
  __shared__ float sub[kParamThreads / 256][8][32];
  if (blockIdx.x == 0) {
    const int nvals = 2 * kt * rt + (gP != nullptr ? 3 * rt : 0);
    const float s = (float)sum_columns(nvals, nrows, rows);
    if ((int)threadIdx.x < nvals) store_param_total(K, R, kt, rt, threadIdx.x, s, gmu, gis, gP, gpb);
    return;
  }
  const int quarter = threadIdx.x / 256, t = threadIdx.x % 256;
  const int64_t block = (int64_t)(blockIdx.x - 1) * (kParamThreads / 256) + quarter;
  if (wide) sum_partials_wide(product, block, 0, product.parts, t, sub[quarter]);
  else sum_partials_thin(product, block, t);
}

// ---- the projection that makes pseudo-coordinates from the degree pair ------------------------
// m[e,d] = tanh(P[d,0] c[u] + P[d,1] c[v] + pb[d]).  One wavefront per row of the walked list, lanes
// over its edges, four edges per lane in flight.  side 0: rows are destinations (CSR walk, the row's
// vertex is v); side 1: rows are sources (transposed list, the row's vertex is u) and the output is in
// that list's order.  What bounds a pass is the gather of c at the other end of every edge, one L1 line
// fill per edge (an edge-parallel version with perfectly even load took the same time).
__global__ void k_pseudo_proj_fwd(int32_t n, const int32_t* __restrict__ indptr,
                                  const int32_t* __restrict__ indices, const float* __restrict__ c, int R,
                                  const float* __restrict__ P, const float* __restrict__ pb, int side,
                                  float* __restrict__ pseudo) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (row >= n) return;
  const float c_row = c[row];
  const int32_t end = indptr[row + 1];
  for (int32_t e0 = indptr[row] + lane; e0 < end; e0 += 256) {
    float c_other[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) c_other[j] = e0 + 64 * j < end ? c[indices[e0 + 64 * j]] : 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (e0 + 64 * j >= end) continue;
      const float cu = side == 0 ? c_other[j] : c_row, cv = side == 0 ? c_row : c_other[j];
      for (int d = 0; d < R; ++d)
        pseudo[(int64_t)(e0 + 64 * j) * R + d] = tanhf(fmaf(P[2 * d], cu, fmaf(P[2 * d + 1], cv, pb[d])));
    }
  }
}

// partial[block][3 * kPsR]: (gP[d,0], gP[d,1], gpb[d]) for d < kPsR, summed over the block's rows.
// A wavefront takes every (number of wavefronts)-th row, so that the long rows of a power-law
// graph (they sit next to each other when vertices are numbered by weight) spread over the grid.
__global__ __launch_bounds__(kPsBlock) void k_pseudo_proj_bwd(
    int32_t n, const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
    const float* __restrict__ c, int R, const float* __restrict__ pseudo, const float* __restrict__ gpseudo,
    float* __restrict__ partial) {
  __shared__ float red[kPsBlock / 64][3 * kPsR];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float s[3 * kPsR];
#pragma unroll
  for (int i = 0; i < 3 * kPsR; ++i) s[i] = 0.f;
  const int64_t waves = (int64_t)gridDim.x * (kPsBlock / 64);
  for (int64_t v = (int64_t)blockIdx.x * (kPsBlock / 64) + w; v < n; v += waves) {
    const float cv = c[v];
    const int32_t end = indptr[v + 1];
    for (int32_t e0 = indptr[v] + lane; e0 < end; e0 += 128) {  // two edges per lane in flight
      const int32_t e1 = e0 + 64;
      const bool ok1 = e1 < end;
      const float cu0 = c[indices[e0]], cu1 = ok1 ? c[indices[e1]] : 0.f;
#pragma unroll
      for (int d = 0; d < kPsR; ++d) {
        if (d >= R) continue;
        const float m0 = pseudo[(int64_t)e0 * R + d], q0 = gpseudo[(int64_t)e0 * R + d];
        const float m1 = ok1 ? pseudo[(int64_t)e1 * R + d] : 0.f, q1 = ok1 ? gpseudo[(int64_t)e1 * R + d] : 0.f;
        const float dpre0 = q0 * (1.f - m0 * m0), dpre1 = q1 * (1.f - m1 * m1);
        s[3 * d] = fmaf(dpre1, cu1, fmaf(dpre0, cu0, s[3 * d]));
        s[3 * d + 1] = fmaf(dpre1, cv, fmaf(dpre0, cv, s[3 * d + 1]));
        s[3 * d + 2] += dpre0 + dpre1;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 3 * kPsR; ++i) {
    float t = s[i];
    for (int off = 1; off < 64; off <<= 1) t += __shfl_xor(t, off, 64);
    if (lane == 0) red[w][i] = t;
  }
  __syncthreads();
  if (threadIdx.x < 3 * kPsR) {
    float t = 0.f;
    for (int q = 0; q < kPsBlock / 64; ++q) t += red[q][threadIdx.x];
    partial[(int64_t)blockIdx.x * 3 * kPsR + threadIdx.x] = t;
  }
}

__global__ void k_pseudo_proj_split(int R, const float* __restrict__ totals, float* __restrict__ gP,
                                    float* __restrict__ gpb) {
  const int d = threadIdx.x;
  if (d >= R) return;
  gP[2 * d] = totals[3 * d];
  gP[2 * d + 1] = totals[3 * d + 1];
  gpb[d] = totals[3 * d + 2];
}

// ---- host side --------------------------------------------------------------------------
template <int L>
static unsigned ps_grid(const gnn_graph_t* g, int side, RowLaunch& rl) {
  constexpr int GPB = kPsBlock / L;
  const RowSplit sp = split_rows(g, side, 4, GPB);  // edges are taken one at a time: count 4 as a chunk
  rl = RowLaunch{sp.hub.end, g->n};
  return sp.hub_grid + sp.rest_grid;
}

static int ps_lanes(int fout) { return pick_group(fout).L; }  // fout <= 256: one float4 slot per lane

// Lanes per group of the chunked kernels for narrow rows, 0 where they do not apply: the K * fout / 4
// float4 slots of a projected row must fit 16 lanes.
static int nr_lanes(int K, int fout) {
  const int q = K * fout / 4;
  if (q > 16 || config_get(kCfgForceSimple)) return 0;
  return q <= 8 ? 8 : 16;
}
template <int G>
static unsigned nr_grid(const gnn_graph_t* g, int side, RowLaunch& rl) {
  constexpr int GPB = kPsBlock / G;
  // an ordinary row is walked by one group, G edges at a time with 8 gathers in flight; rows from 64
  // such chunks on are shared by a workgroup
  const RowSplit sp = split_rows(g, side, 4 * G, GPB);
  rl = RowLaunch{sp.hub.end, g->n};
  return sp.hub_grid + sp.rest_grid;
}

// LDS that k_gmmp_fwd_nr is launched with and does not use: three workgroups fit a CU instead of eight.  Past the L2s the kernel
// is bound by what misses them, and fewer rows in flight miss less.  MoNet forward, without -> with, us: 232 965
// vertices, 1.12 10^8 edges, K = 2, 16 columns (30 MB) 1646 -> 1573, 3 10^7 edges 407 -> 395; 100 000, 10^7, K = 3 (19 MB) 249 ->
// 223, 2 10^7, K = 2 (13 MB) 223 -> 224; two workgroups 1728, 251.  The backward walk, which the vector units bound, loses
// (1625 -> 1775).  A launch per 2 to 8 column blocks of the plan, which the L2s would hold: 2081 to 2440, bound by the
// segments' fixed work.  Rows of 20 edges from the neighbourhood lose, too, which are waited for: 100 000, K = 3 49 -> 64.
constexpr int64_t kFewWorkgroupsBytes = (int64_t)16 << 20;
constexpr unsigned kFewWorkgroupsLds = 34 * 1024;
constexpr int kFewWorkgroupsDegree = 32;
static unsigned nr_fwd_lds(const gnn_graph_t* g, int KF) {
  const bool long_rows = gathers_skewed(g, 0) || g->nnz >= kFewWorkgroupsDegree * (int64_t)g->n;
  return long_rows && (int64_t)sizeof(float) * KF * g->n > kFewWorkgroupsBytes ? kFewWorkgroupsLds : 0;
}

// Rows in flight of k_gmmp_fwd_nr and k_gmmp_bwd_dst_nr: eight, and fewer where gathers are even (gathers_abreast), all of whose
// workgroups then fit a CU.  Forward, uniform, eight -> two | one, us: 50 000 vertices, 60 edges each, K = 2, 16 columns (6.4 MB)
// 43 -> 40 | 50; 100 000, 70, 2, 8 (6.4 MB) 90 -> 67 | 77; 50 000, 60, 3, 16 (9.6 MB) 78 -> 57 | 65; 50 000, 60, 3, 20 (12 MB) 112 -> 82 | 71;
// 100 000, 120, 2, 16 (12.8 MB) 182 -> 135 | 127; 100 000, 120, 3, 16 (19 MB) 268 -> 260 | 215; 230 000, 60, 2, 8 (14.7 MB) 250 ->
// 233 | 172; 50 000, 60, 2, 8 (3.2 MB) 36 -> 37 | 44.  Destination side: 100 000, 70, 2, 16 238 -> 198 | 202; 100 000, 70, 3, 20 484 ->
// 480 | 411.  Neighbours that gather the same rows and skewed gathers lose: 100 000, 70, 2, 16 115 -> 133 and 120 -> 162 (two).
constexpr int64_t kTwoRowsBytes = (int64_t)6 << 20, kOneRowBytes = (int64_t)10 << 20;
constexpr int kOneRowFloats = 20;
// calls fn with the rows in flight and the LDS to launch with
template <typename Fn>
static gnn_status_t with_rows_in_flight(const gnn_graph_t* g, int KF, Fn fn) {
  const int64_t bytes = (int64_t)sizeof(float) * KF * g->n;
  if (bytes <= kTwoRowsBytes || !gathers_abreast(g, 0, KF, kTwoRowsBytes)) return fn(std::integral_constant<int, kNrU>{}, nr_fwd_lds(g, KF));
  if (KF < kOneRowFloats || bytes <= kOneRowBytes) return fn(std::integral_constant<int, 2>{}, 0u);
  return fn(std::integral_constant<int, 1>{}, 0u);
}

// Wavefronts per SIMD that k_gmmp_fwd_nr leaves room for: 7 (72 registers) with one coordinate, 6 with more.  Projected, in groups of eight
// lanes, it would take 73, and keeps two values in scratch memory to have one wavefront more.  Skewed gathers, which wait for their longest rows, are
// repaid for that with two or three kernels, and nothing else is.  Forward, us, room for 7 | 6: 2 x 8 columns, 230 000 vertices, 10 even edges
// 58.7 | 55.0, 2 x 16 65.3 | 59.9, 3 x 8 78.1 | 75.6, 4 x 8 63.0 | 58.9; power law, 2 x 8, 100 000, 60 198.6 | 204.6, 4 x 8 226.9 | 221.1.
template <int G, bool PROJ, int KT, int RT>
static gnn_status_t launch_fwd_nr(const gnn_graph_t* g, const RowLaunch& rl, unsigned grid, const float* hk, const float* pseudo, const ProjArgs& pa,
                                  const float* mu, const float* inv_sigma, const PsParams& pm, float* out, hipStream_t st) {
  return with_rows_in_flight(g, pm.K * pm.F, [&](auto u, unsigned lds) -> gnn_status_t {
    constexpr int U = decltype(u)::value;
    constexpr bool crowded = PROJ && G == 8 && RT == 1 && U == kNrU;
    auto run = [&](auto waves) -> gnn_status_t {
      k_gmmp_fwd_nr<G, PROJ, KT, RT, U, decltype(waves)::value><<<grid, kPsBlock, lds, st>>>(rl, g->rows[0], g->indices, hk, pseudo, pa, mu,
                                                                                             inv_sigma, pm, out);
      GNN_LAUNCH_CHECK();
      return GNN_OK;
    };
    if constexpr (crowded && KT < 4) {
      if (gathers_skewed(g, 0)) return run(std::integral_constant<int, 7>{});
    }
    return run(std::integral_constant<int, (RT == 1 && !crowded ? 7 : 6)>{});
  });
}

// k_monet_res takes graphs with column blocks from so many edges on: below, its launch and its barriers per block are not repaid,
// and where degrees are uneven they are sooner, since k_gmmp_fwd_nr then waits for the longest rows.  k_gmmp_fwd_nr | k_monet_res, K = 2,
// 16 columns, us: uneven 13 000 vertices, 5 10^5 edges 25 | 30 (K = 4: 40 | 33), 20 000, 1.2 10^6 44 | 34, 13 000, 1.3 10^6 40 | 34, 14 000, 4.2 10^6
// 125 | 67 (K = 3); even 30 000, 3 10^6 41 | 46, 50 000, 4.5 10^6 101 | 102 (3 x 20), 5 10^6 104 | 98 (K = 4), 20 000, 6 10^6 60 | 58 (8
// columns), 25 000, 10^7 179 | 154 (3 x 20), 100 000, 1.5 10^7 169 | 159 (8).
// Rows whose edges are not in the order of the blocks leave a graph to k_gmmp_fwd_nr: coordinates of edges could not be found block by
// block, and projected and given coordinates have the same sums, bit for bit.
constexpr int64_t kMonetEdgesUneven = (int64_t)1 << 20, kMonetEdgesEven = (int64_t)5 << 20;
constexpr int64_t kMonetEdgesPerBlock = 16;  // of a row, on average: fewer were not timed
static bool monet_res_applies(const gnn_graph_t* g, int KF) {
  const bool uneven = gathers_skewed(g, 0) || gathers_skewed(g, 1);
  const bool enough = g->nnz >= (uneven ? kMonetEdgesUneven : kMonetEdgesEven) &&
                      g->nnz >= kMonetEdgesPerBlock * (int64_t)g->n * g->nblk;
  return (enough || config_get(kCfgResidentSums) == 2) && g->blocked_pays() && !config_get(kCfgForceSimple) && config_get(kCfgResidentSums) && g->phase_clock != nullptr &&
         g->in_block_order[0] && g->block_cols <= kMonetTabPerThread * kMonetThreads && narrow_table(g->n, KF) && !config_get(kCfgWideOffsets);
}

template <int G, bool PROJ, int KT, int RT>
static gnn_status_t launch_monet_res(const gnn_graph_t* g, const float* hk, const float* pseudo, const ProjArgs& pa, const float* mu,
                                     const float* inv_sigma, const PsParams& pm, float* out, hipStream_t st) {
  constexpr int kLds = 160 * 1024;
  static std::atomic<bool> allowed{false};
  if (!allowed.load(std::memory_order_acquire)) {
    GNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_monet_res<G, PROJ, KT, RT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLds));
    allowed.store(true, std::memory_order_release);
  }
  const int64_t grid = device_cu_count() / kXcds * kXcds;
  const int room = (kLds / 4 - 2 - (g->block_cols + 3) / 4 * 4 - kMonetGroupInts<G, KT>) / monet_slot_ints(pm.F);
  const int cap = std::min(room, kMonetThreads) / 4 * 4;
  // parts of more than half of what a group has on average, and at most twice that (a quarter as long: 970 -> 970 us, see above)
  const RowParts cut = cut_rows(g, 0, std::max<int64_t>(64, g->nnz / (grid * (kMonetThreads / G))), grid, cap);
  k_monet_zero_clock<<<1, kXcds * kClockStride, 0, st>>>(g->phase_clock);
  GNN_LAUNCH_CHECK();
  k_monet_res<G, PROJ, KT, RT><<<(unsigned)grid, kMonetThreads, kLds, st>>>(
      g->n, g->order[0], reinterpret_cast<const int2*>(g->bseg[0]), g->indptr, PROJ ? g->bcol[0] : g->indices, hk, pseudo, pa, mu,
      inv_sigma, pm, g->block_cols, g->nblk, cap, cut, g->phase_clock, (int)config_get(kCfgResidentSpin),
      (int)config_get(kCfgResidentSyncEvery), out);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

// partial slots of the kernels that sum the parameters' gradients: enough for any of them
static int64_t ps_dst_blocks(const gnn_graph_t* g, int fout) {
  RowLaunch rl;
  int64_t b;
  switch (ps_lanes(fout)) {
    case 4: b = ps_grid<4>(g, 0, rl); break;
    case 8: b = ps_grid<8>(g, 0, rl); break;
    case 16: b = ps_grid<16>(g, 0, rl); break;
    case 32: b = ps_grid<32>(g, 0, rl); break;
    default: b = ps_grid<64>(g, 0, rl); break;
  }
  for (int side = 0; side < 2; ++side) b = std::max<int64_t>({b, nr_grid<8>(g, side, rl), nr_grid<16>(g, side, rl)});
  return b;
}

struct GmmpWs {
  size_t total, dhk, partial, gemm;
  int split_k;
  int64_t nblk;
};
static GmmpWs gmmp_ws_layout(const gnn_graph_t* g, int fin, int fout, int K) {
  GmmpWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += ws_granule(bytes); return o; };
  w.nblk = ps_dst_blocks(g, fout);
  w.dhk = take(sizeof(float) * (size_t)g->n * K * fout);
  // doubles where one walk does both sides, floats (with fewer columns) where the destination side has its own
  w.partial = take(sizeof(double) * (size_t)(w.nblk + 1 + sum_partials_scratch_rows((int)w.nblk)) * kPsValsProj);
  w.split_k = gemm_pick_split_k(fin, K * fout, g->n);
  w.gemm = take(w.split_k > 1 ? sizeof(float) * (size_t)w.split_k * fin * K * fout : 0);
  w.total = off;
  return w;
}

static gnn_status_t gmmp_check(const gnn_graph_t* g, int fin, int fout, int K, int R, const char* who) {
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "%s: graph is null", who);
  GNN_REQUIRE(fin > 0 && fout > 0 && K > 0 && R > 0, GNN_ERR_INVALID_ARG, "%s: sizes must be positive", who);
  GNN_REQUIRE(fout % 4 == 0 && fout <= 256, GNN_ERR_UNSUPPORTED,
              "%s: fout = %d must be a multiple of 4, at most 256", who, fout);
  GNN_REQUIRE(K <= kPsK && R <= kPsR, GNN_ERR_UNSUPPORTED, "%s: at most %d kernels and %d dimensions", who, kPsK,
              kPsR);
  return GNN_OK;
}

// calls fn with the lane count of a row group as a compile-time constant
template <typename Fn>
static gnn_status_t for_lanes(int lanes, Fn fn) {
  switch (lanes) {
    case 4: return fn(std::integral_constant<int, 4>{});
    case 8: return fn(std::integral_constant<int, 8>{});
    case 16: return fn(std::integral_constant<int, 16>{});
    case 32: return fn(std::integral_constant<int, 32>{});
    default: return fn(std::integral_constant<int, 64>{});
  }
}

// Calls fn with the numbers of kernels and of dimensions that a kernel is compiled for, as constants: the vector units
// bound the backward kernel, and its work per edge grows with both.
template <typename Fn>
static gnn_status_t for_kernels(int K, int R, Fn fn) {
  auto dims = [&](auto kernels) -> gnn_status_t {
    switch (R) {
      case 1: return fn(kernels, std::integral_constant<int, 1>{});
      case 2: return fn(kernels, std::integral_constant<int, 2>{});
      case 3: return fn(kernels, std::integral_constant<int, 3>{});
      default: return fn(kernels, std::integral_constant<int, 4>{});
    }
  };
  switch (K) {
    case 1:
    case 2: return dims(std::integral_constant<int, 2>{});
    case 3: return dims(std::integral_constant<int, 3>{});
    default: return dims(std::integral_constant<int, 4>{});
  }
}

// what a product gw = x^T dhk that was split over K left to sum up; nothing if it was not
static PartialSum parts_of_product(int fin, int KF, int split_k, const float* parts, float* gw) {
  const int64_t size = split_k > 1 ? (int64_t)fin * KF : 0;
  return {size, size, split_k, parts, gw};
}

// the parameters' gradients from k_gmmp_bwd_nr's partials, and the sum of a product's; the rows of ranges go behind those
static gnn_status_t wide_param_sums(int K, int R, int kt, int rt, int parts, double* partial, float* gmu, float* gis,
                                    float* gP, float* gpb, const PartialSum& product, hipStream_t st) {
  const int nvals = 2 * kt * rt + (gP != nullptr ? 3 * rt : 0);
  int nrows = parts;
  const double* rows = partial;
  if (parts > kParamChunk) {
    double* out = partial + (int64_t)parts * nvals;
    nrows = (int)cdiv(parts, kParamChunk);
    k_gmmp_param_rows<<<(unsigned)nrows, kParamThreads, 0, st>>>(nvals, parts, partial, out);
    GNN_LAUNCH_CHECK();
    rows = out;
  }
  const unsigned blocks = product.count > 0 ? (unsigned)cdiv(sum_blocks(product), kParamThreads / 256) : 0;
  k_gmmp_param_totals<<<1 + blocks, kParamThreads, 0, st>>>(K, R, kt, rt, nrows, rows, gmu, gis, gP, gpb, product, sums_wide(product));
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

// With coordinates given per edge the one walk stores gpseudo through the CSC position -> CSR edge id table, 4 R bytes at a time,
// which pays while the array stays in the caches; beyond, a walk over the in-edges makes gpseudo and the dot products of the
// walk over the out-edges once more.  Backward, us, apart -> one walk, coordinates in both orders: 2 10^6 edges, R = 3, K = 3, 25 MB
// 160 -> 116; 3 10^6, R = 2, K = 2, 24 MB 253 -> 197; 10^7, R = 1, 40 MB 385 -> 431; R = 3, 120 MB 443 -> 551; 1.12 10^8, R = 1
// 2632 -> 4028.  With more kernels and columns the one walk stays ahead for longer (3 10^7 edges, R = 3, K = 3, 20 columns, 360 MB
// 1702 -> 1509), which the rule makes no use of.
constexpr int64_t kOneWalkBytes = (int64_t)32 << 20;
static bool one_walk_pays(const gnn_graph_t* g, int R) { return g->nnz * R * (int64_t)sizeof(float) <= kOneWalkBytes; }

}  // namespace gnn

using namespace gnn;

extern "C" size_t gnn_gmmp_workspace_bytes(const gnn_graph_t* g, int fin, int fout, int k) {
  if (!g || fin <= 0 || fout <= 0 || k <= 0 || fout % 4 != 0 || fout > 256) return 0;
  return gmmp_ws_layout(g, fin, fout, k).total;
}

extern "C" gnn_status_t gnn_gmmp_fwd(const gnn_graph_t* g, int fin, int fout, int k, int r, const float* x,
                                     const float* w_fc, const float* pseudo, const float* mu,
                                     const float* inv_sigma, float* hk, float* out, void* stream) {
  clear_error();
  GNN_TRY(gmmp_check(g, fin, fout, k, r, "gnn_gmmp_fwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w_fc && mu && inv_sigma && hk && out && (pseudo || g->nnz == 0), GNN_ERR_INVALID_ARG,
              "gnn_gmmp_fwd: null pointer");
  GNN_REQUIRE(aligned16(hk) && aligned16(out), GNN_ERR_INVALID_ARG, "gnn_gmmp_fwd: hk, out must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  GNN_TRY(gemm_f32(g->n, k * fout, fin, x, fin, false, w_fc, k * fout, false, hk, k * fout, 1, nullptr, st));
  const PsParams pm{k, r, fout, (int)config_get(kCfgWideOffsets)};
  ProfScope p("gmmp_fwd_fused", st);
  if (const int G = nr_lanes(k, fout)) {
    return for_lanes(G, [&](auto lanes) -> gnn_status_t {
      constexpr int GL = decltype(lanes)::value == 8 ? 8 : 16;
      RowLaunch rl;
      const unsigned grid = nr_grid<GL>(g, 0, rl);
      if (grid != 0) {
        return for_kernels(k, r, [&](auto kernels, auto dims) -> gnn_status_t {
          constexpr int KT = decltype(kernels)::value, RT = decltype(dims)::value;
          if (monet_res_applies(g, k * fout))
            return launch_monet_res<GL, false, KT, RT>(g, hk, pseudo, ProjArgs{}, mu, inv_sigma, pm, out, st);
          return launch_fwd_nr<GL, false, KT, RT>(g, rl, grid, hk, pseudo, ProjArgs{}, mu, inv_sigma, pm, out, st);
        });
      }
      return GNN_OK;
    });
  }
  return for_lanes(ps_lanes(fout), [&](auto lanes) -> gnn_status_t {
    constexpr int L = decltype(lanes)::value;
    RowLaunch rl;
    const unsigned grid = ps_grid<L>(g, 0, rl);
    if (grid != 0) {
      k_gmmp_fwd<L><<<grid, kPsBlock, 0, st>>>(rl, g->order[0], g->indptr, g->indices, hk, pseudo, mu, inv_sigma,
                                              pm, out);
      GNN_LAUNCH_CHECK();
    }
    return GNN_OK;
  });
}

extern "C" gnn_status_t gnn_gmmp_bwd(const gnn_graph_t* g, int fin, int fout, int k, int r, const float* x,
                                     const float* w_fc, const float* pseudo, const float* mu,
                                     const float* inv_sigma, const float* hk, const float* gout, float* gx,
                                     float* gw_fc, float* gmu, float* ginv_sigma, float* gpseudo,
                                     const float* pseudo_t, void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  GNN_TRY(gmmp_check(g, fin, fout, k, r, "gnn_gmmp_bwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w_fc && mu && inv_sigma && hk && gout && gw_fc && gmu && ginv_sigma && (pseudo || g->nnz == 0),
              GNN_ERR_INVALID_ARG, "gnn_gmmp_bwd: null pointer");
  GNN_REQUIRE(aligned16(hk) && aligned16(gout), GNN_ERR_INVALID_ARG,
              "gnn_gmmp_bwd: hk, gout must be 16-byte aligned");
  const GmmpWs W = gmmp_ws_layout(g, fin, fout, k);
  GNN_REQUIRE(ws != nullptr && ws_bytes >= W.total, GNN_ERR_WORKSPACE,
              "gnn_gmmp_bwd: workspace of %zu bytes given, %zu needed", ws_bytes, W.total);
  GNN_REQUIRE(aligned16(ws), GNN_ERR_INVALID_ARG, "gnn_gmmp_bwd: workspace must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(ws);
  float* dhk = reinterpret_cast<float*>(base + W.dhk);
  float* partial = reinterpret_cast<float*>(base + W.partial);
  double* wide = reinterpret_cast<double*>(base + W.partial);
  float* part = reinterpret_cast<float*>(base + W.gemm);
  const PsParams pm{k, r, fout, (int)config_get(kCfgWideOffsets)};
  const int KF = k * fout;
  const int G = nr_lanes(k, fout);
  auto param_sums = [&](unsigned grid) -> gnn_status_t {  // of the destination side's kernels
    float* totals = partial + (int64_t)grid * kPsVals;
    GNN_TRY(sum_partials_two_level(kPsVals, (int)grid, partial, totals + kPsVals, totals, st));
    k_gmmp_param_split<<<1, 64, 0, st>>>(k, r, totals, gmu, ginv_sigma);
    GNN_LAUNCH_CHECK();
    return GNN_OK;
  };
  if (G) {
    const bool apart = gpseudo != nullptr && !one_walk_pays(g, r);
    if (apart) {
      ProfScope p("gmmp_bwd_dst", st);
      GNN_TRY(for_lanes(G, [&](auto lanes) -> gnn_status_t {
        constexpr int GL = decltype(lanes)::value == 8 ? 8 : 16;
        RowLaunch rl;
        const unsigned grid = nr_grid<GL>(g, 0, rl);
        if (grid == 0) return GNN_OK;
        return for_kernels(k, r, [&](auto kernels, auto dims) -> gnn_status_t {
          constexpr int KT = decltype(kernels)::value, RT = decltype(dims)::value;
          return with_rows_in_flight(g, KF, [&](auto u, unsigned lds) -> gnn_status_t {
            k_gmmp_bwd_dst_nr<GL, KT, RT, decltype(u)::value><<<grid, kPsBlock, lds, st>>>(rl, g->rows[0], g->indices, hk, pseudo, mu,
                                                                                           inv_sigma, gout, pm, gpseudo);
            GNN_LAUNCH_CHECK();
            return GNN_OK;
          });
        });
      }));
    }
    ProfScope p(apart ? "gmmp_bwd_src" : "gmmp_bwd", st);
    GNN_TRY(for_lanes(G, [&](auto lanes) -> gnn_status_t {
      constexpr int GL = decltype(lanes)::value == 8 ? 8 : 16;
      RowLaunch rl;
      const unsigned grid = nr_grid<GL>(g, 1, rl);
      if (grid == 0) return GNN_OK;
      return for_kernels(k, r, [&](auto kernels, auto dims) -> gnn_status_t {
        constexpr int KT = decltype(kernels)::value, RT = decltype(dims)::value;
        k_gmmp_bwd_nr<GL, false, KT, RT><<<grid, kPsBlock, 0, st>>>(rl, g->rows[1], g->indices_t, g->eid_t, hk, pseudo, pseudo_t,
                                                                   ProjArgs{}, mu, inv_sigma, gout, pm, dhk, wide,
                                                                   apart ? nullptr : gpseudo);
        GNN_LAUNCH_CHECK();
        return wide_param_sums(k, r, KT, RT, (int)grid, wide, gmu, ginv_sigma, nullptr, nullptr, PartialSum{}, st);
      });
    }));
  } else {
    {
      ProfScope p("gmmp_bwd_dst", st);
      unsigned grid = 0;
      GNN_TRY(for_lanes(ps_lanes(fout), [&](auto lanes) -> gnn_status_t {
        constexpr int L = decltype(lanes)::value;
        RowLaunch rl;
        grid = ps_grid<L>(g, 0, rl);
        if (grid == 0) return GNN_OK;
        k_gmmp_bwd_dst<L><<<grid, kPsBlock, 0, st>>>(rl, g->order[0], g->indptr, g->indices, hk, pseudo, mu,
                                                    inv_sigma, gout, pm, partial, gpseudo);
        GNN_LAUNCH_CHECK();
        return GNN_OK;
      }));
      GNN_TRY(param_sums(grid));
    }
    {
      ProfScope p("gmmp_bwd_src", st);
      GNN_TRY(for_lanes(ps_lanes(fout), [&](auto lanes) -> gnn_status_t {
        constexpr int L = decltype(lanes)::value;
        RowLaunch rl;
        const unsigned grid = ps_grid<L>(g, 1, rl);
        if (grid == 0) return GNN_OK;
        k_gmmp_bwd_src<L><<<grid, kPsBlock, 0, st>>>(rl, g->order[1], g->indptr_t, g->indices_t, g->eid_t, pseudo,
                                                    pseudo_t, mu, inv_sigma, gout, pm, dhk);
        GNN_LAUNCH_CHECK();
        return GNN_OK;
      }));
    }
  }
  GNN_TRY(gemm_f32(fin, KF, g->n, x, fin, true, dhk, KF, false, gw_fc, KF, W.split_k, part, st));
  if (gx) GNN_TRY(gemm_f32(g->n, fin, KF, dhk, KF, false, w_fc, KF, true, gx, fin, 1, nullptr, st));
  return GNN_OK;
}

// workgroups of the projection's backward pass (= partial slots): four rows per workgroup, at most 2048
static int proj_blocks(int64_t n) {
  int64_t b = cdiv(n > 0 ? n : 1, kPsBlock / 64);
  return (int)(b > 2048 ? 2048 : b);
}

extern "C" size_t gnn_pseudo_proj_workspace_bytes(const gnn_graph_t* g) {
  if (!g) return 0;
  const int64_t blocks = proj_blocks(g->n);
  return ws_granule(sizeof(float) * (size_t)(blocks + 1 + sum_partials_scratch_rows((int)blocks)) * 3 * kPsR);
}

extern "C" gnn_status_t gnn_pseudo_proj_fwd(const gnn_graph_t* g, int r, const float* c, const float* proj_w,
                                            const float* proj_b, float* pseudo, float* pseudo_t, void* stream) {
  clear_error();
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "gnn_pseudo_proj_fwd: graph is null");
  GNN_REQUIRE(r > 0 && r <= kPsR, GNN_ERR_UNSUPPORTED, "gnn_pseudo_proj_fwd: r = %d outside 1..%d", r, kPsR);
  if (g->n == 0 || g->nnz == 0) return GNN_OK;
  GNN_REQUIRE(c && proj_w && proj_b && pseudo, GNN_ERR_INVALID_ARG, "gnn_pseudo_proj_fwd: null pointer");
  hipStream_t st = static_cast<hipStream_t>(stream);
  ProfScope p("pseudo_proj_fwd", st);
  const unsigned grid = (unsigned)cdiv((int64_t)g->n * 64, 256);
  k_pseudo_proj_fwd<<<grid, 256, 0, st>>>(g->n, g->indptr, g->indices, c, r, proj_w, proj_b, 0, pseudo);
  GNN_LAUNCH_CHECK();
  if (pseudo_t != nullptr) {
    k_pseudo_proj_fwd<<<grid, 256, 0, st>>>(g->n, g->indptr_t, g->indices_t, c, r, proj_w, proj_b, 1, pseudo_t);
    GNN_LAUNCH_CHECK();
  }
  return GNN_OK;
}

extern "C" gnn_status_t gnn_pseudo_proj_bwd(const gnn_graph_t* g, int r, const float* c, const float* pseudo,
                                            const float* gpseudo, float* gproj_w, float* gproj_b, void* ws,
                                            size_t ws_bytes, void* stream) {
  clear_error();
  GNN_REQUIRE(g != nullptr, GNN_ERR_INVALID_ARG, "gnn_pseudo_proj_bwd: graph is null");
  GNN_REQUIRE(r > 0 && r <= kPsR, GNN_ERR_UNSUPPORTED, "gnn_pseudo_proj_bwd: r = %d outside 1..%d", r, kPsR);
  GNN_REQUIRE(gproj_w && gproj_b, GNN_ERR_INVALID_ARG, "gnn_pseudo_proj_bwd: null pointer");
  GNN_REQUIRE(ws != nullptr && ws_bytes >= gnn_pseudo_proj_workspace_bytes(g), GNN_ERR_WORKSPACE,
              "gnn_pseudo_proj_bwd: workspace of %zu bytes given, %zu needed", ws_bytes,
              gnn_pseudo_proj_workspace_bytes(g));
  GNN_REQUIRE(g->nnz == 0 || (c && pseudo && gpseudo), GNN_ERR_INVALID_ARG, "gnn_pseudo_proj_bwd: null pointer");
  hipStream_t st = static_cast<hipStream_t>(stream);
  ProfScope p("pseudo_proj_bwd", st);
  const int blocks = proj_blocks(g->n);
  float* partial = static_cast<float*>(ws);
  k_pseudo_proj_bwd<<<blocks, kPsBlock, 0, st>>>(g->n, g->indptr, g->indices, c, r, pseudo, gpseudo, partial);
  GNN_LAUNCH_CHECK();
  float* totals = partial + (int64_t)blocks * 3 * kPsR;
  GNN_TRY(sum_partials_two_level(3 * kPsR, blocks, partial, totals + 3 * kPsR, totals, st));
  k_pseudo_proj_split<<<1, 64, 0, st>>>(r, totals, gproj_w, gproj_b);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

// ---- MoNet layer with the projection of the degree pair fused in ------------------------------
static gnn_status_t monet_check(const gnn_graph_t* g, int fin, int fout, int K, int R, const char* who) {
  GNN_TRY(gmmp_check(g, fin, fout, K, R, who));
  GNN_REQUIRE(K * fout <= 64, GNN_ERR_UNSUPPORTED,
              "%s: k * fout = %d above 64 (wider layers: gnn_pseudo_proj_fwd + gnn_gmmp_fwd)", who, K * fout);
  return GNN_OK;
}

extern "C" size_t gnn_monet_workspace_bytes(const gnn_graph_t* g, int fin, int fout, int k) {
  return gnn_gmmp_workspace_bytes(g, fin, fout, k);
}

extern "C" gnn_status_t gnn_monet_fwd(const gnn_graph_t* g, int fin, int fout, int k, int r, const float* x,
                                      const float* w_fc, const float* c, const float* proj_w,
                                      const float* proj_b, const float* mu, const float* inv_sigma, float* hk,
                                      float* out, void* stream) {
  clear_error();
  GNN_TRY(monet_check(g, fin, fout, k, r, "gnn_monet_fwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w_fc && c && proj_w && proj_b && mu && inv_sigma && hk && out, GNN_ERR_INVALID_ARG,
              "gnn_monet_fwd: null pointer");
  GNN_REQUIRE(aligned16(hk) && aligned16(out), GNN_ERR_INVALID_ARG, "gnn_monet_fwd: hk, out must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  GNN_TRY(gemm_f32(g->n, k * fout, fin, x, fin, false, w_fc, k * fout, false, hk, k * fout, 1, nullptr, st));
  const PsParams pm{k, r, fout, (int)config_get(kCfgWideOffsets)};
  const ProjArgs pa{c, proj_w, proj_b};
  ProfScope p("monet_fwd_fused", st);
  return for_lanes(k * fout <= 32 ? 8 : 16, [&](auto lanes) -> gnn_status_t {
    constexpr int GL = decltype(lanes)::value == 8 ? 8 : 16;
    RowLaunch rl;
    const unsigned grid = nr_grid<GL>(g, 0, rl);
    if (grid != 0) {
      return for_kernels(k, r, [&](auto kernels, auto dims) -> gnn_status_t {
        constexpr int KT = decltype(kernels)::value, RT = decltype(dims)::value;
        if (monet_res_applies(g, k * fout))
          return launch_monet_res<GL, true, KT, RT>(g, hk, nullptr, pa, mu, inv_sigma, pm, out, st);
        return launch_fwd_nr<GL, true, KT, RT>(g, rl, grid, hk, nullptr, pa, mu, inv_sigma, pm, out, st);
      });
    }
    return GNN_OK;
  });
}

extern "C" gnn_status_t gnn_monet_bwd(const gnn_graph_t* g, int fin, int fout, int k, int r, const float* x,
                                      const float* w_fc, const float* c, const float* proj_w,
                                      const float* proj_b, const float* mu, const float* inv_sigma,
                                      const float* hk, const float* gout, float* gx, float* gw_fc, float* gmu,
                                      float* ginv_sigma, float* gproj_w, float* gproj_b, void* ws,
                                      size_t ws_bytes, void* stream) {
  clear_error();
  GNN_TRY(monet_check(g, fin, fout, k, r, "gnn_monet_bwd"));
  if (g->n == 0) return GNN_OK;
  GNN_REQUIRE(x && w_fc && c && proj_w && proj_b && mu && inv_sigma && hk && gout && gw_fc && gmu && ginv_sigma &&
                  gproj_w && gproj_b,
              GNN_ERR_INVALID_ARG, "gnn_monet_bwd: null pointer");
  GNN_REQUIRE(aligned16(hk) && aligned16(gout), GNN_ERR_INVALID_ARG,
              "gnn_monet_bwd: hk, gout must be 16-byte aligned");
  const GmmpWs W = gmmp_ws_layout(g, fin, fout, k);
  GNN_REQUIRE(ws != nullptr && ws_bytes >= W.total, GNN_ERR_WORKSPACE,
              "gnn_monet_bwd: workspace of %zu bytes given, %zu needed", ws_bytes, W.total);
  GNN_REQUIRE(aligned16(ws), GNN_ERR_INVALID_ARG, "gnn_monet_bwd: workspace must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(ws);
  float* dhk = reinterpret_cast<float*>(base + W.dhk);
  double* partial = reinterpret_cast<double*>(base + W.partial);
  float* part = reinterpret_cast<float*>(base + W.gemm);
  const PsParams pm{k, r, fout, (int)config_get(kCfgWideOffsets)};
  const ProjArgs pa{c, proj_w, proj_b};
  const int KF = k * fout;
  const int G = KF <= 32 ? 8 : 16;
  unsigned grid = 0;
  {
    ProfScope p("monet_bwd", st);
    GNN_TRY(for_lanes(G, [&](auto lanes) -> gnn_status_t {
      constexpr int GL = decltype(lanes)::value == 8 ? 8 : 16;
      RowLaunch rl;
      grid = nr_grid<GL>(g, 1, rl);
      if (grid == 0) return GNN_OK;
      return for_kernels(k, r, [&](auto kernels, auto dims) -> gnn_status_t {
        constexpr int KT = decltype(kernels)::value, RT = decltype(dims)::value;
        k_gmmp_bwd_nr<GL, true, KT, RT><<<grid, kPsBlock, 0, st>>>(rl, g->rows[1], g->indices_t, g->eid_t, hk,
                                                                  nullptr, nullptr, pa, mu, inv_sigma, gout, pm, dhk,
                                                                  partial, nullptr);
        GNN_LAUNCH_CHECK();
        return GNN_OK;
      });
    }));
  }
  GNN_TRY(gemm_f32(fin, KF, g->n, x, fin, true, dhk, KF, false, W.split_k > 1 ? nullptr : gw_fc, KF, W.split_k, part, st));
  {
    ProfScope p("monet_param_grad", st);
    GNN_TRY(for_kernels(k, r, [&](auto kernels, auto dims) -> gnn_status_t {
      return wide_param_sums(k, r, decltype(kernels)::value, decltype(dims)::value, (int)grid, partial, gmu, ginv_sigma,
                             gproj_w, gproj_b, parts_of_product(fin, KF, W.split_k, part, gw_fc), st);
    }));
  }
  if (gx) GNN_TRY(gemm_f32(g->n, fin, KF, dhk, KF, false, w_fc, KF, true, gx, fin, 1, nullptr, st));
  return GNN_OK;
}
