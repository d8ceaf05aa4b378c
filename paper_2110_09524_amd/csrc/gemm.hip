// fp32 dense products on the MFMA matrix cores: the ExpensiveApply projections that the
// reorganization moves onto vertices (Sec. 4) and their two backward products (App. B, "Apply").
//
// The fp32 MFMA runs at 1/16 of the bf16 rate, so every fp32 operand element is split into three
// bf16 parts, x = h + m + l (8 + 8 + 8 significand bits: the whole fp32 significand), and a
// product is the sum of the six partial products h h, h m, m h, m m, h l, l h with fp32
// accumulators (v_mfma_f32_32x32x16_bf16).  What is left out (m l, l m, l l) is at most 2^-24 of the
// product, the largest error of one fp32 rounding (above 2^-26 for one product in eight).  bf16 ends 16 binary digits above fp32 (2^-133 against
// 2^-149), so below 2^-109 the last part would lose digits: both operands are multiplied by 2^16
// before they are split, and the result by 2^-32.  A result that is not finite in these units (an
// infinity or a NaN among the operands, an operand above 2^111, or a sum above 2^96) is taken from
// the fp32 MFMA, on which its whole tile is computed again, so such values come out as fp32
// arithmetic gives them (232965 x 602 x 256: 469 us, 476 us with one infinity, 1013 us with one in every tile).
//
// Tiling: a workgroup of WR x WC wavefronts owns a BM x BN tile of C.  K advances 16 at a time
// through two LDS buffers: while the matrix cores work on one slab, the wavefronts split the next
// one in registers and park it in the other buffer, and the loads of the slab after that travel.
// The vector instructions of the split have to stand between the MFMAs of the same wavefront: a
// wavefront that issues MFMAs back to back keeps the vector instructions of the others on its SIMD
// waiting (measured: MFMA and FMA loops of two wavefronts take the sum of their times, interleaved
// in one wavefront the larger of the two).  LDS is laid out [part][k / 8][row], so a wavefront's
// operand read is two contiguous runs of 512 bytes whatever the operands' layout in HBM (an operand
// stored k-major is transposed on the way, in registers).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "partial_sums.h"

namespace gnn {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int BK = 16;     // k per slab
constexpr int kParts = 3;
constexpr float kScale = 65536.f;  // of either operand
// Up to this many terms the fp32 chain alone: it rounds once per term, six partial products up to six times.  Relative
// error of x w against 64 bits (40000 x K x 64, 2-norm, four inputs), parts and chain: K = 1 3.4e-8 and 2.5e-8, 2 3.4e-8 and
// 3.1e-8, 3 3.3e-8 and 3.6e-8, 4 3.3e-8 and 4.0e-8, 8 3.1e-8 and 5.4e-8.
constexpr int kDirectK = 2;

// Attention halves in the epilogue of the projection (Sec. 4, text after Eq. 1: the score splits
// into a source half <a_l, z[u]> and a destination half <a_r, z[v]>, both per-vertex): el[m, h] =
// sum_f a_l[h, f] C[m, h*F + f], er likewise, taken from the accumulators before they are stored,
// so z is not read again.  A lane holds one column of a 32-column MFMA tile, so the sum over a
// head is a butterfly over the lanes of the tile that belong to that head (F = 4, 8, 16, 32),
// over all tiles and lanes of a wavefront (F = its columns), or, for a single head that one
// workgroup covers, over its wavefronts as well (through LDS).
// v + (v of the lane the DPP control pairs this lane with), one VALU operation
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  const int t = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true);
  return v + __int_as_float(t);
}
// Sum over aligned segments of `seg` lanes (a power of two, 1 .. 32); every lane of a segment ends
// with the segment's total.  Pairings: lane ^ 1 and lane ^ 2 inside quads, then mirrored halves
// of 8 and of 16 lanes (valid because all lanes of the smaller segment already agree), then the
// other row of 16 through the crossbar.
__device__ __forceinline__ float segment_sum(float v, int seg) {
  if (seg > 1) v = dpp_add<0xB1>(v);    // quad_perm [1,0,3,2]
  if (seg > 2) v = dpp_add<0x4E>(v);    // quad_perm [2,3,0,1]
  if (seg > 4) v = dpp_add<0x141>(v);   // row_half_mirror
  if (seg > 8) v = dpp_add<0x140>(v);   // row_mirror
  if (seg > 16) v += __shfl_xor(v, 16, 64);
  return v;
}

struct AttnEpilogue {
  const float* a_l;
  const float* a_r;
  float* el;
  float* er;
  int H, F;
};

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {  // round to nearest even, both at once
  const floatx2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// One operand of a workgroup's tile: ROWS rows (of A) or columns (of B), fetched 16 k at a time.
// A thread fetches kUnit consecutive k of one row.  Rows past the matrix are clamped to its last one
// (their products land where nothing is stored); only the last, partial slab needs predicated loads.
template <int ROWS, int THREADS, bool KCONTIG>
struct Operand {
  static constexpr int kUnit = ROWS * BK / THREADS;   // 2, 4 or 8
  static constexpr int kPerRow = BK / kUnit;          // threads that fetch one row
  static constexpr int kOctStride = ROWS + 4;         // padded: 8 lanes that store two octets of 4 rows meet different banks
  static constexpr int kPartStride = BK / 8 * kOctStride;   // in 16-byte vectors, like kLds
  static constexpr int kLds = kParts * kPartStride;
  static constexpr int kChainStride = ROWS + 4;             // floats from one k to the next, padded likewise
  static constexpr int kChainLds = BK * kChainStride / 4;   // in 16-byte vectors
  static_assert(kUnit == 2 || kUnit == 4 || kUnit == 8, "a thread stores 4, 8 or 16 bytes of each part");

  float raw[2][kUnit];
  uint32_t off;  // floats from the slab's base to the thread's first one
  const float* base;
  int64_t ld, step;

  static __device__ __forceinline__ int row() { return KCONTIG ? threadIdx.x / kPerRow : threadIdx.x % ROWS; }
  static __device__ __forceinline__ int k() { return kUnit * (KCONTIG ? threadIdx.x % kPerRow : threadIdx.x / ROWS); }

  __device__ __forceinline__ void init(const float* p, int64_t ld_, int64_t row0, int64_t rows, int64_t k_begin) {
    ld = ld_;
    base = KCONTIG ? p + row0 * ld + k_begin : p + k_begin * ld + row0;
    step = KCONTIG ? BK : BK * ld;
    const int64_t r = row0 + row() < rows ? row() : rows - 1 - row0;
    off = (uint32_t)(KCONTIG ? r * ld + k() : k() * ld + r);
  }

  // slab `s`, all of its k in the matrix
  __device__ __forceinline__ void load(int set, int64_t s) {
    const float* b = base + s * step;
    if constexpr (KCONTIG) {
      typedef float vec __attribute__((ext_vector_type(kUnit < 4 ? kUnit : 4), aligned(4)));
      constexpr int V = kUnit < 4 ? kUnit : 4;
#pragma unroll
      for (int j = 0; j < kUnit; j += V) {
        const vec v = *reinterpret_cast<const vec*>(b + off + j);
#pragma unroll
        for (int c = 0; c < V; ++c) raw[set][j + c] = v[c];
      }
    } else {
#pragma unroll
      for (int j = 0; j < kUnit; ++j)  // uniform row address + 32-bit byte offset
        raw[set][j] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(b + j * ld) + 4u * off);
    }
  }

  // the last slab, of which only `rem` < BK values of k exist
  __device__ __forceinline__ void load_partial(int set, int64_t s, int rem) {
    const float* b = base + s * step;
#pragma unroll
    for (int j = 0; j < kUnit; ++j) raw[set][j] = k() + j < rem ? b[(int64_t)off + (KCONTIG ? j : j * ld)] : 0.f;
  }

  // scale * raw = h + m + l in bf16, to LDS
  __device__ __forceinline__ void store(int set, float scale, uint4* lds) const {
    uint32_t w[kParts][kUnit / 2];
#pragma unroll
    for (int q = 0; q < kUnit / 2; ++q) {
      float a = scale * raw[set][2 * q], b = scale * raw[set][2 * q + 1];
#pragma unroll
      for (int p = 0; p < kParts; ++p) {
        w[p][q] = pack_bf16(a, b);
        if (p + 1 < kParts) {  // exact: what the bf16 part left over
          a -= __uint_as_float(w[p][q] << 16);
          b -= __uint_as_float(w[p][q] & 0xffff0000u);
        }
      }
    }
    uint32_t* dst = reinterpret_cast<uint32_t*>(lds + k() / 8 * kOctStride + row()) + k() % 8 / 2;
#pragma unroll
    for (int p = 0; p < kParts; ++p, dst += 4 * kPartStride) {
      if constexpr (kUnit == 8) *reinterpret_cast<uint4*>(dst) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
      else if constexpr (kUnit == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(w[p][0], w[p][1]);
      else *dst = w[p][0];
    }
  }

  // raw itself, k-major, to LDS
  __device__ __forceinline__ void store_chain(int set, float* lds) const {
#pragma unroll
    for (int j = 0; j < kUnit; ++j) lds[(k() + j) * kChainStride + row()] = raw[set][j];
  }

  // part p of the MFMA operand of a 32-row tile: 8 k of row `r`
  static __device__ __forceinline__ bf16x8 frag(const uint4* lds, int p, int oct, int r) {
    return __builtin_bit_cast(bf16x8, lds[p * kPartStride + oct * kOctStride + r]);
  }
};

// acc += A B on the fp32 MFMA, which adds its two products one after the other, each with one rounding: every
// element is fma(a[k], b[k], ...) over ascending k, whatever the tile.  Buffers and prefetch as in the kernel below.
template <int TM, int TN, class OpA, class OpB>
__device__ __forceinline__ void chain_product(OpA& opa, OpB& opb, int64_t k_len, int wm0, int wn0, uint4* lds,
                                              floatx16 (&acc)[TM][TN]) {
  const int lrow = threadIdx.x & 31, lk = threadIdx.x >> 5 & 1;
  auto buffer = [&](int b) { return reinterpret_cast<float*>(lds + b * (OpA::kChainLds + OpB::kChainLds)); };
  auto store = [&](int raw_set, float* dst) {
    opa.store_chain(raw_set, dst);
    opb.store_chain(raw_set, dst + 4 * OpA::kChainLds);
  };
  auto multiply = [&](const float* src) {
#pragma unroll
    for (int k0 = 0; k0 < BK; k0 += 2) {
      const float* pa = src + (k0 + lk) * OpA::kChainStride + wm0 + lrow;
      const float* pb = src + 4 * OpA::kChainLds + (k0 + lk) * OpB::kChainStride + wn0 + lrow;
      float a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = pa[32 * i];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = pb[32 * j];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  const int64_t slabs = k_len / BK;  // whole ones
  if (slabs > 0) {
    opa.load(0, 0);
    opb.load(0, 0);
    const int64_t s1 = slabs > 1 ? 1 : 0;
    opa.load(1, s1);
    opb.load(1, s1);
    store(0, buffer(0));
    auto step = [&](auto parity, int64_t s) {
      constexpr int P = decltype(parity)::value;
      __syncthreads();  // buffer P is complete, the other one has been read
      const int64_t s2 = s + 2 < slabs ? s + 2 : slabs - 1;
      opa.load(P, s2);
      opb.load(P, s2);
      multiply(buffer(P));
      store(P ^ 1, buffer(P ^ 1));
    };
    int64_t s = 0;
    for (; s + 2 <= slabs; s += 2) {
      step(std::integral_constant<int, 0>{}, s);
      step(std::integral_constant<int, 1>{}, s + 1);
    }
    if (s < slabs) step(std::integral_constant<int, 0>{}, s);
  }
  if (const int rem = (int)(k_len - slabs * BK); rem > 0) {
    opa.load_partial(0, slabs, rem);
    opb.load_partial(0, slabs, rem);
    __syncthreads();  // the buffers have been read
    store(0, buffer(0));
    __syncthreads();
    multiply(buffer(0));
  }
}

// How a kernel sums up: kLoop over the slabs of bf16 parts; kShallow the same for products of up to kShallowK terms
enum Mode { kLoop, kShallow };
constexpr int kShallowK = 2 * BK;

// Wavefronts per SIMD that the registers have to leave room for: the accumulators of a 128 x 128 tile allow two.  The
// smaller tiles of x^T g would end a few registers above the limit of three (232965 x 602 x 64: 225 us, 254 with two);
// x w fits three by itself and is slower when held to it (198 -> 215 us).
template <int BM, int BN, bool A_KMAJOR>
constexpr int kMinWaves = A_KMAJOR && BM * BN <= 128 * 64 ? 3 : 2;

template <int BM, int BN, int WR, int WC, bool A_KMAJOR, bool B_KCONTIG, bool EPI, Mode MODE>
__global__ __launch_bounds__(64 * WR * WC, (kMinWaves<BM, BN, A_KMAJOR>)) void k_gemm_f32(
    int64_t M, int N, int64_t K, const float* __restrict__ A, int64_t lda,
    const float* __restrict__ B, int64_t ldb, float* __restrict__ C, int64_t ldc,
    int64_t k_per_split, int64_t split_stride, int tiles_m, int tiles_n, int splits, AttnEpilogue epi) {
  constexpr int THREADS = 64 * WR * WC;  // WR x WC wavefronts
  constexpr int WM = BM / WR, WN = BN / WC;
  constexpr int TM = WM / 32, TN = WN / 32;  // MFMA tiles per wavefront
  static_assert(TM >= 1 && TN >= 1, "a wavefront owns at least one MFMA tile");
  using OpA = Operand<BM, THREADS, !A_KMAJOR>;
  using OpB = Operand<BN, THREADS, B_KCONTIG>;
  __shared__ uint4 lds[2][OpA::kLds + OpB::kLds];

  // Workgroups go to the XCDs round-robin.  All tiles along n of a row of tiles (and all tiles of a
  // k range of a split product) run on one XCD, one after the other: they read the same rows.
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int per = splits > 1 ? tiles_m * tiles_n : tiles_n;  // tiles that share operand rows
  const int set = slot / per * kXcds + xcd, in_set = slot % per;
  const int tm = splits > 1 ? in_set / tiles_n : set, tn = in_set % tiles_n, split = splits > 1 ? set : 0;
  if (tm >= tiles_m || split >= splits) return;  // the grid is rounded up to whole XCD rounds

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm0 = wave / WC * WM, wn0 = wave % WC * WN;
  const int64_t m0 = (int64_t)tm * BM;
  const int n0 = tn * BN;
  const int64_t k_begin = (int64_t)split * k_per_split;
  const int64_t k_end = k_begin + k_per_split < K ? k_begin + k_per_split : K;
  const int lrow = lane & 31, lk = lane >> 5;

  OpA opa;
  OpB opb;
  opa.init(A, lda, m0, M, k_begin);
  opb.init(B, ldb, n0, N, k_begin);

  floatx16 acc[TM][TN];
  if constexpr (MODE == kShallow) {
    // Little more than a fetch and a store, so it takes many wavefronts per CU, that is few registers: both slabs at
    // once, one accumulator pair at a time, and the fp32 chain likewise (106 registers for 128 x 64 instead of 164).
    // x w, us, loop -> here (on the fp32 MFMA alone): 232965 x 16 x 64 17.2 -> 15.6 (15.9), x 256 51 -> 41 (45);
    // 100000 x 8 x 64 11.8 -> 9.0 (9.4), x 24 x 128 22.4 -> 16.6 (21.2); 50000 x 12 x 512 32 -> 21 (25).  At two whole
    // slabs they meet: 232965 x 32 x 64 20.1 -> 20.3, x 256 63 -> 60.  GAT forward with 4 heads of 64 from 16 columns,
    // 232965 vertices: 304 -> 247 (251).
    const int k0 = (int)(K < BK ? K : BK), k1 = (int)K - k0;
    if (k0 == BK) {
      opa.load(0, 0);
      opb.load(0, 0);
    } else {
      opa.load_partial(0, 0, k0);
      opb.load_partial(0, 0, k0);
    }
    if (k1 == BK) {
      opa.load(1, 1);
      opb.load(1, 1);
    } else if (k1 > 0) {
      opa.load_partial(1, 1, k1);
      opb.load_partial(1, 1, k1);
    }
    const bool direct = K <= kDirectK;
    float zero = 0.f;
    if (!direct) {
      opa.store(0, kScale, lds[0]);
      opb.store(0, kScale, lds[0] + OpA::kLds);
      if (k1 > 0) {  // the odd slab: negated, as below
        opa.store(1, -kScale, lds[1]);
        opb.store(1, kScale, lds[1] + OpA::kLds);
      }
      __syncthreads();
      auto multiply = [&](int i, int j, const uint4* src) {
        constexpr int pa[6] = {1, 2, 0, 0, 1, 0}, pb[6] = {1, 0, 2, 1, 0, 0};
        bf16x8 a[kParts], b[kParts];
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
          a[p] = OpA::frag(src, p, lk, wm0 + i * 32 + lrow);
          b[p] = OpB::frag(src + OpA::kLds, p, lk, wn0 + j * 32 + lrow);
        }
        floatx16 sum;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[r] = 0.f;
#pragma unroll
        for (int q = 0; q < 6; ++q) sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa[q]], b[pb[q]], sum, 0, 0, 0);
        return sum;
      };
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[i][j] = multiply(i, j, lds[0]);
          if (k1 > 0) acc[i][j] -= multiply(i, j, lds[1]);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            acc[i][j][r] *= 1.f / (kScale * kScale);
            zero = __builtin_fmaf(acc[i][j][r], 0.f, zero);
          }
        }
    }
    if (__syncthreads_or(direct || zero != 0.f)) {
      float* dst[2] = {reinterpret_cast<float*>(lds[0]), reinterpret_cast<float*>(lds[1])};
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (h == 0 || k1 > 0) {
          opa.store_chain(h, dst[h]);
          opb.store_chain(h, dst[h] + 4 * OpA::kChainLds);
        }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          floatx16 chain;
#pragma unroll
          for (int r = 0; r < 16; ++r) chain[r] = 0.f;
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (h == 0 || k1 > 0)
#pragma unroll
              for (int k = lk; k < BK; k += 2)
                chain = __builtin_amdgcn_mfma_f32_32x32x2f32(
                    dst[h][k * OpA::kChainStride + wm0 + i * 32 + lrow],
                    dst[h][4 * OpA::kChainLds + k * OpB::kChainStride + wn0 + j * 32 + lrow], chain, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (direct || !(fabsf(acc[i][j][r]) <= 3.402823466e38f)) acc[i][j][r] = chain[r];
        }
    }
  } else {
    floatx16 part[2][TM][TN];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) part[h][i][j][r] = 0.f;

    // The matrix core cuts its sums off (towards minus infinity) where fp32 arithmetic rounds, which
    // would pull a long sum down.  So A's elements of odd slabs are stored negated and sum up in part[1], those of
    // even slabs in part[0], and what both lose cancels in their difference.  The sign depends on the slab alone: equal
    // rows have equal results wherever they stand.
    auto store = [&](int raw_set, int parity, uint4* dst) {
      opa.store(raw_set, parity ? -kScale : kScale, dst);
      opb.store(raw_set, kScale, dst + OpA::kLds);
    };
    auto multiply = [&](int parity, const uint4* src) {
      constexpr int pa[6] = {1, 2, 0, 0, 1, 0}, pb[6] = {1, 0, 2, 1, 0, 0};  // smallest products first
      bf16x8 a[kParts][TM], b[kParts][TN];
#pragma unroll
      for (int p = 0; p < kParts; ++p) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[p][i] = OpA::frag(src, p, lk, wm0 + i * 32 + lrow);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[p][j] = OpB::frag(src + OpA::kLds, p, lk, wn0 + j * 32 + lrow);
      }
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            part[parity][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa[q]][i], b[pb[q]][j], part[parity][i][j], 0, 0, 0);
    };

    const int64_t slabs = (k_end - k_begin) / BK;  // whole ones
    if (slabs > 0) {
      opa.load(0, 0);
      opb.load(0, 0);
      const int64_t s1 = slabs > 1 ? 1 : 0;
      opa.load(1, s1);
      opb.load(1, s1);
      store(0, 0, lds[0]);
      // slab s, of parity P: its parts are in lds[P], slab s + 1 is in raw[P ^ 1] or on its way, and
      // raw[P] is free for slab s + 2 (past the end: the last slab again, for nothing)
      auto step = [&](auto parity, int64_t s) {
        constexpr int P = decltype(parity)::value;
        __syncthreads();  // lds[P] is complete, lds[P ^ 1] has been read
        const int64_t s2 = s + 2 < slabs ? s + 2 : slabs - 1;
        opa.load(P, s2);
        opb.load(P, s2);
        multiply(P, lds[P]);
        store(P ^ 1, P ^ 1, lds[P ^ 1]);
        // one MFMA, then the vector instructions that fit its time
#pragma unroll
        for (int q = 0; q < 6 * TM * TN; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
        }
      };
      int64_t s = 0;
      for (; s + 2 <= slabs; s += 2) {
        step(std::integral_constant<int, 0>{}, s);
        step(std::integral_constant<int, 1>{}, s + 1);
      }
      if (s < slabs) step(std::integral_constant<int, 0>{}, s);
    }
    const bool direct = K <= kDirectK;
    if (const int rem = (int)(k_end - k_begin - slabs * BK); rem > 0 && !direct) {
      opa.load_partial(0, slabs, rem);
      opb.load_partial(0, slabs, rem);
      const bool odd = slabs & 1;
      __syncthreads();  // the buffers have been read
      store(0, odd, lds[0]);
      __syncthreads();
      if (odd) multiply(1, lds[0]);
      else multiply(0, lds[0]);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = part[0][i][j][r] - part[1][i][j][r];

    // What is not finite, and very short sums, as the fp32 chain gives them.  Element by element: a result depends on
    // its own row and column, not on what else the tile holds.
    float zero = 0.f;  // stays so as long as everything is finite
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc[i][j][r] *= 1.f / (kScale * kScale);
          zero = __builtin_fmaf(acc[i][j][r], 0.f, zero);
        }
    if (__syncthreads_or(direct || zero != 0.f)) {  // uniform over the workgroup; the buffers have been read
      floatx16 chain[TM][TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) chain[i][j][r] = 0.f;
      chain_product(opa, opb, k_end - k_begin, wm0, wn0, lds[0], chain);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (direct || !(fabsf(acc[i][j][r]) <= 3.402823466e38f)) acc[i][j][r] = chain[i][j][r];
    }
  }

  // accumulator layout of the 32x32 tile: register r of lane l holds
  // row 8*(r/4) + 4*(l/32) + r%4, column l%32
  float* Cout = C + (int64_t)split * split_stride;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + j * 32 + lrow;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t m = m0 + wm0 + i * 32 + (r >> 2) * 8 + lk * 4 + (r & 3);
        if (m < M && n < N) Cout[m * ldc + n] = acc[i][j][r];
      }
    }

  if constexpr (EPI) {
    const int F = epi.F, H = epi.H;
    float wl[TN], wr[TN];
    int hd[TN];           // head of the lane's column in tile j; -1: this lane stores nothing
    const bool whole = F > 32 || H == 1;       // all columns of the wavefront belong to one head
    const bool across = H == 1 && WC > 1;      // and so do those of the wavefronts beside it
    const int seg = whole ? 32 : F;            // lanes of a tile that share a head
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + j * 32 + lrow;
      wl[j] = n < N ? epi.a_l[n] : 0.f;  // a_l, a_r are [H, F] = one value per column of C
      wr[j] = n < N ? epi.a_r[n] : 0.f;
      hd[j] = (lrow & (seg - 1)) == 0 && (n < N || across) ? (H == 1 ? 0 : n / F) : -1;
    }
    float* sub = reinterpret_cast<float*>(lds);  // [WC][BM][2]
    if (across) __syncthreads();               // the last slab has been read
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ml = wm0 + i * 32 + (r >> 2) * 8 + lk * 4 + (r & 3);
        const int64_t m = m0 + ml;
        float vl[TN], vr[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          // columns past N hold products of a clamped column, possibly not finite: left out, not times 0
          const bool in = n0 + wn0 + j * 32 + lrow < N;
          vl[j] = in ? wl[j] * acc[i][j][r] : 0.f;
          vr[j] = in ? wr[j] * acc[i][j][r] : 0.f;
        }
        if (whole) {
#pragma unroll
          for (int j = 1; j < TN; ++j) {
            vl[0] += vl[j];
            vr[0] += vr[j];
          }
        }
#pragma unroll
        for (int j = 0; j < (whole ? 1 : TN); ++j) {
          const float sl = segment_sum(vl[j], seg), sr = segment_sum(vr[j], seg);
          if (across) {
            if (lrow == 0) *reinterpret_cast<float2*>(sub + 2 * (wave % WC * BM + ml)) = make_float2(sl, sr);
          } else if (hd[j] >= 0 && m < M) {
            epi.el[m * H + hd[j]] = sl;
            epi.er[m * H + hd[j]] = sr;
          }
        }
      }
    if (across) {
      __syncthreads();
      for (int ml = threadIdx.x; ml < BM; ml += THREADS) {
        if (m0 + ml >= M) break;
        float sl = 0.f, sr = 0.f;
#pragma unroll
        for (int c = 0; c < WC; ++c) {
          sl += sub[2 * (c * BM + ml)];
          sr += sub[2 * (c * BM + ml) + 1];
        }
        epi.el[m0 + ml] = sl;
        epi.er[m0 + ml] = sr;
      }
    }
  }
}

// ---- products with few tiles ---------------------------------------------------------------------
// Where a tile of k_gemm_f32 to a workgroup leaves the chip half empty, its slabs one after the other are what the product takes.  Here a
// workgroup has a tile of 32 rows and deals the slabs out to its wavefronts, W runs of them.  A run's operands, 8 consecutive k
// of a row or column to a lane, come straight from memory into the MFMA's layout and are split there: no LDS and no barrier before the
// end, where the W sums meet in LDS, in the order of k.
struct Parts {
  bf16x8 v[kParts];
};
// scale * raw = h + m + l in bf16
__device__ __forceinline__ Parts split_octet(const float (&raw)[8], float scale) {
  uint32_t w[kParts][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float a = scale * raw[2 * q], b = scale * raw[2 * q + 1];
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
      w[p][q] = pack_bf16(a, b);
      if (p + 1 < kParts) {
        a -= __uint_as_float(w[p][q] << 16);
        b -= __uint_as_float(w[p][q] & 0xffff0000u);
      }
    }
  }
  Parts r;
#pragma unroll
  for (int p = 0; p < kParts; ++p) r.v[p] = __builtin_bit_cast(bf16x8, make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]));
  return r;
}

template <int TN, int W, bool BKC, bool EPI>
__global__ __launch_bounds__(64 * W) void k_gemm_few(int64_t M, int N, int K, const float* __restrict__ A, int64_t lda,
                                                     const float* __restrict__ B, int64_t ldb, float* __restrict__ C,
                                                     int64_t ldc, int tiles_m, AttnEpilogue epi) {
  static_assert(W == 4 || W == 8, "a wavefront closes 16 / W registers of the tile");
  constexpr int R = 16 / W;
  __shared__ float l_sum[W][TN][16][64];
  const int lane = threadIdx.x & 63, lrow = lane & 31, lk = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t m0 = (int64_t)(blockIdx.x % tiles_m) * 32;
  const int n0 = (int)(blockIdx.x / tiles_m) * 32 * TN;
  const int64_t row = m0 + lrow < M ? m0 + lrow : M - 1;  // past the matrix: its last row, for nothing
  int col[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) col[j] = min(n0 + 32 * j + lrow, N - 1);

  typedef float vec4 __attribute__((ext_vector_type(4), aligned(4)));
  const float* pa = A + row * lda + 8 * lk;
  auto load8 = [&](float (&raw)[8], const float* p, int k) {  // p: this lane's k of slab k / BK
    if (k + BK <= K) {
      const vec4 lo = *reinterpret_cast<const vec4*>(p), hi = *reinterpret_cast<const vec4*>(p + 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) raw[q] = lo[q], raw[4 + q] = hi[q];
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) raw[q] = k + 8 * lk + q < K ? p[q] : 0.f;
    }
  };
  float ra[2][8], rb[2][TN][8];
  auto load = [&](auto slot, int s) {
    constexpr int S = decltype(slot)::value;
    const int k = BK * s;
    load8(ra[S], pa + k, k);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if constexpr (BKC) {
        load8(rb[S][j], B + col[j] * ldb + k + 8 * lk, k);
      } else {
        const float* p = B + (int64_t)(k + 8 * lk) * ldb + col[j];
        if (k + BK <= K) {
#pragma unroll
          for (int q = 0; q < 8; ++q) rb[S][j][q] = p[q * ldb];
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q) rb[S][j][q] = k + 8 * lk + q < K ? p[q * ldb] : 0.f;
        }
      }
    }
  };
  floatx16 part[2][TN];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[h][j][r] = 0.f;
  const int slabs = (K + BK - 1) / BK, per = (slabs + W - 1) / W;
  const int s0 = min(w * per, slabs), s1 = min(s0 + per, slabs);
  // The product's odd slabs are summed negated, as in k_gemm_f32: in part[1], or in part[0] of a run that starts with one.  (Were
  // it a run's odd slabs, runs of one slab would all lose to the same side: a GMM layer of 8104 vertices, 114 -> 3 x 20, then is off by 3.4e-7, not 1.4e-7.)
  const bool odd_first = (s0 & 1) != 0;
  auto step = [&](auto slot, int s) {
    constexpr int S = decltype(slot)::value;
    constexpr int ia[6] = {1, 2, 0, 0, 1, 0}, ib[6] = {1, 0, 2, 1, 0, 0};  // smallest products first
    const Parts a = split_octet(ra[S], (S != 0) != odd_first ? -kScale : kScale);
    Parts b[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = split_octet(rb[S][j], kScale);
    if (s + 2 < s1) load(slot, s + 2);
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        part[S][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v[ia[q]], b[j].v[ib[q]], part[S][j], 0, 0, 0);
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  if (s0 < s1) load(even, s0);
  if (s0 + 1 < s1) load(odd, s0 + 1);
  for (int s = s0; s < s1; s += 2) {
    step(even, s);
    if (s + 1 < s1) step(odd, s + 1);
  }
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) l_sum[w][j][r][lane] = odd_first ? part[1][j][r] - part[0][j][r] : part[0][j][r] - part[1][j][r];
  __syncthreads();

  // wavefront w closes registers R w .. of the tile, which hold rows 8 (r / 4) + 4 lk + r % 4
  float acc[TN][R];
  float zero = 0.f;  // stays so as long as everything is finite
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < R; ++i) {
      float sum = l_sum[0][j][R * w + i][lane];
#pragma unroll
      for (int q = 1; q < W; ++q) sum += l_sum[q][j][R * w + i][lane];
      acc[j][i] = sum * (1.f / (kScale * kScale));
      zero = __builtin_fmaf(acc[j][i], 0.f, zero);
    }
  if (__any(zero != 0.f)) {  // what is not finite, as the fp32 chain gives it
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      floatx16 chain;
#pragma unroll
      for (int r = 0; r < 16; ++r) chain[r] = 0.f;
      for (int k0 = 0; k0 < K; k0 += 2) {
        const int k = k0 + lk;
        const float a = k < K ? A[row * lda + k] : 0.f;
        const float b = k < K ? B[BKC ? col[j] * ldb + k : k * ldb + col[j]] : 0.f;
        chain = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, chain, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (r / R == w && !(fabsf(acc[j][r % R]) <= 3.402823466e38f)) acc[j][r % R] = chain[r];
    }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int r = R * w + i, n = n0 + 32 * j + lrow;
      const int64_t m = m0 + (r >> 2) * 8 + lk * 4 + (r & 3);
      if (m < M && n < N) C[m * ldc + n] = acc[j][i];
    }
  if constexpr (EPI) {  // el, er as in k_gemm_f32; the wavefront has all columns of its rows
    const int F = epi.F, H = epi.H;
    const bool whole = F > 32 || H == 1;  // all of the tile's columns belong to one head
    const int seg = whole ? 32 : F;
    float wl[TN], wr[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + 32 * j + lrow;
      wl[j] = n < N ? epi.a_l[n] : 0.f;
      wr[j] = n < N ? epi.a_r[n] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int r = R * w + i;
      const int64_t m = m0 + (r >> 2) * 8 + lk * 4 + (r & 3);
      float vl[TN], vr[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const bool in = n0 + 32 * j + lrow < N;  // columns past N hold products of a clamped one
        vl[j] = in ? wl[j] * acc[j][i] : 0.f;
        vr[j] = in ? wr[j] * acc[j][i] : 0.f;
      }
      if (whole) {
#pragma unroll
        for (int j = 1; j < TN; ++j) {
          vl[0] += vl[j];
          vr[0] += vr[j];
        }
      }
#pragma unroll
      for (int j = 0; j < (whole ? 1 : TN); ++j) {
        const float sl = segment_sum(vl[j], seg), sr = segment_sum(vr[j], seg);
        const int n = n0 + 32 * j + lrow;
        if ((lrow & (seg - 1)) == 0 && n < N && m < M) {
          const int h = H == 1 ? 0 : n / F;
          epi.el[m * H + h] = sl;
          epi.er[m * H + h] = sr;
        }
      }
    }
  }
}


// c = a b, a [M,K], b [K,N], every element fma(a[k], b[k], ...) over ascending k: the fp32 MFMA adds its two products one
// after the other, each with one rounding.  The MFMAs (64 cycles each) are busy 60 % of the time; while one wavefront issues a slab's
// worth of them, the vector instructions of the others on its SIMD wait, so the loop keeps those few: uniform addresses,
// one LDS buffer, the fetch one slab ahead, vectors of 2 floats of A and VB of B (VB = 4 where N and ldb are multiples of
// 4), three wavefronts per SIMD.  chain_product above, made for the recomputation (two buffers, tile indices in vector
// registers), takes 12 % longer: 65536 x 128 x 512 93 us here and 104 there, 131072 x 320 x 128 121 and 137.
template <int BM, int BN, int VB>
__global__ __launch_bounds__(256, 3) void k_chain_f32(int64_t M, int N, int64_t K, const float* __restrict__ A,
                                                      int64_t lda, const float* __restrict__ B, int64_t ldb,
                                                      float* __restrict__ C, int64_t ldc) {
  constexpr int TM = BM / 64, TN = BN / 64, VA = 2, PAD = 4;
  constexpr int NA = BM * BK / 256 / VA, NB = BN * BK / 256 / VB;  // loads per thread and slab
  __shared__ __align__(16) float as[BK][BM + PAD], bs[BK][BN + PAD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lrow = lane & 31, lk = lane >> 5;
  const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);
  const int64_t m0 = (int64_t)blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // load i of a thread: VA consecutive k of a row of A, VB consecutive columns of a row of B; rows and columns past the
  // matrix are clamped to the last ones (their products are not stored)
  auto a_row = [](int i) { return (int)(threadIdx.x + 256 * i) / (BK / VA); };
  auto a_k = [](int i) { return VA * (int)((threadIdx.x + 256 * i) % (BK / VA)); };
  auto b_k = [](int i) { return (int)(threadIdx.x + 256 * i) / (BN / VB); };
  auto b_col = [](int i) { return VB * (int)((threadIdx.x + 256 * i) % (BN / VB)); };
  typedef float vec_a __attribute__((ext_vector_type(VA), aligned(4)));
  typedef float vec_b __attribute__((ext_vector_type(VB), aligned(4)));
  uint32_t offa[NA], offb[NB];
  float ra[NA][VA], rb[NB][VB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int64_t r = (m0 + a_row(i) < M ? m0 + a_row(i) : M - 1) - m0;
    offa[i] = (uint32_t)(r * lda + a_k(i));
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int64_t c = (n0 + b_col(i) <= N - VB ? n0 + b_col(i) : N - VB) - n0;
    offb[i] = (uint32_t)(b_k(i) * ldb + c);
  }
  const float* pa = A + m0 * lda;
  const float* pb = B + n0;
  const int64_t step_b = BK * ldb;
  auto load = [&](int64_t k0) {
    const int64_t rem = K - k0;
    if (rem >= BK) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const vec_a v = *reinterpret_cast<const vec_a*>(pa + offa[i]);
#pragma unroll
        for (int c = 0; c < VA; ++c) ra[i][c] = v[c];
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if constexpr (VB == 1) rb[i][0] = pb[offb[i]];
        else {
          const vec_b v = *reinterpret_cast<const vec_b*>(pb + offb[i]);
#pragma unroll
          for (int c = 0; c < VB; ++c) rb[i][c] = v[c];
        }
      }
    } else {  // the last, partial slab: element by element
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int c = 0; c < VA; ++c) ra[i][c] = a_k(i) + c < rem ? pa[offa[i] + c] : 0.f;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int c = 0; c < VB; ++c) rb[i][c] = b_k(i) < rem ? pb[offb[i] + c] : 0.f;
    }
    pa += BK;
    pb += step_b;
  };
  load(0);
  for (int64_t k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int c = 0; c < VA; ++c) as[a_k(i) + c][a_row(i)] = ra[i][c];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      float* dst = &bs[b_k(i)][b_col(i)];
      if constexpr (VB == 4) *reinterpret_cast<float4*>(dst) = make_float4(rb[i][0], rb[i][1], rb[i][2], rb[i][3]);
      else *dst = rb[i][0];
    }
    __syncthreads();
    if (k0 + BK < K) load(k0 + BK);
#pragma unroll
    for (int ks = 0; ks < BK / 2; ++ks) {
      const int k = ks * 2 + lk;
      float a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = as[k][wm0 + i * 32 + lrow];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = bs[k][wn0 + j * 32 + lrow];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + j * 32 + lrow;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t m = m0 + wm0 + i * 32 + (r >> 2) * 8 + lk * 4 + (r & 3);
        if (m < M && n < N) C[m * ldc + n] = acc[i][j][r];
      }
    }
}

__global__ __launch_bounds__(256) void k_sum_partials(PartialSum j) { sum_partials_thin(j, blockIdx.x, threadIdx.x); }
__global__ __launch_bounds__(256) void k_sum_partials_wide(PartialSum j, int chunk) {
  __shared__ float sub[8][32];
  sum_partials_wide(j, blockIdx.x, blockIdx.y, chunk, threadIdx.x, sub);
}
// Two sums in one launch, a's workgroups first: either is some 5 us of memory latency on a few workgroups.  Training pass, a launch each ->
// this, us: GAT, 20 000 vertices, 10^5 edges, 500 -> 8 x 8 125.9 -> 121.4, 1856, 1.3 10^5, 16 -> 1 x 64 57.6 -> 52.9; GMM (with the last
// step of the parameters' gradients, too) 100 000, 2 10^6, 64 -> 3 x 64 291.5 -> 285.8, 17 036, 1.3 10^5, 22 -> 4 x 32 68.4 -> 65.1.
__global__ __launch_bounds__(256) void k_sum_partials_two(PartialSum a, PartialSum b, unsigned blocks_a, bool wide_a, bool wide_b) {
  __shared__ float sub[8][32];
  auto sum = [&](const PartialSum& j, unsigned block, bool wide) {  // uniform
    if (wide) sum_partials_wide(j, block, 0, j.parts, threadIdx.x, sub);
    else sum_partials_thin(j, block, threadIdx.x);
  };
  // not one call for the one or the other: the compiler would copy both descriptions to scratch memory, and index there
  if (blockIdx.x < blocks_a) sum(a, blockIdx.x, wide_a);
  else sum(b, blockIdx.x - blocks_a, wide_b);
}

gnn_status_t sum_partials_of(const PartialSum& j, hipStream_t s) {
  if (j.count <= 0) return GNN_OK;
  if (sums_wide(j)) k_sum_partials_wide<<<dim3(sum_blocks(j), 1), 256, 0, s>>>(j, j.parts);
  else k_sum_partials<<<sum_blocks(j), 256, 0, s>>>(j);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

gnn_status_t sum_partials_strided(int64_t count, int parts, const float* partials, int64_t stride,
                                  float* out, hipStream_t s) {
  return sum_partials_of({count, stride, parts, partials, out}, s);
}

// partials is [parts][2][count]: the first halves are summed into out0, the second into out1
gnn_status_t sum_partials_pair(int64_t count, int parts, const float* partials, float* out0, float* out1,
                               hipStream_t s) {
  return sum_partials_of({2 * count, 2 * count, parts, partials, out0, out1, count}, s);
}

gnn_status_t sum_partials_two(const PartialSum& a, const PartialSum& b, hipStream_t s) {
  const unsigned blocks_a = sum_blocks(a);
  k_sum_partials_two<<<blocks_a + sum_blocks(b), 256, 0, s>>>(a, b, blocks_a, sums_wide(a), sums_wide(b));
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

gnn_status_t sum_partials(int64_t count, int parts, const float* partials, float* out, hipStream_t s) {
  return sum_partials_strided(count, parts, partials, count, out, s);
}

// Two levels for very many parts: ranges of kSumChunk parts into `scratch`
// (sum_partials_scratch_rows(parts) rows of `count` floats), then those rows into `out`.
int sum_partials_scratch_rows(int parts) { return (int)cdiv(parts, kSumChunk); }

gnn_status_t sum_partials_ranges(PartialSum& j, float* scratch, hipStream_t s) {
  const int rows = sum_partials_scratch_rows(j.parts);
  if (j.count <= 0 || rows <= 1) return GNN_OK;
  k_sum_partials_wide<<<dim3((unsigned)cdiv(j.count, 32), (unsigned)rows), 256, 0, s>>>({j.count, j.stride, j.parts, j.partials, scratch},
                                                                                       kSumChunk);
  GNN_LAUNCH_CHECK();
  j.partials = scratch;
  j.parts = rows;
  j.stride = j.count;
  return GNN_OK;
}

gnn_status_t sum_partials_two_level(int64_t count, int parts, const float* partials, float* scratch,
                                    float* out, hipStream_t s) {
  PartialSum j{count, count, parts, partials, out};
  GNN_TRY(sum_partials_ranges(j, scratch, s));
  return sum_partials_of(j, s);
}

// ---- choice of the tile -----------------------------------------------------------------
// Measured (x w, us; the fp32 MFMA on 128-row tiles before -> now): 232965 x 602 x 256 638 -> 470,
// x 128 346 -> 262, x 64 202 -> 200, x 32 209 -> 180; 232965 x 1024 x 1024 3965 -> 2600; 20000 x 500 x 64
// 30 -> 22; 65536 x 128 x 512 84 -> 65.  The wide products keep the matrix cores busy 36 to 45 %
// of the time, with 3/8 of the cycles that the fp32 MFMA would need; the narrow ones are bound by the fetch
// of A, whose rows of 602 floats straddle cache lines (608 floats: 160 us at x 64).
//
// 128 output columns per tile unless the last such tile would be at least half empty; 32 for the
// narrowest products
static int gemm_tile_cols(int N) {
  if (N <= 32) return 32;
  if (N <= 64) return 64;
  const int waste = (N + 127) / 128 * 128 - N;
  return waste >= 64 ? 64 : 128;
}

// 128 rows per tile; 64 where there are no more, or where 128 would leave a CU fewer than two tiles to
// overlap (20000 x 500 x 64: 22 us against 28 us; 32768 x 64 x 128: 10.5 against 13.8; with 8 tiles per CU,
// 65536 x 128 x 512, 128 rows win: 67 us against 79 us)
static int gemm_tile_rows(int64_t M, int N, int bn, int split_k) {
  if (bn < 64) return 128;
  return M <= 64 || (split_k == 1 && cdiv(M, 128) * cdiv(N, bn) < 512) ? 64 : 128;
}

// Parts of K that different workgroups sum: what fills the chip once with the three workgroups a CU
// holds, at least 128 of K each
int gemm_pick_split_k(int64_t M, int N, int64_t K) {
  const int64_t tiles = cdiv(M, 128) * cdiv(N, gemm_tile_cols(N));
  if (tiles >= 128 || K < kGemmSplitTerms) return 1;
  int64_t want = 768 / tiles;
  const int64_t max_by_k = K / 128;
  if (want > max_by_k) want = max_by_k;
  if (want > 512) want = 512;
  return want < 1 ? 1 : (int)want;
}

template <int BM, int BN, int WR, int WC, bool AK, bool BKC, bool EPI, Mode MODE>
static gnn_status_t launch(int64_t M, int N, int64_t K, const float* a, int64_t lda, const float* b, int64_t ldb,
                           float* c, int64_t ldc, int split_k, float* partials, const AttnEpilogue& epi,
                           hipStream_t s) {
  // A launch may not have 2^32 threads, so products of very many rows go out in pieces of whole tiles (one up to 2^30 rows
  // of 128-row tiles).  A split product has at most 512 x 128 tiles.
  constexpr int64_t kMaxGrid = (int64_t)1 << 23;
  const int64_t tn = cdiv(N, BN);
  GNN_REQUIRE(tn <= kMaxGrid / kXcds, GNN_ERR_UNSUPPORTED, "gemm_f32: grid too large");
  const int64_t max_rows = split_k > 1 ? M : kMaxGrid / (kXcds * tn) * kXcds * BM;
  const int64_t kps = split_k > 1 ? cdiv(cdiv(K, split_k), BK) * BK : K;
  ProfScope p(EPI ? "gemm_f32_mfma_attn" : split_k > 1 ? "gemm_f32_mfma_splitk" : "gemm_f32_mfma", s);
  for (int64_t m0 = 0; m0 < M; m0 += max_rows) {
    const int64_t rows = M - m0 < max_rows ? M - m0 : max_rows, tm = cdiv(rows, BM);
    // workgroups: whole rounds over the XCDs of the sets of tiles that share rows
    const int64_t sets = split_k > 1 ? split_k : tm, per = split_k > 1 ? tm * tn : tn;
    const int64_t grid = cdiv(sets, kXcds) * kXcds * per;
    GNN_REQUIRE(grid <= kMaxGrid, GNN_ERR_UNSUPPORTED, "gemm_f32: grid too large");
    AttnEpilogue piece = epi;
    if (EPI) {
      piece.el += m0 * epi.H;
      piece.er += m0 * epi.H;
    }
    float* out = split_k > 1 ? partials : c + m0 * ldc;
    const int64_t ldo = split_k > 1 ? N : ldc;
    k_gemm_f32<BM, BN, WR, WC, AK, BKC, EPI, MODE><<<(unsigned)grid, 64 * WR * WC, 0, s>>>(
        rows, N, K, a + (AK ? m0 : m0 * lda), lda, b, ldb, out, ldo, kps, M * (int64_t)N, (int)tm, (int)tn, split_k, piece);
    GNN_LAUNCH_CHECK();
  }
  return GNN_OK;
}

template <bool AK, bool BKC, bool EPI, Mode MODE>
static gnn_status_t launch_tile(int64_t M, int N, int64_t K, const float* a, int64_t lda, const float* b, int64_t ldb,
                                float* c, int64_t ldc, int split_k, float* partials, const AttnEpilogue& epi,
                                hipStream_t s) {
  // The shallow product in 128-column tiles leaves two wavefronts per SIMD, so it takes 64 columns (232965 x 16 x 256:
  // 41 us against 50), with an epilogue over heads of 64 columns all of them in one wavefront; only one head of more than
  // 64 columns needs the wide tile.
  const int bn = MODE == kShallow && N > 32 && (epi.F <= 32 || epi.H > 1) ? 64 : gemm_tile_cols(N), bm = gemm_tile_rows(M, N, bn, split_k);
#define GNN_GEMM_TILE(...) \
  return launch<__VA_ARGS__, AK, BKC, EPI, MODE>(M, N, K, a, lda, b, ldb, c, ldc, split_k, partials, epi, s)
  if (bn == 32) GNN_GEMM_TILE(128, 32, 4, 1);
  if constexpr (MODE == kShallow && EPI) {
    if (bn == 64 && epi.H > 1 && epi.F == 64) GNN_GEMM_TILE(128, 64, 4, 1);
  }
  if (bn == 64 && bm == 64) GNN_GEMM_TILE(64, 64, 2, 2);
  if (bn == 64) GNN_GEMM_TILE(128, 64, 2, 2);
  if (bm == 64) GNN_GEMM_TILE(64, 128, 2, 2);
  GNN_GEMM_TILE(128, 128, 2, 2);
#undef GNN_GEMM_TILE
}

template <int TN, int W, bool BKC, bool EPI>
static gnn_status_t launch_few_tile(int64_t M, int N, int64_t K, const float* a, int64_t lda, const float* b, int64_t ldb,
                                    float* c, int64_t ldc, const AttnEpilogue& epi, hipStream_t s) {
  const int64_t tm = cdiv(M, 32), tn = cdiv(N, 32 * TN);
  ProfScope p(EPI ? "gemm_f32_mfma_attn" : "gemm_f32_mfma", s);
  k_gemm_few<TN, W, BKC, EPI><<<(unsigned)(tm * tn), 64 * W, 0, s>>>(M, N, (int)K, a, lda, b, ldb, c, ldc, (int)tm, epi);
  GNN_LAUNCH_CHECK();
  return GNN_OK;
}

// Up to two tiles of 32 x 64 to a CU; below one, twice as many wavefronts to a tile, and tiles half as wide where those are
// no more than the CUs.  x w, us, k_gemm_f32 -> here: 2000 x 500 x 64 15.4 -> 6.4, 8000 17.5 -> 10.4, 16384 (512 tiles) 19.3 -> 18.0, 20000
// (625) 22.6 against 24.8; 2000 x 602 x 256 25.3 -> 11.7, 5000 (628) 27.3 against 28.2; 8000 x 256 x 32 10.6 -> 5.4; 16384 x 64 x 64
// 6.2 -> 5.6, 32768 7.5 against 9.3.  Its sums are shorter: error against 64 bits, 2-norm, 1000 x 65 x 33 8.2e-8 -> 5.6e-8,
// 5000 x 602 x 32 2.6e-7 -> 1.0e-7.
constexpr int kFewTilesPerCu = 2;
bool gemm_has_few_tiles(int64_t M, int N, int64_t K) {
  return K > kShallowK && K < (1 << 24) && cdiv(M, 32) * cdiv(N, 64) <= (int64_t)kFewTilesPerCu * device_cu_count();
}

// Where K can be split as well.  A tile's slabs are a fixed number of wavefronts' work, so long sums are for parts of K on the whole chip and
// a launch that adds them up; most tiles to that work have a chip that one round of them nearly fills, fewest one that goes for a second
// with narrow rows.  GAT layer on loops, K split | slabs dealt out, us: 100 rows, 8 x 8, 1433 terms 18.3 | 15.4, 2048 16.7 | 18.6, 60 000 28.5 | 335;
// 2000, 8 x 8, 1433 20.6 | 16.2, 3703 26.6 | 31.7; 6144, 8 x 8, 2048 31.7 | 31.0, 3703 41.4 | 48.6, 2 x 64 (384 tiles), 1433 51.0 | 39.6, 2048
// 47.7 | 50.1; 2000, 4 x 64 (252 tiles), 3703 52.3 | 49.6, 8192 76.8 | 93.5; 8000, 1 x 16 (250), 3703 43.8 | 31.5, 8192 96.6 | 64.2, 8 x 8 57.9 |
// 50.3, 103 | 99; 12 000, 8 x 8 (375), 602 38.4 | 27.9, 1433 40.6 | 44.8, 3703 63.1 | 88.2.
bool gemm_few_or_split(int64_t M, int N, int64_t K) {
  if (!gemm_has_few_tiles(M, N, K)) return false;
  const int64_t tiles = cdiv(M, 32) * cdiv(N, 64), cus = device_cu_count();
  if (tiles <= cus && 8 * tiles > 7 * cus) return N <= 64 || K <= 4096;
  return K <= (tiles > cus && N <= 64 ? 1024 : 1792);
}

template <bool BKC, bool EPI>
static gnn_status_t launch_few(int64_t M, int N, int64_t K, const float* a, int64_t lda, const float* b, int64_t ldb,
                               float* c, int64_t ldc, const AttnEpilogue& epi, hipStream_t s) {
  const int64_t tm = cdiv(M, 32), cus = device_cu_count();
  // attention halves: all columns of a head are one wavefront's
  const bool wide = EPI && N > 32 && (epi.H == 1 || epi.F == 64);
  const int tn = N <= 32 || (!wide && tm * cdiv(N, 32) <= cus) ? 1 : 2;
  const bool many = tm * cdiv(N, 32 * tn) <= cus && K > 6 * BK;
#define GNN_FEW(TN_, W_) return launch_few_tile<TN_, W_, BKC, EPI>(M, N, K, a, lda, b, ldb, c, ldc, epi, s)
  if (tn == 1 && many) GNN_FEW(1, 8);
  if (tn == 1) GNN_FEW(1, 4);
  if (many) GNN_FEW(2, 8);
  GNN_FEW(2, 4);
#undef GNN_FEW
}

template <int BM, int BN, int VB>
static gnn_status_t launch_chain_tile(int64_t M, int N, int64_t K, const float* a, int64_t lda, const float* b, int64_t ldb,
                                      float* c, int64_t ldc, hipStream_t s) {
  // rows and columns of tiles in pieces, so that a launch stays below 2^32 threads along x and 2^16 workgroups along y
  constexpr int64_t kMaxRows = (int64_t)BM << 23, kMaxCols = (int64_t)BN << 15;
  ProfScope p("gemm_f32_chain", s);
  for (int64_t m0 = 0; m0 < M; m0 += kMaxRows)
    for (int64_t n0 = 0; n0 < N; n0 += kMaxCols) {
      const int64_t rows = std::min(M - m0, kMaxRows);
      const int cols = (int)std::min(N - n0, kMaxCols);
      k_chain_f32<BM, BN, VB><<<dim3((unsigned)cdiv(rows, BM), (unsigned)cdiv(cols, BN)), 256, 0, s>>>(
          rows, cols, K, a + m0 * lda, lda, b + n0, ldb, c + m0 * ldc + n0, ldc);
      GNN_LAUNCH_CHECK();
    }
  return GNN_OK;
}

static gnn_status_t launch_chain(int64_t M, int N, int64_t K, const float* a, int64_t lda, const float* b, int64_t ldb,
                                 float* c, int64_t ldc, hipStream_t s) {
  const int bn = gemm_tile_cols(N) == 128 ? 128 : 64, bm = gemm_tile_rows(M, N, bn, 1);
  const bool vec = N % 4 == 0 && ldb % 4 == 0;
#define GNN_CHAIN_TILE(BM_, BN_)                                                                 \
  return vec ? launch_chain_tile<BM_, BN_, 4>(M, N, K, a, lda, b, ldb, c, ldc, s)               \
             : launch_chain_tile<BM_, BN_, 1>(M, N, K, a, lda, b, ldb, c, ldc, s)
  if (bn == 64 && bm == 64) GNN_CHAIN_TILE(64, 64);
  if (bn == 64) GNN_CHAIN_TILE(128, 64);
  if (bm == 64) GNN_CHAIN_TILE(64, 128);
  GNN_CHAIN_TILE(128, 128);
#undef GNN_CHAIN_TILE
}

gnn_status_t gemm_f32(int64_t M, int N, int64_t K, const float* a, int64_t lda, bool a_kmajor,
                      const float* b, int64_t ldb, bool b_kcontig, float* c, int64_t ldc,
                      int split_k, float* partials, hipStream_t s) {
  if (M <= 0 || N <= 0) return GNN_OK;
  GNN_REQUIRE(K > 0, GNN_ERR_INVALID_ARG, "gemm_f32: K must be positive");
  GNN_REQUIRE(lda > 0 && ldb > 0 && lda < (1 << 24) && ldb < (1 << 24), GNN_ERR_UNSUPPORTED,
              "gemm_f32: leading dimensions must be below 2^24 (32-bit tile offsets)");
  GNN_REQUIRE(cdiv(M, 32) < (int64_t)INT32_MAX && split_k >= 1 && split_k <= 65535,
              GNN_ERR_UNSUPPORTED, "gemm_f32: grid too large");
  GNN_REQUIRE(split_k == 1 || partials != nullptr, GNN_ERR_INVALID_ARG,
              "gemm_f32: split-K without a partials buffer");
  GNN_REQUIRE(split_k == 1 || ldc == N, GNN_ERR_INVALID_ARG,
              "gemm_f32: split-K needs a dense output (ldc == N)");
  const AttnEpilogue none{nullptr, nullptr, nullptr, nullptr, 0, 0};
  const bool shallow = K <= kShallowK && split_k == 1;
  if (!a_kmajor && split_k == 1 && gemm_has_few_tiles(M, N, K))
    return b_kcontig ? launch_few<true, false>(M, N, K, a, lda, b, ldb, c, ldc, none, s)
                     : launch_few<false, false>(M, N, K, a, lda, b, ldb, c, ldc, none, s);
#define GNN_GEMM_RUN(...) \
  GNN_TRY((launch_tile<__VA_ARGS__>(M, N, K, a, lda, b, ldb, c, ldc, split_k, partials, none, s)))
  if (a_kmajor) {
    if (b_kcontig) GNN_GEMM_RUN(true, true, false, kLoop);
    else GNN_GEMM_RUN(true, false, false, kLoop);
  } else if (b_kcontig) {
    if (shallow) GNN_GEMM_RUN(false, true, false, kShallow);
    else GNN_GEMM_RUN(false, true, false, kLoop);
  } else {
    if (shallow && K <= kDirectK) return launch_chain(M, N, K, a, lda, b, ldb, c, ldc, s);
    if (shallow) GNN_GEMM_RUN(false, false, false, kShallow);
    else GNN_GEMM_RUN(false, false, false, kLoop);
  }
#undef GNN_GEMM_RUN
  if (split_k == 1 || c == nullptr) return GNN_OK;
  ProfScope p("gemm_sum_partials", s);
  return sum_partials(M * (int64_t)N, split_k, partials, c, s);
}

gnn_status_t gemm_f32_chain(int64_t M, int N, int64_t K, const float* a, int64_t lda, const float* b, int64_t ldb,
                            float* c, int64_t ldc, hipStream_t s) {
  if (M <= 0 || N <= 0) return GNN_OK;
  GNN_REQUIRE(K > 0, GNN_ERR_INVALID_ARG, "gemm_f32_chain: K must be positive");
  GNN_REQUIRE(lda > 0 && ldb > 0 && lda < (1 << 24) && ldb < (1 << 24) && cdiv(M, 32) < (int64_t)INT32_MAX,
              GNN_ERR_UNSUPPORTED, "gemm_f32_chain: sizes out of range");
  return launch_chain(M, N, K, a, lda, b, ldb, c, ldc, s);
}

// z = x w with el, er from the epilogue; only for shapes gemm_attn_epilogue_ok() accepts: heads inside
// one 32-column MFMA tile, heads that are the 64 columns of a wavefront, or one head inside a tile of C
bool gemm_attn_epilogue_ok(int heads, int f) {
  const int N = heads * f;
  if (f == 4 || f == 8 || f == 16 || f == 32) return true;
  if (heads == 1) return N <= gemm_tile_cols(N);
  return f == 64 && gemm_tile_cols(N) == 128;
}

gnn_status_t gemm_f32_attn(int64_t M, int heads, int f, int64_t K, const float* x, const float* w,
                           const float* a_l, const float* a_r, float* z, float* el, float* er,
                           hipStream_t s) {
  const int N = heads * f;
  if (M <= 0) return GNN_OK;
  GNN_REQUIRE(gemm_attn_epilogue_ok(heads, f), GNN_ERR_UNSUPPORTED, "gemm_f32_attn: unsupported head width");
  GNN_REQUIRE(K > 0 && K < (1 << 24) && N < (1 << 24) && cdiv(M, 32) < (int64_t)INT32_MAX, GNN_ERR_UNSUPPORTED,
              "gemm_f32_attn: sizes out of range");
  const AttnEpilogue epi{a_l, a_r, el, er, heads, f};
  if (gemm_has_few_tiles(M, N, K) && (heads > 1 || N <= 64)) return launch_few<false, true>(M, N, K, x, K, w, N, z, N, epi, s);
  if (K <= kShallowK) return launch_tile<false, false, true, kShallow>(M, N, K, x, K, w, N, z, N, 1, nullptr, epi, s);
  return launch_tile<false, false, true, kLoop>(M, N, K, x, K, w, N, z, N, 1, nullptr, epi, s);
}

}  // namespace gnn

using namespace gnn;

extern "C" gnn_status_t gnn_linear_fwd(int64_t n, int fin, int fout, const float* x, const float* w,
                                       float* y, void* stream) {
  clear_error();
  GNN_REQUIRE(n >= 0 && fin > 0 && fout > 0, GNN_ERR_INVALID_ARG, "gnn_linear_fwd: bad sizes");
  if (n == 0) return GNN_OK;
  GNN_REQUIRE(x && w && y, GNN_ERR_INVALID_ARG, "gnn_linear_fwd: null pointer");
  return gemm_f32(n, fout, fin, x, fin, false, w, fout, false, y, fout, 1, nullptr,
                  static_cast<hipStream_t>(stream));
}
