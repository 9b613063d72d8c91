// One layer of the forward pass in one kernel: aggregation, dense layer, bias and ReLU.
//
//   y = x W_self + m W_neigh + b (+ ReLU), m_i = mean / sum of x[src] over row i of the block (GCN: y = m W + b, m_i the
//   mean over the row itself and its sources).
//
// A workgroup makes 16 or 32 rows by 64 to 256 columns of y.  It walks the input columns in chunks: the chunk of both operands is put
// together in LDS (16 bytes per lane; a row's sources are added in edge order) and multiplied with the chunk's rows of the weights, a wavefront
// making its columns of all or half of the rows.
//
// The products run on the bf16 matrix instructions (v_mfma_f32_16x16x32_bf16, fp32 accumulators): an fp32 number is the sum
// of three bf16 numbers, h + m + l, without a remainder (8 + 8 + 8 bits, each part the rest rounded to nearest: |m| <= 2^-8 |x|,
// |l| <= 2^-17 |x|), and of the nine products of two such sums all but l l, which is below 2^-33 of the product, are taken.
// The instruction adds its 32 products to the accumulator without rounding to nearest (a product by itself came out up to
// 2^-23 too small), so h h, whose products are whole numbers of 16 bits, is summed apart from the other seven, and the two sums
// meet in an fp32 addition: one product by itself then has the rounding of an fp32 product (1.004 x 2^-24 at most, seen over
// 10^6; with the six largest products in one accumulator it was 2.6 x 2^-24).  32 products are added at a time where the fp32
// instruction rounds after every four.  Root mean square of the error over the sum of magnitudes, in 2^-24, these kernels / the
// fp32 ones: N(0,1) x Glorot, 4 columns 0.31 / 0.39, 32 0.14 / 0.32, 602 0.08 / 0.31; U[1,2) 0.66 / 0.72, 0.72 / 1.21, 1.64 / 4.5.
// Only where all but a few of a long contraction's products are zero is it larger (three of 602: 0.72 / 0.64), because a step of
// 32 with one product in it is rounded twice.  Eight bf16 instructions take half of the matrix pipe's time of the eight fp32 ones
// they stand for.
//   Numbers that the parts cannot hold (infinities, NaN, magnitudes that round up to infinity in bf16) leave infinities or
// NaN in the accumulators they touch, and nothing else but a true overflow does.  A workgroup that finds one in its tile
// makes the tile again with the fp32 instructions.
#include <type_traits>
#include "dci_internal.h"
#include "dci_parts.h"

namespace dci {

__device__ __forceinline__ f32x4 load4(const float* p) {
  typedef __attribute__((address_space(1))) const f32x4_u* g4;
  return *(g4)(p);
}

constexpr float kMaxFloat = 3.402823466e38f;

__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 x, u32x4 y, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
}

// Four columns loaded `shift` columns early, because fewer than four are left of the row: moved to their places, zero beyond it.
__device__ __forceinline__ f32x4 shifted(f32x4 v, int shift) {
  f32x4 o;
  o.x = shift == 1 ? v.y : shift == 2 ? v.z : shift == 3 ? v.w : 0.f;
  o.y = shift == 1 ? v.z : shift == 2 ? v.w : 0.f;
  o.z = shift == 1 ? v.w : 0.f;
  o.w = 0.f;
  return o;
}

// ---- layers of many rows ---------------------------------------------------------------------------
// A workgroup makes 32 rows by 64 to 256 columns of y, tile after tile; its input columns are walked in chunks of 128 (64), both operands of
// a chunk as parts in LDS.  One half of the wavefronts puts chunks together (32 or 16 lanes to a row, two rows each, 16 bytes per lane), the
// other half multiplies them, each wavefront by its 16 C columns of the weights, whose parts come from memory in the order in which the lanes
// hold them.  The chunks of a workgroup's tiles follow each other without a gap.
//   What bounds it: the requests for the sources' rows and, beside them on the same path, those for the weights' parts, which wait behind the
// rows and take 20 to 30 us of the widest layers' 130 to 200, wherever they are read from.  The matrix instructions are hidden.
//   Why this shape (us, one round of chunks of 64 columns with a barrier each, two workgroups of eight wavefronts per compute unit / this):
//   * one workgroup of sixteen wavefronts for a compute unit and all 256 columns in it: rows are put together and weights read once where two
//     workgroups or column groups did it twice, and a row is asked for in pieces of 512 bytes, of which those that start off a 128-byte
//     line touch five lines for four where pieces of 256 touch three for two.  18.6 k rows x 2 x 602 x 256, 10 sources each, 164 / 136; 60 k x 2 x 128
//     x 512, 25 sources, 235 / 195; 2 k x 2 x 256 x 256, 15 sources, 33 / 24.
//   * a ring of three buffers (four with one operand) without barriers, so that a row with a long list holds up nothing until the ring is empty;
//   * rows shared out in halves of tiles, so that no workgroup has more than one half more than another;
//   * up to 64 outputs two wavefronts share columns and take a row tile each, because four would leave half of the multiplying ones idle:
//     20 k x 2 x 96 x 64, 15 sources, 32.2 / 29.3, with 128 columns (half of them padding) 30.4;
//   * multiplying wavefronts whose columns are past the last one leave the chunks to the others: 17 k x 2 x 256 x 172, 15 sources, 59.7, with their
//     padding multiplied 61.6;
//   * inputs of up to 64 columns with up to 128 outputs stay with chunks of 64 and two workgroups of eight wavefronts, since half of a chunk of
//     128 would be empty: 20 k x 2 x 64 x 64, 5 sources, 20.5 / 19.1, in the other shape 23.1; 8.7 k x 2 x 64 x 100, 15 sources, 18.9 / 19.3, 21.1 (8.2 k
//     to 9 k rows are the ones that lost, 0 to 5 %; 4 k gained 9 %, 17 k 7 %);
//   * one round of eight loads in flight per lane: eight such wavefronts to a compute unit ask for enough, and with two the registers' moves cost
//     1 to 3 %.  Places for as many sources as a fan-out can have, because those beyond them are read one after the other (chunks of 64, 12 k
//     rows of 64 sources x 2 x 256 x 256: 120 us, with 32 places 248).
//   Sixteen wavefronts on a compute unit leave a lane 128 registers: 16 and 32 columns to a wavefront fit, 64 do not.
constexpr int kLayerRows = 32, kLayerFlags = 64;

// W wavefronts of either kind: chunks of 16 W columns, 4 W lanes to a row, 16 W C / RS columns of y.  Eight of each fill a compute unit
// with one workgroup, four of each with two.  RS: wavefronts that share columns, each with 2 / RS of the row tiles.
template <int W>
struct LayerShape {
  static constexpr int kThreads = 128 * W, kChunk = 16 * W, kLanes = 4 * W, kPerCu = 8 / W;
};

template <int W, bool GCN>
struct LayerLds {
  static constexpr int kOps = GCN ? 1 : 2, kBuffers = W == 4 ? 2 : GCN ? 4 : 3;
  // [buffer][operand][k step of 32][row tile][part]: 64 lanes' fragments of 8 bf16; lane (g, r) = (l / 16, l % 16) holds
  // columns 8g .. 8g+7 of row r, in the place (r + 4g + k step) % 16 of its group so that the writes of a row spread over the banks
  __attribute__((aligned(16))) unsigned char a[kBuffers][kOps][W / 2][2][3][1024];
  // where a row's first sources are (all of them, in batches of dci_sample_khop, but for the last eight of the longest lists in the
  // shape that has no room for them)
  static constexpr int kSlots = W == 8 && !GCN ? 56 : 64;
  static_assert(kSlots % 8 == 0, "sources are read in rounds of eight");
  const float* src[kLayerRows][kSlots];
  int again[kLayerFlags];            // tiles to make again with the fp32 instructions
  int full[4], free[4];              // per buffer: wavefronts that have put their part of a chunk there / are done with it, over all chunks
};

// Chunks pass from the wavefronts that put them together to those that multiply them through a ring of buffers, without a barrier: either kind
// waits for the other only where the ring is empty or full (the workgroup's wavefronts are all on the compute unit).
__device__ __forceinline__ void ring_wait(const int* count, int target) {
  while (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target) __builtin_amdgcn_s_sleep(1);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
__device__ __forceinline__ void ring_signal(int* count, int lane) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if (lane == 0) (void)__hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <int C>
using vec_t = float __attribute__((ext_vector_type(C)));

template <bool EXACT>
__device__ __forceinline__ void put4(unsigned char* p, f32x4 v) {
  if (EXACT) {
    *reinterpret_cast<f32x4*>(p) = v;
  } else {
    const Split2 s0 = split2(v.x * kScale, v.y * kScale), s1 = split2(v.z * kScale, v.w * kScale);
    *reinterpret_cast<u32x2*>(p) = u32x2{s0.h, s1.h};
    *reinterpret_cast<u32x2*>(p + 1024) = u32x2{s0.m, s1.m};
    *reinterpret_cast<u32x2*>(p + 2048) = u32x2{s0.l, s1.l};
  }
}

__device__ __forceinline__ const float* source_row(const LayerArgs& a, long long e) {
  const int s = a.blk_src[e], r = a.rowref ? a.rowref[s] : -1;
  return r >= 0 ? a.cache + (long long)r * a.D : a.x + (long long)s * a.D;
}

// y for this lane's part of a tile: rows 4g .. 4g+3 of NT row tiles from the t0-th, columns col .. col + C-1
template <int C, int NT>
__device__ __forceinline__ void store_tile(const LayerArgs& a, long long row0, int rows, int col, int t0, int g, const f32x4 (&acc)[NT][C]) {
  const int N = a.N;
  float bias[C];
#pragma unroll
  for (int c = 0; c < C; ++c) bias[c] = a.bias[col + c < N ? col + c : N - 1];
  const bool whole = col + C <= N;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * (t0 + t) + 4 * g + r;
      if (i < rows) {
        vec_t<C> v;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          v[c] = acc[t][c][r] + bias[c];
          if (a.relu) v[c] = v[c] > 0.f ? v[c] : 0.f;
        }
        typedef vec_t<C> __attribute__((aligned(4))) vec_c_u;
        float* y = a.y + (row0 + i) * N + col;
        if (whole) {
          *reinterpret_cast<vec_c_u*>(y) = v;
        } else {
#pragma unroll
          for (int c = 0; c < C; ++c)
            if (col + c < N) y[c] = v[c];
        }
      }
    }
}

// A tile with the fp32 instructions, chunk by chunk, nothing overlapped.
template <int W, int C, int RS, bool GCN>
__device__ __forceinline__ void layer_tile_exact(const LayerArgs& a, LayerLds<W, GCN>& lds, long long row0, int rows, int cg) {
  constexpr int NT = 2 / RS, kCols = W / RS, kChunk = LayerShape<W>::kChunk, kLanes = LayerShape<W>::kLanes;
  const int tid = (int)threadIdx.x, lane = tid & 63, g = lane >> 4, r16 = lane & 15, gl = tid & (kLanes - 1), i = tid / kLanes;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, N = a.N;
  const int p_ks = gl >> 3, p_g = (gl & 7) >> 1;
  const int p_slot = p_ks * 6144 + (i >> 4) * 3072 + (p_g * 16 + ((i + 4 * p_g + p_ks) & 15)) * 16 + (gl & 1) * 1024;
  const int col = ((cg * kCols + wave % kCols) * 16 + r16) * C, t0 = wave / kCols % RS;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[NT][C];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[t][c] = zero;
#pragma unroll 1
  for (int k_lo = 0; k_lo < D; k_lo += kChunk) {
    const int k_col = k_lo + 4 * gl, k_ld = k_col < D - 4 ? k_col : D - 4, shift = k_col - k_ld;
    f32x4 own = zero, sum = zero;
    if (i < rows) {
      own = load4(a.x + (row0 + i) * D + k_ld);
      if (GCN) sum = own;
      const long long e0 = a.blk_indptr[row0 + i], e1 = a.blk_indptr[row0 + i + 1];
      for (long long e = e0; e < e1; ++e) sum += load4(source_row(a, e) + k_ld);
      const float cnt = (float)(e1 - e0) + (GCN ? 1.f : 0.f);
      if (a.mode != DCI_MODEL_SAGE_SUM && cnt != 0.f) sum = f32x4{sum.x / cnt, sum.y / cnt, sum.z / cnt, sum.w / cnt};
    }
    if (!GCN) put4<true>(&lds.a[0][0][0][0][0][0] + p_slot, shift ? shifted(own, shift) : own);
    put4<true>(&lds.a[0][GCN ? 0 : 1][0][0][0][0] + p_slot, shift ? shifted(sum, shift) : sum);
    __syncthreads();
    if (wave < W) {
#pragma unroll 1
      for (int st = GCN ? W / 2 : 0; st < W; ++st) {
        const int op = st / (W / 2), ks = st % (W / 2);
        const float* weights = op ? a.w_neigh : a.w_self;
        float raw[8][C];  // zero past the last row, the last column past it (not stored)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const int k = k_lo + 32 * ks + 8 * g + j;
            raw[j][c] = k < D ? weights[(long long)k * N + (col + c < N ? col + c : N - 1)] : 0.f;
          }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const unsigned char* p = &lds.a[0][GCN ? 0 : op][ks][t0 + t][0][0] + (g * 16 + ((r16 + 4 * g + ks) & 15)) * 16;
          const f32x4 x[2] = {*reinterpret_cast<const f32x4*>(p), *reinterpret_cast<const f32x4*>(p + 1024)};
#pragma unroll
          for (int c = 0; c < C; ++c) {
            f32x4 part = zero;
#pragma unroll
            for (int j = 0; j < 8; ++j) part = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j >> 2][j & 3], raw[j][c], part, 0, 0, 0);
            acc[t][c] += part;
          }
        }
      }
    }
    __syncthreads();
  }
  if (wave < W) store_tile<C, NT>(a, row0, rows, col, t0, g, acc);
}

// The parts of one row tile's k step
struct RowParts {
  bf16x8 p[3];
};
template <int W, bool GCN>
__device__ __forceinline__ RowParts row_parts(const LayerLds<W, GCN>& lds, int buf, int op, int ks, int t, int lane) {
  const int g = lane >> 4, r16 = lane & 15;
  const unsigned char* const at = &lds.a[buf][op][ks][t][0][0] + (g * 16 + ((r16 + 4 * g + ks) & 15)) * 16;
  RowParts r;
#pragma unroll
  for (int p = 0; p < 3; ++p) r.p[p] = *reinterpret_cast<const bf16x8*>(at + p * 1024);
  return r;
}

// Multiplies one chunk of n_ks k steps.  b[0]: the parts of the chunk's first column tiles, asked for before; left there: those of the
// next chunk (w_next).  NT: row tiles, from the t0-th.  The rows'
// parts are read from LDS one row tile ahead of the matrix instructions.
template <int W, int C, bool GCN, int NT>
__device__ __forceinline__ void multiply_chunk(const LayerLds<W, GCN>& lds, int buf, int lane, int t0, const char* w, size_t w_op, size_t w_step, int n_ks,
                                               const char* w_next, u32x4 (&b)[2][C < 2 ? 1 : 2][3], f32x4 (&acc)[NT][C]) {
  constexpr int kPair = C < 2 ? 1 : 2, kPairs = C / kPair, kOps = GCN ? 1 : 2, kUnits = kOps * kPairs;
  typedef __attribute__((address_space(1))) const u32x4* gw_t;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  RowParts a_next = row_parts<W, GCN>(lds, buf, 0, 0, t0, lane);
#pragma unroll
  for (int ks = 0; ks < W / 2; ++ks) {
    // (GCN's steps come in twos, so that the next chunk starts with b[0]: where their number is odd the last multiplies zeros with the same weights)
    if (ks >= n_ks && !(GCN && kPairs == 1 && (ks & 1) && ks == n_ks)) break;
#pragma unroll
    for (int uu = 0; uu < kUnits; ++uu) {
      const int u = ks * kUnits + uu, pair = uu % kPairs;
      // the unit after this one: of this k step, of the next, or of the next chunk
      const bool last = uu + 1 == kUnits;
      const int un = last ? 0 : uu + 1, kn = last ? ks + 1 : ks;
      {
        const char* p = w + kn * w_step;
        if (last && kn >= n_ks) p = GCN && kPairs == 1 && (kn & 1) ? w + ks * w_step : w_next;
        if (!last && !GCN) p += un / kPairs * w_op;
#pragma unroll
        for (int c = 0; c < kPair; ++c)
#pragma unroll
          for (int q = 0; q < 3; ++q) b[(u + 1) & 1][c][q] = *((gw_t)(p + ((un % kPairs * kPair + c) * 3 + q) * 1024) + lane);
      }
      // the step's 32 products are added up from zero, h h by itself and the others smallest first, and join the running sum as
      // one number
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const RowParts a = a_next;
        if (t + 1 < NT) a_next = row_parts<W, GCN>(lds, buf, uu / kPairs, ks, t0 + t + 1, lane);
        else if (kn < W / 2) a_next = row_parts<W, GCN>(lds, buf, un / kPairs, kn, t0, lane);  // (past the chunk's last step: not used)
        f32x4 top[kPair], rest[kPair];
#define DCI_MM(TO_, A_, P_, IN_) \
  _Pragma("unroll") for (int c = 0; c < kPair; ++c) TO_[c] = mfma_bf16(a.p[A_], b[u & 1][c][P_], IN_)
        DCI_MM(rest, 2, 1, zero);
        DCI_MM(rest, 1, 2, rest[c]);
        DCI_MM(rest, 2, 0, rest[c]);
        DCI_MM(rest, 0, 2, rest[c]);
        DCI_MM(rest, 1, 1, rest[c]);
        DCI_MM(rest, 1, 0, rest[c]);
        DCI_MM(rest, 0, 1, rest[c]);
        DCI_MM(top, 0, 0, zero);
#undef DCI_MM
#pragma unroll
        for (int c = 0; c < kPair; ++c) acc[t][pair * kPair + c] += top[c] + rest[c];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

template <int W, int C, int RS, bool GCN>
__global__ __launch_bounds__(LayerShape<W>::kThreads, 4) void k_sage_layer(LayerArgs a) {
  constexpr int NT = 2 / RS, kCols = W / RS, kChunk = LayerShape<W>::kChunk, kLanes = LayerShape<W>::kLanes;
  __shared__ LayerLds<W, GCN> lds;
  const long long M = a.counts[a.hop];
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D;
  constexpr int kSlots = LayerLds<W, GCN>::kSlots;
  // The rows in halves of a tile (16), shared out evenly: a workgroup takes a stretch of them, two at a time.  The workgroups of the column
  // groups of a stretch are neighbours on one XCD.
  const int b = (int)blockIdx.x, n_wgs = (int)gridDim.x / a.n_col_groups;
  const int cg = (b >> 3) % a.n_col_groups, wg = (b >> 3) / a.n_col_groups * 8 + (b & 7);
  const long long n_halves = (M + 15) / 16, h_begin = wg * n_halves / n_wgs, h_end = (wg + 1) * n_halves / n_wgs;
  constexpr int kBuffers = LayerLds<W, GCN>::kBuffers;
  if (tid < kLayerFlags) lds.again[tid] = 0;
  if (tid < kBuffers) lds.full[tid] = lds.free[tid] = 0;
  __syncthreads();
  const int n_chunks = (D + kChunk - 1) / kChunk;

  if (wave >= W) {
    // ---- puts the chunks together, ahead of the others
    __builtin_amdgcn_s_setprio(2);  // its loads are asked for before the others' matrix instructions are issued
    const int pt = tid - 64 * W, gl = pt & (kLanes - 1), grp = pt / kLanes;
    const int p_ks = gl >> 3, p_g = (gl & 7) >> 1;
    const int p_slot = p_ks * 6144 + (p_g * 16 + ((grp + 4 * p_g + p_ks) & 15)) * 16 + (gl & 1) * 8;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    int buf = 0, lap = 0;  // the chunk's buffer, and how often the ring has been round
    for (long long h = h_begin; h < h_end; h += 2) {
      const int halves = h_end - h < 2 ? 1 : 2;
      const long long row0 = 16 * h;
      const int rows = M - row0 < 16 * halves ? (int)(M - row0) : 16 * halves;
      const float* own[2];
      long long e0[2];
      int deg[2];
      bool ok[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int i = 16 * t + grp;
        ok[t] = i < rows;
        own[t] = a.x + (row0 + (ok[t] ? i : 0)) * D;
        e0[t] = ok[t] ? a.blk_indptr[row0 + i] : 0;
        deg[t] = ok[t] ? (int)(a.blk_indptr[row0 + i + 1] - e0[t]) : 0;
      }
      // A row's sources come in rounds of eight loads, across rows and chunks; the next round is asked for as soon as one has been added.
      int rounds[2];  // of the wavefront's row with the most
      int whole[2];   // rounds in which each of its rows has eight sources
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        int n = deg[t] < kSlots ? deg[t] : kSlots;
        int least = n;
        for (int d = kLanes; d < 64; d <<= 1) {
          const int o = __shfl_xor(n, d, 64), o_least = __shfl_xor(least, d, 64);
          n = o > n ? o : n;
          least = o_least < least ? o_least : least;
        }
        n = __builtin_amdgcn_readfirstlane(n);
        rounds[t] = n > 8 ? (n + 7) / 8 : 1;
        whole[t] = __builtin_amdgcn_readfirstlane(least) / 8;
      }
      // (written and read by one group of lanes; places without a source, up to the last that a round asks for, hold the row itself)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < kSlots; s += kLanes)
          if (s < 8 * rounds[t] && s + gl < kSlots) lds.src[16 * t + grp][s + gl] = s + gl < deg[t] ? source_row(a, e0[t] + s + gl) : own[t];
      f32x4 v[8], own_new;
      int n_k = 0, n_t = 0, n_r = 0;  // the round to ask for next
      auto ask = [&]() {
        if (n_k >= n_chunks) return;
        const int k_col = n_k * kChunk + 4 * gl, k_ld = k_col < D - 4 ? k_col : D - 4;
        const float* const* p = &lds.src[16 * n_t + grp][8 * n_r];
        if (n_r == 0) own_new = load4((n_t ? own[1] : own[0]) + k_ld);
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = load4(p[u] + k_ld);
        if (++n_r == (n_t ? rounds[1] : rounds[0])) {
          n_r = 0;
          if (++n_t == halves) {
            n_t = 0;
            ++n_k;
          }
        }
      };
      int k = 0, t = 0, r = 0;  // the round to add
      f32x4 sum = zero, own_v = zero;
      auto add = [&]() {
        const int deg_t = t ? deg[1] : deg[0];
        if (r == 0) {
          own_v = own_new;
          sum = GCN ? own_v : zero;
        }
        if (r < (t ? whole[1] : whole[0])) {
#pragma unroll
          for (int u = 0; u < 8; ++u) sum += v[u];
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const bool in = 8 * r + u < deg_t;
            sum.x = in ? sum.x + v[u].x : sum.x;
            sum.y = in ? sum.y + v[u].y : sum.y;
            sum.z = in ? sum.z + v[u].z : sum.z;
            sum.w = in ? sum.w + v[u].w : sum.w;
          }
        }
        asm volatile("" : "+v"(sum), "+v"(own_v));  // added here, before the places are asked for again
        ask();
        if (++r < (t ? rounds[1] : rounds[0])) return;
        // the row's part of the chunk is complete
        r = 0;
        const int k_col = k * kChunk + 4 * gl, k_ld = k_col < D - 4 ? k_col : D - 4, shift = k_col - k_ld;
        for (int e = kSlots; e < deg_t; ++e) sum += load4(source_row(a, (t ? e0[1] : e0[0]) + e) + k_ld);
        const float cnt = (float)deg_t + (GCN ? 1.f : 0.f);
        if (a.mode != DCI_MODEL_SAGE_SUM && cnt != 0.f) sum = f32x4{sum.x / cnt, sum.y / cnt, sum.z / cnt, sum.w / cnt};
        if (shift) {
          sum = shifted(sum, shift);
          if (!GCN) own_v = shifted(own_v, shift);
        }
        const bool ok_t = t ? ok[1] : ok[0];
        if (t == 0) ring_wait(&lds.free[buf], W * lap);
        if (!GCN) put4<false>(&lds.a[buf][0][0][t][0][0] + p_slot, ok_t ? own_v : zero);
        put4<false>(&lds.a[buf][GCN ? 0 : 1][0][t][0][0] + p_slot, ok_t ? sum : zero);
        if (++t < halves) return;
        t = 0;
        ++k;
        ring_signal(&lds.full[buf], lane);
        if (++buf == kBuffers) {
          buf = 0;
          ++lap;
        }
      };
      ask();
      while (k < n_chunks) add();
    }
    __syncthreads();
  } else {
    // ---- multiplies
    constexpr int kPair = C < 2 ? 1 : 2;
    typedef __attribute__((address_space(1))) const u32x4* gw_t;
    // the parts of the weights: [operand][k step][wavefront, of all column groups][tile][part][lane]
    // (wavefronts whose columns are all past the last one only hand the buffers back)
    constexpr size_t kPieceBytes = (size_t)C * 3 * 1024;
    const int my_wave = cg * kCols + wave % kCols;
    const bool has_cols = my_wave * 16 * C < a.N;
    const size_t w_step = parts_pieces(a.N, C) * kPieceBytes, w_op = w_step * ((D + 31) / 32);
    const int t0 = wave / kCols;
    const char* const w_base = reinterpret_cast<const char*>(a.w_split) + my_wave * kPieceBytes;
    u32x4 b[2][kPair][3];
    int buf = 0, lap = 0, it = 0;
    if (h_begin < h_end && has_cols) {
#pragma unroll
      for (int c = 0; c < kPair; ++c)
#pragma unroll
        for (int p = 0; p < 3; ++p) b[0][c][p] = *((gw_t)(w_base + (c * 3 + p) * 1024) + lane);
    }
    // a tile of which this wavefront multiplies N_ row tiles (0: it only hands the buffers back)
    auto tile = [&](auto n_rows_, long long h) {
      constexpr int kRowTiles = decltype(n_rows_)::value, kAcc = kRowTiles ? kRowTiles : 1;
      f32x4 acc[kAcc][C];
#pragma unroll
      for (int t = 0; t < kAcc; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int k = 0; k < n_chunks; ++k) {
        ring_wait(&lds.full[buf], W * (lap + 1));
        const char* w = w_base + (size_t)(W / 2 * k) * w_step;
        const int left = (D - k * kChunk + 31) / 32;
        if (kRowTiles)
          multiply_chunk<W, C, GCN, kAcc>(lds, buf, lane, t0, w, w_op, w_step, left < W / 2 ? left : W / 2, k + 1 < n_chunks ? w + W / 2 * w_step : w_base,
                                          b, acc);
        ring_signal(&lds.free[buf], lane);
        if (++buf == kBuffers) {
          buf = 0;
          ++lap;
        }
      }
      if (!kRowTiles) return;
      bool bad = false;
#pragma unroll
      for (int t = 0; t < kAcc; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            bad |= !(__builtin_fabsf(acc[t][c][r]) <= kMaxFloat);
            acc[t][c][r] *= kUnscale;
          }
      if (bad) lds.again[it % kLayerFlags] = 1;
      store_tile<C, kAcc>(a, 16 * h, M - 16 * h < kLayerRows ? (int)(M - 16 * h) : kLayerRows, ((cg * kCols + wave % kCols) * 16 + (lane & 15)) * C, t0,
                          lane >> 4, acc);
    };
    long long h = h_begin;
    for (; h + 1 < h_end; h += 2, ++it) {
      if (has_cols) tile(std::integral_constant<int, NT>(), h);
      else tile(std::integral_constant<int, 0>(), h);
    }
    if (h < h_end) {  // half a tile is left
      if (has_cols && t0 == 0) tile(std::integral_constant<int, 1>(), h);
      else tile(std::integral_constant<int, 0>(), h);
    }
    __syncthreads();
  }
  // tiles with a number that the parts cannot hold, once more (and, past 64 tiles, those whose flag they share)
  int it = 0;
  for (long long h = h_begin; h < h_end; h += 2, ++it) {
    if (!lds.again[it % kLayerFlags]) continue;
    const long long row0 = 16 * h, end = 16 * h_end < M ? 16 * h_end : M;
    layer_tile_exact<W, C, RS, GCN>(a, lds, row0, end - row0 < kLayerRows ? (int)(end - row0) : kLayerRows, cg);
  }
}

__global__ __launch_bounds__(256) void k_split_weights(SplitArgs a) { split_weights(a, (int)blockIdx.x); }

// ---- layers of few rows ---------------------------------------------------------------------------
// A workgroup of sixteen wavefronts makes 16 rows by 64 columns of y: wavefront w puts row w together (256 columns of it at
// a time, 16 bytes per lane, the places of the sources in scalar registers), then multiplies one k step of 32 of the chunk
// with the weights it asked for beforehand; the sixteen partial tiles are added up through LDS.
//   Bound by the latency of its chain of look-ups (row count and list bounds, sources, their cache slots, their rows); all sixteen rows
// and all of the weights are asked for at once, and the list bounds beside the row count.  A layer of 40 x 2 x 256 x 256 takes 10 us;
// as three kernels it took 15.
constexpr int kSmallThreads = 1024, kSmallRows = 16, kSmallCols = 64, kSmallChunk = 256;

template <bool GCN, bool EXACT>
__device__ __forceinline__ float small_tile(const LayerArgs& a, unsigned char* lds, long long row0, int rows, int deg, int ref,
                                            long long e0, int col0) {
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int D = a.D, N = a.N;
  int col = col0 + 4 * r16;
  if (col > N - 4) col = N - 4;
  f32x4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int i = wave;
  const bool ok = i < rows;
  const float* own_row = a.x + (row0 + (ok ? i : 0)) * D;
#pragma unroll 1
  for (int k_lo = 0; k_lo < D; k_lo += kSmallChunk) {
    const int steps1 = ((D - k_lo < kSmallChunk ? D - k_lo : kSmallChunk) + 31) / 32;  // k steps of an operand in this chunk
    const int op = GCN ? 1 : (wave >= steps1 ? 1 : 0), ks = op && !GCN ? wave - steps1 : wave;
    const bool has = ks < steps1;
    f32x4 raw[8];
    if (has) {
      const float* W = op ? a.w_neigh : a.w_self;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = k_lo + 32 * ks + 8 * g + j;
        raw[j] = load4(W + (long long)(k < D ? k : D - 1) * N + col);
      }
    }
    // ---- this wavefront's row
    const int k_col = k_lo + 4 * lane;
    const int k_ld = k_col < D - 4 ? k_col : D - 4;
    const int shift = k_col - k_ld;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 own = load4(own_row + k_ld);
    f32x4 sum = GCN ? own : zero;
    for (int e = 0; e < deg; e += 8) {
      int r_l = ref;  // lane l: where source l of the first 64 is
      if (e >= 64) {
        const int s = e + (lane & 7) < deg ? a.blk_src[e0 + e + (lane & 7)] : 0;
        const int r = a.rowref ? a.rowref[s] : -1;
        r_l = r >= 0 ? r : ~s;
      }
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int at = e + u < deg ? e + u : deg - 1;
        const int r = __builtin_amdgcn_readlane(r_l, e >= 64 ? at - e : at);
        v[u] = load4((r >= 0 ? a.cache : a.x) + (long long)(r >= 0 ? r : ~r) * D + k_ld);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (e + u < deg) sum += v[u];
    }
    const float cnt = (float)deg + (GCN ? 1.f : 0.f);
    if (a.mode != DCI_MODEL_SAGE_SUM && cnt != 0.f) sum = f32x4{sum.x / cnt, sum.y / cnt, sum.z / cnt, sum.w / cnt};
    const int w_step = lane >> 3, w_g = (lane & 7) >> 1;
    unsigned char* const p_w = lds + w_step * 3072 + (w_g * 16 + ((i + 4 * w_g + (w_step & 3)) & 15)) * 16 + (lane & 1) * (EXACT ? 1024 : 8);
    auto put = [&](int op_, f32x4 v) {
      if (shift) v = shifted(v, shift);
      if (!ok) v = zero;
      unsigned char* p = p_w + op_ * (kSmallChunk / 32 * 3072);
      if (EXACT) {
        *reinterpret_cast<f32x4*>(p) = v;
      } else {
        const Split2 s0 = split2(v.x * kScale, v.y * kScale), s1 = split2(v.z * kScale, v.w * kScale);
        *reinterpret_cast<u32x2*>(p) = u32x2{s0.h, s1.h};
        *reinterpret_cast<u32x2*>(p + 1024) = u32x2{s0.m, s1.m};
        *reinterpret_cast<u32x2*>(p + 2048) = u32x2{s0.l, s1.l};
      }
    };
    if (!GCN) put(0, own);
    put(1, sum);
    __syncthreads();
    // ---- this wavefront's k step
    if (has) {
      const unsigned char* p = lds + (op * (kSmallChunk / 32) + ks) * 3072 + (g * 16 + ((r16 + 4 * g + (ks & 3)) & 15)) * 16;
      if (!EXACT) {
        const bf16x8 ah = *reinterpret_cast<const bf16x8*>(p), am = *reinterpret_cast<const bf16x8*>(p + 1024),
                     al = *reinterpret_cast<const bf16x8*>(p + 2048);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          u32x4 b[3];
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const Split2 s = split2(raw[2 * jj][c] * kScale, raw[2 * jj + 1][c] * kScale);
            b[0][jj] = s.h;
            b[1][jj] = s.m;
            b[2][jj] = s.l;
          }
          f32x4 rest = mfma_bf16(al, b[1], zero);  // as in multiply_chunk
          rest = mfma_bf16(am, b[2], rest);
          rest = mfma_bf16(al, b[0], rest);
          rest = mfma_bf16(ah, b[2], rest);
          rest = mfma_bf16(am, b[1], rest);
          rest = mfma_bf16(am, b[0], rest);
          rest = mfma_bf16(ah, b[1], rest);
          acc[c] += mfma_bf16(ah, b[0], zero) + rest;
        }
      } else {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(p), hi = *reinterpret_cast<const f32x4*>(p + 1024);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          f32x4 part = zero;
#pragma unroll
          for (int j = 0; j < 8; ++j)
            part = __builtin_amdgcn_mfma_f32_16x16x4f32(j < 4 ? lo[j & 3] : hi[j & 3],
                                                        k_lo + 32 * ks + 8 * g + j < D ? raw[j][c] : 0.f, part, 0, 0, 0);
          acc[c] += part;
        }
      }
    }
    __syncthreads();
  }
  // ---- add up the wavefronts' tiles: [wavefront][row][column]
  const int n_parts = D < kSmallChunk ? (GCN ? 1 : 2) * ((D + 31) / 32) : (GCN ? 8 : 16);
  float* const red = reinterpret_cast<float*>(lds);
  if (wave < n_parts)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<f32x4*>(red + wave * (kSmallRows * kSmallCols) + (4 * g + r) * kSmallCols + 4 * r16) =
          f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
  __syncthreads();
  // (in pairs: sixteen one after the other round 2 x 602 products of one sign to 4.4 x 2^-24 of their sum at most, pairs to
  // 2.3; the kernel that split the contraction eight ways had 3.7)
  float sum[16];
#pragma unroll
  for (int w = 0; w < 16; ++w) sum[w] = w < n_parts ? red[w * (kSmallRows * kSmallCols) + tid] : 0.f;
#pragma unroll
  for (int n = 8; n > 0; n >>= 1)
#pragma unroll
    for (int w = 0; w < n; ++w) sum[w] += sum[w + n];
  const float v = sum[0];
  return EXACT ? v : v * kUnscale;
}

template <bool GCN>
__global__ __launch_bounds__(kSmallThreads) void k_sage_layer_small(LayerArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[16 * kSmallRows * kSmallCols * 4];
  static_assert(sizeof(lds) >= 2 * kSmallChunk / 32 * 3072, "both operands of a chunk");
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cg = (int)blockIdx.x % a.n_col_groups;
  const long long row0 = (long long)((int)blockIdx.x / a.n_col_groups) * kSmallRows;
  // the row's list bounds are read beside the row count, not after it (the array has room for the layer's bound)
  long long i = row0 + wave;
  if (i > a.cap_rows - 1) i = a.cap_rows - 1;
  const long long M = a.counts[a.hop];
  const long long b0 = a.blk_indptr[i], b1 = a.blk_indptr[i + 1];
  if (row0 >= M) return;
  const int rows = M - row0 < kSmallRows ? (int)(M - row0) : kSmallRows;
  const long long e0 = wave < rows ? b0 : 0;
  const int deg = wave < rows ? (int)(b1 - b0) : 0;
  int ref = 0;
  if (lane < deg) {
    const int s = a.blk_src[e0 + lane];
    const int r = a.rowref ? a.rowref[s] : -1;
    ref = r >= 0 ? r : ~s;
  }
  const int col0 = cg * kSmallCols;
  float v = small_tile<GCN, false>(a, lds, row0, rows, deg, ref, e0, col0);
  if (__syncthreads_or(!(__builtin_fabsf(v) <= kMaxFloat))) v = small_tile<GCN, true>(a, lds, row0, rows, deg, ref, e0, col0);
  const int r = tid >> 6;
  int col = col0 + (tid & 60);
  if (col > a.N - 4) col = a.N - 4;
  col += tid & 3;
  if (r < rows) {
    v += a.bias[col];
    if (a.relu) v = v > 0.f ? v : 0.f;
    a.y[(row0 + r) * a.N + col] = v;
  }
}

// Which kernel, by the bounds on the layer's rows and on the length of their lists (batches fill a fifth of the rows' bound to all
// of it; f: sources of every row):
//   * the one for few rows while its workgroups have a compute unit each, all of the bound taken for the rows of the seeds' block, half
//     of it for the next one's (0.5 - 0.7 of it in batches of 256 to 1,024 seeds, fan-outs of 5 to 10) and a fifth for those behind.  Three layers of 16 - 289 rows (request of 16 seeds): a pass
//     79 us against 94 with aggregation, dense layer and sum of the split contraction as kernels of their own.  On either side
//     of the line, this kernel / the other: 4,096 rows x 2 x 256 x 64 (256 workgroups), f = 5, 12.2 us / 19.0, x 100 (512) 22.1 / 19.8, x 172
//     (768) 31.1 / 21.7; 1,024 x 2 x 100 x 256 (256), f = 10, 10.8 / 16.3, 2,048 x 2 x 256 x 256 (512), f = 15, 28.3 / 23.8.
//   * above it k_sage_layer, in the shape that its width asks for (LayerPlan; figures at the kernel).  It and the layer's two kernels: 1 k rows x 2 x 256 x
//     512, f = 10, 24.7 us / 24.8; 3.1 k x 2 x 75 x 130, f = 8, 14.9 / 19.3; 2 k x 2 x 300 x 320, f = 25, 30.8 / 32.3; 6 k x 2 x 602 x 192, f = 10, 53.9 / 77.5.
//     More than 256 outputs are two column groups or more, which put the same rows together again.
//   * neither where lists are long: in few workgroups the lists' latency is not hidden.  With lists of more than 10,000 numbers the
//     layer's two kernels are ahead (x 256 outputs, one kernel / the two; the two have a launch more, 1 - 2 us).  k_sage_layer_small,
//     1,024 rows: D = 100, f = 64 0.86; D = 256, f = 25 0.93, f = 40 30.1 us / 26.3, f = 64 43 / 31; D = 300, f = 40 42 / 29; D = 602, f = 15 33.4
//     / 31.8, f = 25 50 / 36, f = 64 106 / 55.  (Where it has two compute units for every workgroup it is only behind for more
//     than 64 sources times pieces of 256 columns: 512 x 2 x D x 256, D = 256, f = 64 0.97; D = 300, f = 25 1.00, f = 64 1.26; D = 602, f = 25 1.16.)
//     k_sage_layer, 2,048 rows: D = 64, f = 64 19.3 / 18.3; D = 256, f = 25 26.0 / 27.3, f = 64 36.0 / 33.6; D = 300, f = 25 30.2 / 31.9, f = 40 32.7
//     / 34.8; D = 602, f = 25 45 / 52, f = 64 73 / 73.
//   * none of them where the lists are long and every column group puts the same rows together again, or rows are no whole 128-byte
//     lines, so that a piece of 512 bytes touches five for four.  The aggregation reads them once and in one piece, and the dense
//     layer follows.  18.6 k x 2 x D x N, this kernel / the two: f = 64, 602 x 256 512 us / 528, 602 x 1,024 1,051 / 815, 256 x 256 188 / 233,
//     256 x 1,024 409 / 364; f = 25, 602 x 256 233 / 278, 602 x 1,024 526 / 571, 256 x 256 92 / 127, 100 x 1,024 114 / 130; f = 15, 602 x 256 165 / 215,
//     602 x 512 235 / 319, 300 x 768 180 / 237 (60 k rows 653 / 752); f = 10, 300 x 300 114 / 122, 256 x 300 90 / 103.
//   The lines of the last two lie where a slower form of k_sage_layer (chunks of 64 columns, column groups of 64) met the two kernels.  Some
// layers beyond them, which the two kernels make, would now be faster in one: of these 602 x 256 and x 1,024, 100 x 1,024 and the last two with the
// lists named, by 8 to 16 %, and 60 k x 2 x 100 x 256, f = 25, by 21 %.
constexpr int64_t kSmallReads = 10000, kFewRowsPerCu = 40;

static size_t split_bytes(const LayerPlan& p, int ops) {
  return (size_t)ops * ((p.D + 31) / 32) * parts_pieces(p.N, p.C) * p.C * 3 * 1024;
}

// -1 not one of these kernels, 0 k_sage_layer_small, 1 k_sage_layer.  rows: about what a batch has; fan: the longest list.
static int kernel_for(const dci_ctx* ctx, const LayerPlan& p, int64_t rows, int64_t fan) {
  const bool short_lists = fan * p.D <= kSmallReads;
  const int64_t wgs = (rows + kSmallRows - 1) / kSmallRows * ((p.N + kSmallCols - 1) / kSmallCols);
  if (p.N >= 4 && wgs <= ctx->num_cus)
    return short_lists || (2 * wgs <= ctx->num_cus && fan * ((p.D + kSmallChunk - 1) / kSmallChunk) <= 64) ? 0 : -1;
  const int64_t g = (p.N + 255) / 256;
  if (g <= 4 && rows * g <= (int64_t)ctx->num_cus * kFewRowsPerCu) return short_lists ? 1 : -1;
  if (p.N > 256 && p.N <= 384) return -1;
  const bool lines = p.D % 32 == 0;  // rows are whole 128-byte lines
  return (lines ? fan * (g + 1) <= 128 : fan * (g < 3 ? 3 : g) <= 60) ? 1 : -1;
}

bool layers_plan(const dci_ctx* ctx, const dci_blocks* blocks, int32_t model, const int32_t* dims, void* scratch,
                 size_t scratch_bytes, LayerPlan* plans) {
  const int ops = model == DCI_MODEL_GCN_AVG ? 1 : 2, n_layers = blocks->n_hops;
  Arena ar(reinterpret_cast<char*>(scratch), scratch_bytes);
  for (int32_t l = 0; l < n_layers; ++l) {
    LayerPlan& p = plans[l];
    const int h = n_layers - 1 - l;
    p.D = dims[l];
    p.N = dims[l + 1];
    p.cap_rows = blocks->cap_rows[h];
    p.w_split = nullptr;
    if (p.D < 4 || p.cap_rows < 1) return false;
    const int64_t rows = h == 0 ? p.cap_rows : h == 1 ? p.cap_rows / 2 : p.cap_rows / 5;
    p.C = kernel_for(ctx, p, rows, (blocks->cap_edges[h] + p.cap_rows - 1) / p.cap_rows);
    if (p.C > 0) {
      const bool narrow = p.D <= 64 && p.N <= 128;
      p.rs = !narrow && p.N <= 64 ? 2 : 1;
      p.cols = narrow || p.N <= 64 ? 4 : 8;
      p.C = p.N > (narrow ? 64 : 128) ? 2 : 1;
      p.w_split = ar.take<char>(split_bytes(p, ops));
    }
  }
  return ar.ok();
}

SplitArgs layers_split_args(int32_t model, int32_t first, int32_t n_layers, const LayerPlan* plans, const float* const* w_self,
                            const float* const* w_neigh) {
  const bool gcn = model == DCI_MODEL_GCN_AVG;
  SplitArgs sa;
  for (int32_t l = first; l < n_layers; ++l) {
    const LayerPlan& p = plans[l];
    if (p.C <= 0) continue;
    sa.first[sa.n] = sa.wgs;
    sa.w[sa.n][0] = gcn ? w_neigh[l] : w_self[l];
    sa.w[sa.n][1] = w_neigh[l];
    sa.out[sa.n] = p.w_split;
    sa.D[sa.n] = p.D;
    sa.N[sa.n] = p.N;
    sa.C[sa.n] = p.C;
    sa.waves[sa.n] = parts_pieces(p.N, p.C);
    sa.ops[sa.n] = gcn ? 1 : 2;
    sa.wgs += (int)((split_bytes(p, sa.ops[sa.n]) / (3 * 1024) + 3) / 4);  // four tiles to a workgroup
    ++sa.n;
  }
  return sa;
}

int32_t layers_split_weights(dci_ctx* ctx, const SplitArgs& sa) {
  if (sa.wgs == 0) return DCI_OK;
  hipLaunchKernelGGL(k_split_weights, dim3((unsigned)sa.wgs), dim3(256), 0, ctx->stream, sa);
  DCI_LAUNCH_CHECK(ctx);
  return DCI_OK;
}

int32_t layer_launch(dci_ctx* ctx, const LayerPlan& plan, const LayerArgs& args) {
  LayerArgs a = args;
  const bool gcn = a.mode == DCI_MODEL_GCN_AVG;
  a.D = plan.D;
  a.N = plan.N;
  a.cap_rows = plan.cap_rows;
  a.w_split = plan.w_split;
  if (plan.C == 0) {
    a.n_col_groups = (a.N + kSmallCols - 1) / kSmallCols;
    const int64_t n = (plan.cap_rows + kSmallRows - 1) / kSmallRows * a.n_col_groups;
    hipLaunchKernelGGL((gcn ? k_sage_layer_small<true> : k_sage_layer_small<false>), dim3((unsigned)n), dim3(kSmallThreads), 0,
                       ctx->stream, a);
    DCI_LAUNCH_CHECK(ctx);
    return DCI_OK;
  }
  a.n_col_groups = (a.N + 16 * plan.C * plan.cols - 1) / (16 * plan.C * plan.cols);
  const int W = plan.cols * plan.rs;
  // one workgroup (two of the narrow shape) to a compute unit, as many for every column group, in eights for the XCDs; no more than there are
  // halves of tiles
  int64_t n = (int64_t)ctx->num_cus * (8 / W) / (8 * a.n_col_groups), most = ((plan.cap_rows + 15) / 16 + 7) / 8;
  if (n > most) n = most;
  if (n < 1) n = 1;
  const dim3 grid((unsigned)(8 * n * a.n_col_groups));
#define DCI_LAYER(W_, C_, RS_)                                                                                             \
  hipLaunchKernelGGL((gcn ? k_sage_layer<W_, C_, RS_, true> : k_sage_layer<W_, C_, RS_, false>), grid, dim3(LayerShape<W_>::kThreads), 0, \
                     ctx->stream, a)
  if (W == 4 && plan.C == 1) DCI_LAYER(4, 1, 1);
  else if (W == 4) DCI_LAYER(4, 2, 1);
  else if (plan.rs == 2) DCI_LAYER(8, 1, 2);
  else if (plan.C == 1) DCI_LAYER(8, 1, 1);
  else DCI_LAYER(8, 2, 1);
#undef DCI_LAYER
  DCI_LAUNCH_CHECK(ctx);
  return DCI_OK;
}

}  // namespace dci
