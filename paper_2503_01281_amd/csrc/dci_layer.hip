// One layer of the forward pass in one kernel: aggregation, dense layer, bias and ReLU.
//
//   y = x W_self + m W_neigh + b (+ ReLU), m_i = mean / sum of x[src] over row i of the block (GCN: y = m W + b, m_i the
//   mean over the row itself and its sources).
//
// A workgroup of four wavefronts makes 16 T rows by 64 C columns of y.  It walks the input columns in chunks of 64: the
// chunk of both operands is put together in LDS (16 lanes per row, 16 bytes per lane; a row's sources are added in edge
// order) and multiplied with the chunk's rows of the weights, a wavefront making all 16 T rows of 16 C columns.
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
// A workgroup makes 32 rows by 64 C columns of y.  Its input columns are walked in chunks of 64; both operands of a chunk stand
// in LDS as parts (two buffers).  Wavefronts 4-7 put chunks together (16 lanes per row, two rows each, 16 bytes per lane),
// wavefronts 0-3 multiply the chunk before, each by its 16 C columns of the weights, whose parts come from memory in the order
// in which the lanes hold them.  One barrier per chunk; the chunks of a workgroup's tiles follow each other without a gap.
//   What bounds it: asking for the sources' rows in pieces of 256 bytes (a piece that does not start on a 128-byte line touches
// three of them), 91 of the 94 us of 32.6 k rows x 2 x 300 x 128 with 369 k sources, 128 of the 166 us of 18.6 k x 2 x 602 x 256
// with 274 k; the aggregation alone, whole rows at a time, takes 70 and 85 there, and with the fp32 dense layer that followed
// it 129 and 200.  The products alone take 37 and 72 us.
//   Why this shape: wavefronts of their own for the two kinds of work, because a wavefront's vector and matrix instructions
// take turns (one role after the other in every wavefront: 121 us where this takes 94); 32 rows, so that two workgroups fit
// on a compute unit and the rounds of tiles are short; two rounds of loads on their way at any time (one at a time: 98 us); places for
// as many sources as a fan-out can have, because those beyond them are read one after the other (12 k rows of 64 sources x 2 x 256 x
// 256: 120 us, with 32 places 248; x 2 x 602 x 256: 380, 644).
//   Two workgroups on a compute unit leave a lane 128 registers.  With 64 columns to a wavefront that is 34 too few (27 for GCN), and they
// go to scratch memory, some of them in the loop over the chunks; 16 and 32 columns fit.
constexpr int kLayerThreads = 512, kLayerRows = 32, kLayerChunk = 64, kLayerSlots = 64, kLayerPerCu = 2, kLayerFlags = 64;

struct LayerLds {
  // [buffer][operand][k step of 32][row tile][part]: 64 lanes' fragments of 8 bf16; lane (g, r) = (l / 16, l % 16) holds
  // columns 8g .. 8g+7 of row r, in the place (r + 4g) % 16 of its group so that the writes of a row spread over the banks
  __attribute__((aligned(16))) unsigned char a[2][2][2][2][3][1024];
  const float* src[kLayerRows][kLayerSlots];  // where a row's first sources are (all of them, in batches of dci_sample_khop)
  static_assert(kLayerSlots >= DCI_MAX_FANOUT, "a list of the longest fan-out");
  int again[kLayerFlags];                     // tiles to make again with the fp32 instructions
};

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

// y for this lane's part of a tile: rows 4g .. 4g+3 of both row tiles, columns col .. col + C-1
template <int C>
__device__ __forceinline__ void store_tile(const LayerArgs& a, long long row0, int rows, int col, int g, const f32x4 (&acc)[2][C]) {
  const int N = a.N;
  float bias[C];
#pragma unroll
  for (int c = 0; c < C; ++c) bias[c] = a.bias[col + c < N ? col + c : N - 1];
  const bool whole = col + C <= N;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * t + 4 * g + r;
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
template <int C, bool GCN>
__device__ __forceinline__ void layer_tile_exact(const LayerArgs& a, LayerLds& lds, long long row0, int rows, int cg) {
  const int tid = (int)threadIdx.x, lane = tid & 63, g = lane >> 4, r16 = lane & 15, gl = tid & 15, i = tid >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, N = a.N;
  const int p_g = (gl & 7) >> 1;
  const int p_slot = (gl >> 3) * 6144 + (i >> 4) * 3072 + (p_g * 16 + ((i + 4 * p_g) & 15)) * 16 + (gl & 1) * 1024;
  const int frag = (g * 16 + ((r16 + 4 * g) & 15)) * 16;
  const int col = (cg * 64 + (wave & 3) * 16 + r16) * C;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[2][C];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[t][c] = zero;
#pragma unroll 1
  for (int k_lo = 0; k_lo < D; k_lo += kLayerChunk) {
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
    put4<true>(&lds.a[0][1][0][0][0][0] + p_slot, shift ? shifted(sum, shift) : sum);
    __syncthreads();
    if (wave < 4) {
#pragma unroll 1
      for (int st = GCN ? 2 : 0; st < 4; ++st) {
        const int op = st >> 1, ks = st & 1;
        const float* W = op ? a.w_neigh : a.w_self;
        float raw[8][C];  // zero past the last row, the last column past it (not stored)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const int k = k_lo + 32 * ks + 8 * g + j;
            raw[j][c] = k < D ? W[(long long)k * N + (col + c < N ? col + c : N - 1)] : 0.f;
          }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const unsigned char* p = &lds.a[0][op][ks][t][0][0] + frag;
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
  if (wave < 4) store_tile<C>(a, row0, rows, col, g, acc);
}

// Multiplies one chunk.  b[0]: the parts of the chunk's first column tiles, asked for before; left there: those of the next
// chunk (w_next; nullptr: there is none).
template <int C, bool GCN>
__device__ __forceinline__ void multiply_chunk(const LayerLds& lds, int buf, int lane, const char* w, size_t w_op, size_t next_ks,
                                               const char* w_next, u32x4 (&b)[2][C < 2 ? 1 : 2][3], f32x4 (&acc)[2][C]) {
  constexpr int kSteps = GCN ? 2 : 4, kPair = C < 2 ? 1 : 2, kPairs = C / kPair, kUnits = kSteps * kPairs;
  typedef __attribute__((address_space(1))) const u32x4* gw_t;
  const int g = lane >> 4, r16 = lane & 15;
  const int frag = (g * 16 + ((r16 + 4 * g) & 15)) * 16;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  bf16x8 af[2][3];
#pragma unroll
  for (int u = 0; u < kUnits; ++u) {
    const int st = u / kPairs, pair = u % kPairs;
    if (pair == 0) {
      const int op = GCN ? 1 : st & 1, ks = GCN ? st : st >> 1;
      const unsigned char* const p0 = &lds.a[buf][op][ks][0][0][0] + frag;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int p = 0; p < 3; ++p) af[t][p] = *reinterpret_cast<const bf16x8*>(p0 + t * 3072 + p * 1024);
    }
    {
      const int st_n = (u + 1) / kPairs;
      const char* p = u + 1 == kUnits ? w_next : w + (GCN ? 0 : (st_n & 1) * w_op) + ((GCN ? st_n : st_n >> 1) ? next_ks : 0);
#pragma unroll
      for (int c = 0; c < kPair; ++c)
#pragma unroll
        for (int q = 0; q < 3; ++q) b[(u + 1) & 1][c][q] = *((gw_t)(p + ((((u + 1) % kPairs) * kPair + c) * 3 + q) * 1024) + lane);
    }
    // the step's 32 products are added up from zero, h h by itself and the others smallest first, and join the running sum as
    // one number
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x4 top[kPair], rest[kPair];
#define DCI_MM(TO_, A_, P_, IN_) \
  _Pragma("unroll") for (int c = 0; c < kPair; ++c) TO_[c] = mfma_bf16(af[t][A_], b[u & 1][c][P_], IN_)
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
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  static_assert(kUnits % 2 == 0, "the next chunk starts with b[0]");
}

template <int C, bool GCN>
__global__ __launch_bounds__(kLayerThreads, 4) void k_sage_layer(LayerArgs a) {
  __shared__ LayerLds lds;
  const long long M = a.counts[a.hop];
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D;
  const long long row_tiles = (M + kLayerRows - 1) / kLayerRows;
  const long long n_tiles = (row_tiles + 7) / 8 * 8 * a.n_col_groups;
  // tile number -> column group and row tile: the column groups of a row tile run on one XCD
  auto place = [&](long long q, int* cg) -> long long {
    const long long j = q >> 3;
    *cg = (int)(j % a.n_col_groups);
    return j / a.n_col_groups * 8 + (q & 7);
  };
  if (tid < kLayerFlags) lds.again[tid] = 0;
  const int n_chunks = (D + kLayerChunk - 1) / kLayerChunk;

  if (wave >= 4) {
    // ---- puts the chunks together, one ahead of the others
    const int pt = tid - 256, gl = pt & 15, grp = pt >> 4;
    const int p_g = (gl & 7) >> 1;
    const int p_slot = (gl >> 3) * 6144 + (p_g * 16 + ((grp + 4 * p_g) & 15)) * 16 + (gl & 1) * 8;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    int buf = 0;
    for (long long q = blockIdx.x; q < n_tiles; q += gridDim.x) {
      int cg;
      const long long rt = place(q, &cg);
      if (rt >= row_tiles) continue;
      const long long row0 = rt * kLayerRows;
      const int rows = M - row0 < kLayerRows ? (int)(M - row0) : kLayerRows;
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
      // A row's sources come in rounds of eight loads; two rounds are on their way at any time, across rows and chunks: a
      // place is asked for again, two rounds on, as soon as it has been added.
      int rounds[2];  // of the wavefront's row with the most
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        int n = deg[t] < kLayerSlots ? deg[t] : kLayerSlots;
        for (int d = 16; d < 64; d <<= 1) {
          const int o = __shfl_xor(n, d, 64);
          n = o > n ? o : n;
        }
        n = __builtin_amdgcn_readfirstlane(n);
        rounds[t] = n > 8 ? (n + 7) / 8 : 1;
      }
      // (written and read by one group of lanes; places without a source, up to the last that a round asks for, hold the row itself)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < kLayerSlots; s += 16)
          if (s < 8 * rounds[t]) lds.src[16 * t + grp][s + gl] = s + gl < deg[t] ? source_row(a, e0[t] + s + gl) : own[t];
      f32x4 v0[8], v1[8], own0, own1;
      int n_k = 0, n_t = 0, n_r = 0;  // the round to ask for next
      auto ask = [&](f32x4 (&v)[8], f32x4& own_v) {
        if (n_k >= n_chunks) return;
        const int k_col = n_k * kLayerChunk + 4 * gl, k_ld = k_col < D - 4 ? k_col : D - 4;
        const float* const* p = &lds.src[16 * n_t + grp][8 * n_r];
        if (n_r == 0) own_v = load4((n_t ? own[1] : own[0]) + k_ld);
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = load4(p[u] + k_ld);
        if (++n_r == (n_t ? rounds[1] : rounds[0])) {
          n_r = 0;
          if (++n_t == 2) {
            n_t = 0;
            ++n_k;
          }
        }
      };
      int k = 0, t = 0, r = 0;  // the round to add
      f32x4 sum = zero, own_v = zero;
      auto add = [&](f32x4 (&v)[8], f32x4& own_new) {
        const int deg_t = t ? deg[1] : deg[0];
        if (r == 0) {
          own_v = own_new;
          sum = GCN ? own_v : zero;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const bool in = 8 * r + u < deg_t;
          sum.x = in ? sum.x + v[u].x : sum.x;
          sum.y = in ? sum.y + v[u].y : sum.y;
          sum.z = in ? sum.z + v[u].z : sum.z;
          sum.w = in ? sum.w + v[u].w : sum.w;
        }
        asm volatile("" : "+v"(sum), "+v"(own_v));  // added here, before the places are asked for again
        ask(v, own_new);
        if (++r < (t ? rounds[1] : rounds[0])) return;
        // the row's part of the chunk is complete
        r = 0;
        const int k_col = k * kLayerChunk + 4 * gl, k_ld = k_col < D - 4 ? k_col : D - 4, shift = k_col - k_ld;
        for (int e = kLayerSlots; e < deg_t; ++e) sum += load4(source_row(a, (t ? e0[1] : e0[0]) + e) + k_ld);
        const float cnt = (float)deg_t + (GCN ? 1.f : 0.f);
        if (a.mode != DCI_MODEL_SAGE_SUM && cnt != 0.f) sum = f32x4{sum.x / cnt, sum.y / cnt, sum.z / cnt, sum.w / cnt};
        if (shift) {
          sum = shifted(sum, shift);
          if (!GCN) own_v = shifted(own_v, shift);
        }
        const bool ok_t = t ? ok[1] : ok[0];
        if (!GCN) put4<false>(&lds.a[buf][0][0][t][0][0] + p_slot, ok_t ? own_v : zero);
        put4<false>(&lds.a[buf][1][0][t][0][0] + p_slot, ok_t ? sum : zero);
        if (++t < 2) return;
        t = 0;
        ++k;
        buf ^= 1;
        __syncthreads();
      };
      ask(v0, own0);
      ask(v1, own1);
      while (true) {
        add(v0, own0);
        if (k == n_chunks) break;
        add(v1, own1);
        if (k == n_chunks) break;
      }
    }
    __syncthreads();
  } else {
    // ---- multiplies
    constexpr int kPair = C < 2 ? 1 : 2;
    typedef __attribute__((address_space(1))) const u32x4* gw_t;
    // the parts of the weights: [operand][k step][column group][wavefront][tile][part][lane]
    const size_t w_step = (size_t)a.n_col_groups * 4 * C * 3 * 1024, w_op = w_step * ((D + 31) / 32);
    const char* const w0 = reinterpret_cast<const char*>(a.w_split) + (size_t)wave * C * 3 * 1024;
    u32x4 b[2][kPair][3];
    int buf = 0, it = 0;
    bool begun = false;
    for (long long q = blockIdx.x; q < n_tiles; q += gridDim.x, ++it) {
      int cg;
      const long long rt = place(q, &cg);
      if (rt >= row_tiles) continue;
      const char* const w_base = w0 + (size_t)cg * 4 * C * 3 * 1024;
      if (!begun) {
#pragma unroll
        for (int c = 0; c < kPair; ++c)
#pragma unroll
          for (int p = 0; p < 3; ++p) b[0][c][p] = *((gw_t)(w_base + (c * 3 + p) * 1024) + lane);
        begun = true;
      }
      // the weights that the tile after this one starts with
      const char* w_after = w_base;
      if (a.n_col_groups > 1 && q + gridDim.x < n_tiles) {
        int cg_n;
        (void)place(q + gridDim.x, &cg_n);
        w_after = w0 + (size_t)cg_n * 4 * C * 3 * 1024;
      }
      f32x4 acc[2][C];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int k = 0; k < n_chunks; ++k, buf ^= 1) {
        __syncthreads();
        const char* w = w_base + (size_t)(2 * k) * w_step;
        // (the last chunk may have one k step of 32 only; the other multiplies zeros with the same weights)
        multiply_chunk<C, GCN>(lds, buf, lane, w, w_op, k * kLayerChunk + 32 < D ? w_step : 0, k + 1 < n_chunks ? w + 2 * w_step : w_after, b, acc);
      }
      bool bad = false;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            bad |= !(__builtin_fabsf(acc[t][c][r]) <= kMaxFloat);
            acc[t][c][r] *= kUnscale;
          }
      const long long row0 = rt * kLayerRows;
      const int rows = M - row0 < kLayerRows ? (int)(M - row0) : kLayerRows;
      if (bad) lds.again[it % kLayerFlags] = 1;
      store_tile<C>(a, row0, rows, (cg * 64 + wave * 16 + (lane & 15)) * C, lane >> 4, acc);
    }
    __syncthreads();
  }
  // tiles with a number that the parts cannot hold, once more (and, past 64 tiles, those whose flag they share)
  int it = 0;
  for (long long q = blockIdx.x; q < n_tiles; q += gridDim.x, ++it) {
    int cg;
    const long long rt = place(q, &cg);
    if (rt >= row_tiles || !lds.again[it % kLayerFlags]) continue;
    const long long row0 = rt * kLayerRows;
    layer_tile_exact<C, GCN>(a, lds, row0, M - row0 < kLayerRows ? (int)(M - row0) : kLayerRows, cg);
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
//     of the line, this kernel / the other: 4,096 rows x 2 x 256 x 64 (256 workgroups), f = 5, 12.3 us / 16.8, x 100 (512) 21.8 / 17.4, x 172
//     (768) 31.0 / 19.6; 1,024 x 2 x 100 x 256 (256), f = 10, 0.78, 2,048 x 2 x 256 x 256 (512), f = 15, 1.5.
//   * above it, the fewest columns per wavefront that make no more than four column groups and five tiles for four compute units: 1 k rows
//     x 2 x 256 x 512, f = 10, with 16 columns (eight groups) 20.7 us, 32 columns 21.8, 64 columns 26.5; 3.1 k (fewer than a fifth of 15,015,
//     291 tiles) x 2 x 75 x 130 with 16 columns 15.8, 32 columns 17.6; 2 k x 2 x 300 x 320, f = 25, with 16 columns (five groups) 43.7, 32
//     columns 36.9; 6 k x 2 x 602 x 192, f = 10, with 64 columns 56, 16 columns, which put the rows together three times in 564 tiles, 78.
//   * neither where lists are long: in few workgroups the lists' latency is not hidden.  With lists of more than 10,000 numbers the
//     layer's two kernels are ahead (x 256 outputs, one kernel / the two; the two have a launch more, 1 - 2 us).  k_sage_layer_small,
//     1,024 rows: D = 100, f = 64 0.86; D = 256, f = 25 0.93, f = 40 30.1 us / 26.3, f = 64 43 / 31; D = 300, f = 40 42 / 29; D = 602, f = 15 33.4
//     / 31.8, f = 25 50 / 36, f = 64 106 / 55.  (Where it has two compute units for every workgroup it is only behind for more
//     than 64 sources times pieces of 256 columns: 512 x 2 x D x 256, D = 256, f = 64 0.97; D = 300, f = 25 1.00, f = 64 1.26; D = 602, f = 25 1.16.)
//     k_sage_layer, 2,048 rows: D = 64, f = 64 21.7 / 29.3; D = 256, f = 25 29.8 / 30.5, f = 64 49.6 / 42.6; D = 300, f = 25 35.6 / 36.1, f = 40 43.3
//     / 40.6; D = 602, f = 25 60 / 53, f = 64 110 / 82.
//   * where there are more tiles than that, as many columns as the layer has, up to 64, because putting a tile's rows together is
//     what takes the time: 18.6 k x 2 x 602 x 256, f = 10, with 64 columns 166 us, 32 columns 162, 16 columns 251.
//   * none of them where the lists are long and every column group puts the same rows together again, or rows are no whole 128-byte
//     lines, so that a piece of 256 bytes touches three.  The aggregation reads them once and in one piece, and the dense
//     layer follows.  18.6 k x 2 x D x N, this kernel / the two: f = 64, 602 x 256 624 us / 534, 602 x 1,024 1,668 / 832, 256 x 256
//     0.83 of the two, 256 x 1,024 1.05; f = 25, 602 x 256 297 / 286, 602 x 1,024 691 / 575, 256 x 256 0.78, 100 x 1,024 1.08; f = 15,
//     602 x 256 0.87, 602 x 512 0.88, 300 x 768 0.78 (60 k rows 1.03).  2 k x 2 x 602 x 256: f = 10 0.88, f = 25 1.11.
//     Where they are even the two are taken: with four lanes they are 5 % ahead (batches of two hops, f = 10 and 25, 68 columns, 144
//     us a batch against 151; on one lane 176 either way).  For the same reason 257 to 384 columns, a second group of 256 for less
//     than half of its columns, are not for these kernels: three layers of 256, 300, 300 and 47 columns, 2,048 seeds, on four lanes 263 us a batch,
//     285 with them, on one lane 305 and 297; from 100 columns 190 and 218, 225 and 230.
constexpr int64_t kSmallReads = 10000;

static size_t split_bytes(const LayerPlan& p, int ops) {
  return (size_t)ops * ((p.D + 31) / 32) * ((p.N + 64 * p.C - 1) / (64 * p.C)) * 4 * p.C * 3 * 1024;
}

// LayerPlan::C.  rows: about what a batch has; fan: the longest list.
static int kernel_for(const dci_ctx* ctx, const LayerPlan& p, int64_t rows, int64_t fan) {
  auto groups = [&](int C) -> int64_t { return (p.N + 64 * C - 1) / (64 * C); };
  const bool short_lists = fan * p.D <= kSmallReads;
  const int64_t wgs = (rows + kSmallRows - 1) / kSmallRows * groups(1);
  if (p.N >= 4 && wgs <= ctx->num_cus)
    return short_lists || (2 * wgs <= ctx->num_cus && fan * ((p.D + kSmallChunk - 1) / kSmallChunk) <= 64) ? 0 : -1;
  for (int C = 1; C <= 4; C *= 2)
    if (groups(C) <= 4 && rows * groups(C) <= (int64_t)ctx->num_cus * kLayerRows * 5 / 4) return short_lists ? C : -1;
  if (p.N > 256 && p.N <= 384) return -1;
  const bool lines = p.D % 32 == 0;  // rows are whole 128-byte lines
  const int C = p.N <= 64 ? 1 : p.N <= 128 ? 2 : 4;
  const int64_t g = groups(C);
  return lines ? (fan * (g + 1) <= 128 ? C : -1) : (fan * (g < 3 ? 3 : g) <= 60 ? C : -1);
}

bool layers_plan(const dci_ctx* ctx, const dci_blocks* blocks, int32_t model, const int32_t* dims, bool input_apart, void* scratch,
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
    p.C = l == 0 && input_apart ? -1 : kernel_for(ctx, p, rows, (blocks->cap_edges[h] + p.cap_rows - 1) / p.cap_rows);
    if (p.C > 0) p.w_split = ar.take<char>(split_bytes(p, ops));
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
    sa.ops[sa.n] = gcn ? 1 : 2;
    sa.wgs += (int)(split_bytes(p, sa.ops[sa.n]) / (4 * 3 * 1024));  // four tiles to a workgroup
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
  a.n_col_groups = (a.N + 64 * plan.C - 1) / (64 * plan.C);
  const int64_t row_tiles = (plan.cap_rows + kLayerRows - 1) / kLayerRows;
  int64_t n = (row_tiles + 7) / 8 * 8 * a.n_col_groups;
  // (a multiple of eight: a workgroup's tiles are then all of one XCD's, and once one is past the last row tile so are those behind it,
  // which the weights fetched ahead rely on)
  const int64_t most = (int64_t)ctx->num_cus * kLayerPerCu / 8 * 8;
  if (n > most) n = most > 8 ? most : 8;
  const dim3 grid((unsigned)n);
#define DCI_LAYER(C_) \
  hipLaunchKernelGGL((gcn ? k_sage_layer<C_, true> : k_sage_layer<C_, false>), grid, dim3(kLayerThreads), 0, ctx->stream, a)
  if (plan.C == 1) DCI_LAYER(1);
  else if (plan.C == 2) DCI_LAYER(2);
  else DCI_LAYER(4);
#undef DCI_LAYER
  DCI_LAUNCH_CHECK(ctx);
  return DCI_OK;
}

}  // namespace dci
