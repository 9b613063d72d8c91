// Fp32 numbers as sums of three bf16 numbers: what k_sage_layer and k_sage_layer_small multiply, and the weights in that form.
#ifndef DCI_PARTS_H_
#define DCI_PARTS_H_

#include "dci_internal.h"

namespace dci {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef f32x4 __attribute__((aligned(4))) f32x4_u;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Two numbers as three pairs of bf16: x = h + m + l.
struct Split2 {
  unsigned h, m, l;
};
__device__ __forceinline__ Split2 split2(float x0, float x1) {
  Split2 s;
  f32x2 x = {x0, x1};
  s.h = __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2));
  x.x -= __builtin_bit_cast(float, s.h << 16);
  x.y -= __builtin_bit_cast(float, s.h & 0xFFFF0000u);
  s.m = __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2));
  x.x -= __builtin_bit_cast(float, s.m << 16);
  x.y -= __builtin_bit_cast(float, s.m & 0xFFFF0000u);
  s.l = __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2));
  return s;
}

// The matrix instructions take a bf16 number below 2^-126 for zero, so both operands are scaled by 2^24: the last bit of the
// smallest fp32 number is then 2^-125, and no part of a number is lost.  What grows too large that way (a number of
// 2^104, a sum of 2^80) shows as an infinity.
constexpr float kScale = 16777216.f, kUnscale = 1.f / (16777216.f * 16777216.f);

// Pieces of 16 C columns that the parts of N columns are: whole blocks of 64 columns, and no more, whatever the number of wavefronts that
// read them, because a layer whose parts do not fit into the scratch takes the whole pass to two kernels a layer.
__host__ __device__ constexpr int parts_pieces(int N, int C) { return (N + 63) / 64 * 4 / C; }

// The weights of a forward pass's layers as parts, in the order in which k_sage_layer's lanes hold them.
struct SplitArgs {
  int n = 0;                 // layers
  int wgs = 0;               // workgroups in all
  int first[DCI_MAX_HOPS + 1];  // first workgroup of each
  const float* w[DCI_MAX_HOPS][2];  // self, neighbour (GCN: the one matrix in the first place)
  void* out[DCI_MAX_HOPS];
  int D[DCI_MAX_HOPS], N[DCI_MAX_HOPS], C[DCI_MAX_HOPS], ops[DCI_MAX_HOPS];
  int waves[DCI_MAX_HOPS];  // pieces of 16 C columns
};

// Workgroup `block` (256 threads) of SplitArgs::wgs.
__device__ __forceinline__ void split_weights(const SplitArgs& a, int block) {
  int l = 0;
  while (l + 1 < a.n && block >= a.first[l + 1]) ++l;
  const int D = a.D[l], N = a.N[l], C = a.C[l];
  const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
  // one wavefront per tile of 32 rows by 16 columns: [operand][k step][piece][tile]
  const int id = (block - a.first[l]) * 4 + (int)(threadIdx.x >> 6);
  const int n32 = (D + 31) / 32, n_w = a.waves[l];
  const int c = id % C, w = id / C % n_w, ks = id / C / n_w % n32, op = id / C / n_w / n32;
  if (op >= a.ops[l]) return;
  const int col = (w * 16 + r16) * C + c;
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = 32 * ks + 8 * g + j;
    v[j] = k < D && col < N ? a.w[l][op][(long long)k * N + col] * kScale : 0.f;
  }
  u32x4 p[3];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const Split2 s = split2(v[2 * jj], v[2 * jj + 1]);
    p[0][jj] = s.h;
    p[1][jj] = s.m;
    p[2][jj] = s.l;
  }
  u32x4* out = reinterpret_cast<u32x4*>(a.out[l]) + (size_t)id * 3 * 64 + lane;
  for (int q = 0; q < 3; ++q) out[q * 64] = p[q];
}

}  // namespace dci

#endif  // DCI_PARTS_H_
