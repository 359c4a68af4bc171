// Projections of the attention module (paper App. B.5: "qkv proj", "o proj")
// and of the MLP module: C[M, N] = act(A[M, K] W[N, K]^T + bias[N]),
// activations and weights bf16, fp32 accumulation on the matrix core, one
// rounding to bf16 on the way out; act is nothing or the MLP's GELU.
//
// Both operands are contiguous along K, which is what the MFMA operands want:
// with the weight rows as the A operand and the token rows as the B operand a
// 16 x 16 sub-tile is C^T[n, m], every lane owns one token and 4 of its outputs.
// Three kernels share the layouts below: gemm_stream.hpp for problems that fill
// the chip with large tiles, gemm_tile.hpp for the others, gemm_heads.hpp for
// few tokens where q and k are normalised per head behind the projection.
//
// Operand layout in LDS.  A stage holds 64 columns of K of a tile's token rows
// and weight rows, 128 bytes per row = one cache line: with 32 columns (half
// lines) the same kernel ran at 816 instead of 901 TFLOP/s (25440 x 3456 x
// 1152), because L2 serves a half line at the price of a whole one.  A copy
// round of a wavefront (one global -> LDS instruction) is 8 rows; row r's 16-byte
// chunk q is stored at position q ^ ((r >> 1) & 7).  A 16-byte LDS read is served
// in four cycles of 16 lanes, lanes {0-3, 12-15, 20-23, 24-27} together, then
// {4-7, 8-11, 16-19, 28-31}, and the same in the upper half; an operand read
// (lane = 16 chunk + row) therefore mixes chunk q of rows 0-3, 12-15 with chunk
// q ^ 1 of rows 4-11, which this permutation sends to 16 different bank groups
// (bank conflict counter: 0).
//
// K may be an odd multiple of 32.  The upper half of the last slice then repeats
// the lower one in LDS and is not computed: zeros against the repeated weights
// would turn an infinite weight into a NaN.
//
// Weight rows of a pair of sub-tiles are taken in the order 8 (i >> 2) + 4 u +
// (i & 3) (sub-tile u, operand row i), so that the two accumulators of a lane are
// 8 consecutive features, the 16 bytes of a store.
//
// Stores.  A lane's 16 bytes belong to token l16, so storing them from the
// accumulator layout would hand the 16 lanes of a quarter wavefront 16 different
// rows: that pattern sustains 29 GB/s per CU where consecutive lanes on
// consecutive 16 bytes of a 128-byte segment reach 76 (288-byte rows 93).  The
// results therefore take a turn through 2 KB of LDS per wavefront (same swizzle)
// and leave as 128-byte segments.
#pragma once
#include "mfma_util.hpp"

namespace pab {

struct GemmParams {
  const bf16_t *A;      // [M, K]
  const bf16_t *W;      // [N, K]
  const bf16_t *bias;   // [N] or nullptr
  bf16_t *C;            // feature n of token m goes to C[(n / n_split) * plane_stride + m * ldc + n % n_split]
  int M, N, K;
  long long ldc;        // row pitch of C in elements
  int n_split;          // features per output plane (N: one plane; else a multiple of 8)
  long long plane_stride;
  int n_mt, n_nt;       // token / feature tiles (gemm_stream: n_mt full token tiles)
  int by_feature;       // gemm_tile, gemm_heads: 1: consecutive tiles share their features, 0: their tokens,
  int n_inner, n_inner2;   // ... as many as there are token (1) or feature tiles (0), of the first and of the second problem
  int ms_tail;          // gemm_stream: the token rows behind the full tiles are cut into tiles of 64 ms_tail rows
  int n_units;          // gemm_stream: full tiles (n_mt x n_nt), then tail tiles, then those of the second problem
  // GEMM_PLAIN: a second problem of the same K, ldc, n_split and plane_stride in the same launch (n_units2 = 0: none)
  const bf16_t *A2, *W2, *bias2;
  bf16_t *C2;
  int M2, N2, n_nt2, n_units2;
  int ms2;              // gemm_stream: token rows / 64 of its tiles
  // GEMM_NORM (gemm_stream: heads of 72, gemm_tile: of 32) and gemm_heads, the query / key / value projection: layernorm over the head
  // dimension of planes 0 and 1, then the rotation
  const bf16_t *gq, *bq, *gk, *bk;   // [head dim] scale and shift for q and for k
  int S, rope;          // tokens per frame (frame index = token / S); 1: rotate by the frame index (gemm_stream: S >= 64)
  unsigned S_magic;     // gemm_tile: 2^32 / S, at most 2^32 - 1
  float eps;
};

enum { GEMM_PLAIN = 0, GEMM_GELU = 1, GEMM_NORM = 2 };   // what happens to the sums

// chunk permutation of stage row r
__device__ __forceinline__ int gemm_swizzle(int r) { return (r >> 1) & 7; }

typedef const __attribute__((address_space(3))) bf16x8 *lds_cptr8;
typedef __attribute__((address_space(3))) bf16x8 *lds_ptr8;
typedef __attribute__((address_space(3))) bf16x4 *lds_ptr4;
__device__ __forceinline__ bf16x8 lds_read8(unsigned addr) { return *(lds_cptr8)(size_t)addr; }
__device__ __forceinline__ void lds_write8(unsigned addr, bf16x8 v) { *(lds_ptr8)(size_t)addr = v; }
__device__ __forceinline__ void lds_write4(unsigned addr, bf16x4 v) { *(lds_ptr4)(size_t)addr = v; }

// GELU in its tanh form: 0.5 x (1 + tanh u) = x / (1 + exp(-2u)), u = sqrt(2/pi) (x + 0.044715 x^3)
// (fused product written out: the same bits wherever it is inlined, see gemm_stream.hpp on rows that two tiles compute)
__device__ __forceinline__ float gelu(float x) {
#pragma clang fp contract(off)
  const float u2 = -2.302208198f * __builtin_fmaf(0.044715f * x * x, x, x);   // -2 sqrt(2/pi) log2(e) (..)
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u2));
}

}  // namespace pab
