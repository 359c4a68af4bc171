// Query / key / value projection of few tokens with the paper's "layernorm2" and "pos emb" behind it: gemm_tile's K loop on
// tiles of BM tokens x BN features, BN whole heads, one workgroup per CU.  Like there the latency of the K loop is the
// bound, so KG groups of WM x WN wavefronts take the slices g (mod KG), each through a ring of its own.
//
// The groups' sums meet in LDS as one fp32 tile.  A head's elements lie across several wavefronts; its statistics are taken
// by four lanes per (token, head), and what leaves is 16 bytes per lane with consecutive lanes on consecutive chunks of a
// row.  The separate pass over q and k that this replaces is a launch of 4 - 5 us: temporal module of 1260 tokens and 576
// features 28.0 -> 23.8 us, a small clip's blocks 1996 -> 1845.  Tiles of 128 tokens (two LDS stages per group instead of three)
// take what has more 64-token tiles than CUs: spatial module of 2400 tokens and 576 features 40.7 -> 35.8, 1280 of 1152
// 53.8 -> 47.5, 4000 of 288 31.2 -> 27.2.
#pragma once
#include "gemm_common.hpp"
#include "rope_table.hpp"

namespace pab {

template <int WM, int WN, int MS, int NS, int NST, int KG, int HD>
__global__ __launch_bounds__(64 * WM * WN * KG, WM * WN * KG / 4) void gemm_heads_kernel(const GemmParams p) {
  constexpr int NW = WM * WN, BM = 16 * MS * WM, BN = 16 * NS * WN, BK = 64;
  constexpr int ROWS = BM + BN, STAGE = 128 * ROWS;      // bytes
  constexpr int ROUNDS = ROWS / 8, MYR = (ROUNDS + NW - 1) / NW;   // copy rounds of a slice, per wavefront (the last may repeat)
  constexpr int CP = BN + 4;                             // pitch of the fp32 tile
  constexpr int HPT = BN / HD, STATS = 4 * BM * CP;      // heads of a tile; byte offset of the statistics behind the tile
  constexpr int CPT = BN / 8, THREADS = 64 * NW * KG;    // 16-byte chunks of a tile row
  static_assert(BM % 8 == 0 && BN % HD == 0 && HD % 8 == 0, "tiles of whole heads");
  static_assert((NST == 2 || NST == 3) && MYR < 16, "vmcnt immediates");
  static_assert(STATS + 8 * BM * HPT <= KG * NST * STAGE, "the epilogue must fit the rings");
  static_assert(4 * BM * HPT % 64 == 0, "whole wavefronts take the statistics");

  __shared__ __attribute__((aligned(16))) unsigned char smem[KG * NST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int kg = __builtin_amdgcn_readfirstlane(tid >> 6) / NW, wave = __builtin_amdgcn_readfirstlane(tid >> 6) % NW;
  const int l16 = lane & 15, q16 = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char *)smem) + NST * STAGE * kg;

  // every XCD takes a contiguous run of tiles, in the order in which it touches fewer rows (tile_order in launch_plan.hpp)
  const int n_tiles = p.n_mt * p.n_nt, per = (n_tiles + 7) >> 3;
  const int id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || id >= n_tiles) return;
  const int outer = id / p.n_inner, in = id - outer * p.n_inner;
  const int m0 = (p.by_feature ? in : outer) * BM, n0 = (p.by_feature ? outer : in) * BN;
  const int M = p.M, N = p.N, K = p.K, nk = (K + BK - 1) / BK;

  // round r copies stage rows 8 r .. 8 r + 7, token rows first; rows past the matrix re-read its last one
  auto my_round = [&](int i) { return min(wave + NW * i, ROUNDS - 1); };
  unsigned voff[MYR], vback[MYR];                        // byte offset; what a half slice takes off it to repeat columns 0-31
#pragma unroll
  for (int i = 0; i < MYR; ++i) {
    const int row = 8 * my_round(i) + (lane >> 3), cq = (lane & 7) ^ gemm_swizzle(row);
    const int src = row < BM ? min(m0 + row, M - 1) : min(n0 + row - BM, N - 1);
    voff[i] = (unsigned)(2 * (src * (long long)K + 8 * cq));
    vback[i] = cq >= 4 ? 64 : 0;
  }
  auto issue = [&](int kt, int stage) __attribute__((always_inline)) {
    const long long k0 = (long long)__builtin_amdgcn_readfirstlane(kt) * BK;
    const bool half = (K & 32) && kt == nk - 1;
#pragma unroll
    for (int i = 0; i < MYR; ++i) {
      const int r = my_round(i);
      dma16_to_lds((r < BM / 8 ? p.A : p.W) + k0, voff[i] - (half ? vback[i] : 0), lds0 + STAGE * stage + 1024 * r);
    }
  };
  const int n_mine = (nk - kg + KG - 1) / KG, n_step = (nk + KG - 1) / KG;   // slices of this group; steps of all groups
  const int npre = n_mine < NST - 1 ? n_mine : NST - 1;
  for (int s = 0; s < npre; ++s) issue(KG * s + kg, s);

  // accumulators of the first group start from the bias: a lane's features of sub-tile b are 16 b + 4 q16 + 0..3
  f32x4 acc[MS][NS];
#pragma unroll
  for (int b = 0; b < NS; ++b) {
    const int n = n0 + 16 * (wn * NS + b) + 4 * q16;
    f32x4 bv = {0.0f, 0.0f, 0.0f, 0.0f};
    if (kg == 0 && p.bias && n < N) {
      const bf16x4 b4 = *reinterpret_cast<const bf16x4 *>(p.bias + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[e] = (float)b4[e];
    }
#pragma unroll
    for (int a = 0; a < MS; ++a) acc[a][b] = bv;
  }
  const unsigned op = 128 * l16 + 16 * (q16 ^ gemm_swizzle(l16));
  const unsigned t_off = 128 * wm * 16 * MS + op, w_off = 128 * (BM + wn * 16 * NS) + op;

  int stage = 0, next = npre % NST;
  for (int s = 0; s < n_step; ++s) {
    // slice s of the group has landed (this wavefront's share); one more may be in flight
    if (NST == 3 && s + 1 < n_mine) __builtin_amdgcn_s_waitcnt(0x0F70 | MYR);
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();                        // ... everyone's share; all are done with slice s - 1
    if (s + NST - 1 < n_mine) {
      issue(KG * (s + NST - 1) + kg, next);
      next = next + 1 == NST ? 0 : next + 1;
    }
    if (KG > 1 && s >= n_mine) break;       // the last step, for groups that have no slice left
    const int kt = KG * s + kg;
    const unsigned st = lds0 + STAGE * stage;
    stage = stage + 1 == NST ? 0 : stage + 1;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if (ks == 1 && (K & 32) && kt == nk - 1) break;
      bf16x8 tf[MS], wf[NS];
#pragma unroll
      for (int a = 0; a < MS; ++a) tf[a] = lds_read8(st + (ks ? t_off ^ 64 : t_off) + 2048 * a);
#pragma unroll
      for (int b = 0; b < NS; ++b) wf[b] = lds_read8(st + (ks ? w_off ^ 64 : w_off) + 2048 * b);
#pragma unroll
      for (int b = 0; b < NS; ++b)
#pragma unroll
        for (int a = 0; a < MS; ++a) acc[a][b] = mfma16(wf[b], tf[a], acc[a][b]);
    }
  }

  // ---- the groups' sums as one fp32 tile, row-major, one group after the other (the rings are free) ----
  float *tile = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int g = 0; g < KG; ++g) {
    __syncthreads();
    if (kg == g) {
#pragma unroll
      for (int a = 0; a < MS; ++a)
#pragma unroll
        for (int b = 0; b < NS; ++b) {
          f32x4 *t = reinterpret_cast<f32x4 *>(tile + (16 * (wm * MS + a) + l16) * CP + 16 * (wn * NS + b) + 4 * q16);
          *t = g ? *t + acc[a][b] : acc[a][b];
        }
    }
  }
  __syncthreads();
  f32x2 *stats = reinterpret_cast<f32x2 *>(smem + STATS);   // [row][head]: mean, 1 / standard deviation
  for (int i = tid >> 2; i < BM * HPT; i += THREADS / 4) {
    const float *h = tile + i / HPT * CP + i % HPT * HD + 2 * (lane & 3);
    f32x2 v[HD / 8];
    float s = 0.0f, ss = 0.0f;
#pragma unroll
    for (int e = 0; e < HD / 8; ++e) {
      v[e] = *reinterpret_cast<const f32x2 *>(h + 8 * e);
      s += v[e][0] + v[e][1];
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    const float mean = s * (1.0f / HD);
#pragma unroll
    for (int e = 0; e < HD / 8; ++e) {
      const float d0 = v[e][0] - mean, d1 = v[e][1] - mean;
      ss += d0 * d0 + d1 * d1;
    }
    ss += __shfl_xor(ss, 1);
    ss += __shfl_xor(ss, 2);
    if ((lane & 3) == 0) stats[i] = f32x2{mean, 1.0f / sqrtf(ss * (1.0f / HD) + p.eps)};
  }
  __syncthreads();
  for (int i = tid; i < BM * CPT; i += THREADS) {
    const int row = i / CPT, c = i % CPT, m = m0 + row, n = n0 + 8 * c;
    if (m >= M || n >= N) continue;         // N is a multiple of 8
    const float *t = tile + row * CP + 8 * c;
    const f32x4 lo = *reinterpret_cast<const f32x4 *>(t), hi = *reinterpret_cast<const f32x4 *>(t + 4);
    float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    const int plane = n / p.n_split;
    if (plane < 2) {
      const int head = 8 * c / HD, d0 = 8 * c - head * HD;
      const f32x2 st = stats[row * HPT + head];
      const bf16x8 g = *reinterpret_cast<const bf16x8 *>((plane ? p.gk : p.gq) + d0);
      const bf16x8 b = *reinterpret_cast<const bf16x8 *>((plane ? p.bk : p.bq) + d0);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (v[e] - st[0]) * st[1] * (float)g[e] + (float)b[e];
      if (p.rope) {
        const int frame = m / p.S;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const f32x2 f = rope_factor<HD>(frame, (d0 + e) / 2);
          const float x = v[e], y = v[e + 1];
          v[e] = x * f[0] - y * f[1];
          v[e + 1] = x * f[1] + y * f[0];
        }
      }
    }
    bf16x8 y;
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = (bf16_t)v[e];
    *reinterpret_cast<bf16x8 *>(p.C + plane * p.plane_stride + (n - plane * p.n_split) + m * p.ldc) = y;
  }
}

}  // namespace pab
