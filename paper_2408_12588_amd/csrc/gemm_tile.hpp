// Projection kernel for everything that does not fill the chip with the large
// tiles of gemm_stream.hpp: one workgroup per tile, WM x WN wavefronts of MS x NS
// sub-tiles, K in slices of 64 columns through a ring of NST LDS stages, copied
// NST - 1 slices ahead, one barrier per slice.
//
// Such a problem is bound by the latency of its K loop, not by a rate: a slice
// of a lone 64 x 64 tile takes 0.26 us, of a 128 x 128 tile 0.55 us, so the host
// picks the smallest tile that the L2 traffic allows (about 60 GB/s per CU).
// 1260 x 576 x 2304: 33.8 us with the former 128 x 256 tiles on 15 CUs, 13.9 us
// with 180 tiles of 64 x 64, 10.1 with the K groups below; 1260 x 1728 x 576: 13.8 -> 9.0 us.
//
// The latency is that of barrier, operand reads and MFMAs, one behind the other,
// with one wavefront per SIMD: more slices in flight did not help (4, 6, 9 stages:
// 5.4 -> 5.6 .. 6.2 us at 1260 x 576 x 576), more wavefronts do.  Where every tile has a
// CU to itself, KG groups of WM x WN wavefronts share it: group g takes the
// slices g (mod KG) through a ring of its own, and the groups' fp32 sums are added
// through LDS at the end (1260 x 576 x 2304 13.9 -> 10.1 us with three groups).
// Two groups also take tiles of 96, 160 and 192 tokens x 128 features: the loop is one
// round, so its length is that of the tile; the next height up costs less than a second
// round of 128 tokens (4413 x 1008 x 4032 53.6 -> 39.7 us with 160, 5709 x 1024 x 4096
// 54.8 -> 45.3 with 192).
#pragma once
#include <type_traits>
#include "gemm_common.hpp"
#include "rope_table.hpp"

namespace pab {

template <int WM, int WN, int MS, int NS, int NST, int KG, int EPI>
__global__ __launch_bounds__(64 * WM * WN * KG, KG > 1 ? WM * WN * KG / 4 : 2) void gemm_tile_kernel(const GemmParams p) {
  constexpr int NW = WM * WN, BM = 16 * MS * WM, BN = 16 * NS * WN, BK = 64;
  constexpr int ROWS = BM + BN, STAGE = 128 * ROWS;      // bytes
  constexpr int ROUNDS = ROWS / 8, MYR = ROUNDS / NW, TOKR = BM / 8 / NW;   // copy rounds: all, per wavefront, of token rows
  constexpr int SEG = NS >= 4 ? 64 : 32;                 // features stored at a time
  static_assert(ROUNDS % NW == 0 && (BM / 8) % NW == 0, "copy rounds must deal evenly to the wavefronts");
  static_assert(NS % 2 == 0 && (NS == 2 || NS % 4 == 0), "sub-tiles come in pairs");
  static_assert(NST >= 2 && NST <= 3 && (NST - 2) * MYR < 16, "vmcnt immediates");
  constexpr int PART = 1024 * MS * NS * NW;              // bytes of a group's sums
  static_assert(NW * 2048 + (KG - 1) * PART <= KG * NST * STAGE, "output staging must fit the rings");

  __shared__ __attribute__((aligned(16))) unsigned char smem[KG * NST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int kg = __builtin_amdgcn_readfirstlane(tid >> 6) / NW, wave = __builtin_amdgcn_readfirstlane(tid >> 6) % NW;
  const int l16 = lane & 15, q16 = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const unsigned lds_all = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char *)smem);
  const unsigned lds0 = lds_all + NST * STAGE * kg;      // the group's ring

  // every XCD takes a contiguous run of tiles, in the order in which it touches fewer rows (tile_order in launch_plan.hpp)
  constexpr bool PAIR = EPI == GEMM_PLAIN;               // the tiles of a second problem follow those of the first
  const int n_first = p.n_mt * p.n_nt, n_tiles = n_first + (PAIR ? p.n_units2 : 0), per = (n_tiles + 7) >> 3;
  int id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || id >= n_tiles) return;
  const bool second = PAIR && id >= n_first;
  id -= second ? n_first : 0;
  const bf16_t *A = second ? p.A2 : p.A, *W = second ? p.W2 : p.W, *bias = second ? p.bias2 : p.bias;
  bf16_t *C = second ? p.C2 : p.C;
  const int M = second ? p.M2 : p.M, N = second ? p.N2 : p.N, inner = second ? p.n_inner2 : p.n_inner;
  const int outer = id / inner, in = id - outer * inner;
  const int m0 = (p.by_feature ? in : outer) * BM, n0 = (p.by_feature ? outer : in) * BN;
  const int K = p.K, nk = (K + BK - 1) / BK;

  // round r = wave + NW i: stage rows 8 r .. 8 r + 7, token rows first.  Rows past the matrix re-read its last row; what
  // they produce is never stored.  LDS row i of a 32-row weight pair: sub-tile i >> 4, operand row i & 15.
  unsigned voff[MYR];
  const int cq = (lane & 7) ^ gemm_swizzle(8 * wave + (lane >> 3));   // 8 NW rows further the swizzle is the same
  static_assert(NW % 2 == 0, "swizzle period of 16 rows");
#pragma unroll
  for (int i = 0; i < MYR; ++i) {
    const int row = 8 * (wave + NW * i) + (lane >> 3);
    int src;
    if (i < TOKR) {
      src = min(m0 + row, M - 1);
    } else {
      const int w = row - BM;
      src = min(n0 + (w & ~31) + 8 * ((w & 15) >> 2) + 4 * ((w >> 4) & 1) + (w & 3), N - 1);
    }
    voff[i] = (unsigned)(2 * (src * (long long)K + 8 * cq));
  }
  auto issue = [&](int kt, int stage) __attribute__((always_inline)) {
    const long long k0 = (long long)__builtin_amdgcn_readfirstlane(kt) * BK;
    const unsigned back = (K & 32) && kt == nk - 1 && cq >= 4 ? 64 : 0;   // a half slice repeats columns 0-31
#pragma unroll
    for (int i = 0; i < MYR; ++i)
      dma16_to_lds((i < TOKR ? A : W) + k0, voff[i] - back, lds0 + STAGE * stage + 1024 * (wave + NW * i));
  };
  // group g takes the slices kt = g (mod KG); all groups go through the same number of steps
  const int n_mine = (nk - kg + KG - 1) / KG, n_step = (nk + KG - 1) / KG;
  const int npre = n_mine < NST - 1 ? n_mine : NST - 1;
  for (int s = 0; s < npre; ++s) issue(KG * s + kg, s);

  // accumulators start from the bias: lane's features of sub-tile b are 32 (b / 2) + 8 q16 + 4 (b % 2) + 0..3
  f32x4 acc[MS][NS];
#pragma unroll
  for (int b = 0; b < NS; ++b) {
    const int n = n0 + wn * 16 * NS + 32 * (b >> 1) + 8 * q16 + 4 * (b & 1);
    f32x4 bv = {0.0f, 0.0f, 0.0f, 0.0f};
    if (kg == 0 && bias && n < N) {
      const bf16x4 b4 = *reinterpret_cast<const bf16x4 *>(bias + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[e] = (float)b4[e];
    }
#pragma unroll
    for (int a = 0; a < MS; ++a) acc[a][b] = bv;
  }
  const int sw = gemm_swizzle(l16);
  const unsigned op = 128 * l16 + 16 * (q16 ^ sw);
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

  if (KG > 1) {   // groups 1 .. leave their sums in LDS, 16 bytes per lane, group 0 adds them to its own
    __syncthreads();
    typedef __attribute__((address_space(3))) f32x4 *lds_ptr_f4;
    const unsigned part = lds_all + 2048 * NW + 1024 * MS * NS * wave + 16 * lane;
    if (kg) {
#pragma unroll
      for (int a = 0; a < MS; ++a)
#pragma unroll
        for (int b = 0; b < NS; ++b) *(lds_ptr_f4)(size_t)(part + PART * (kg - 1) + 1024 * (NS * a + b)) = acc[a][b];
    }
    __syncthreads();
    if (kg) return;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g)
#pragma unroll
      for (int a = 0; a < MS; ++a)
#pragma unroll
        for (int b = 0; b < NS; ++b) acc[a][b] += *(lds_ptr_f4)(size_t)(part + PART * g + 1024 * (NS * a + b));
  }

  if constexpr (EPI == GEMM_NORM) {
    // query / key / value projection, heads of 32: a pair of sub-tiles is one head of 16 tokens, 8 consecutive elements in each
    // of the four lanes of a token
    auto across = [](float x) {   // sum over those lanes (lane bits 4 and 5)
      const auto u = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      x = __uint_as_float(u[0]) + __uint_as_float(u[1]);
      const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      return __uint_as_float(v[0]) + __uint_as_float(v[1]);
    };
    f32x2 turn[MS][4];
    if (p.rope) {
#pragma unroll
      for (int a = 0; a < MS; ++a) {
        const int m = m0 + 16 * (wm * MS + a) + l16;
        int frame = (int)__umulhi((unsigned)m, p.S_magic);   // m / S or one less
        frame += m - frame * p.S >= p.S;
#pragma unroll
        for (int e = 0; e < 4; ++e) turn[a][e] = rope_factor<32>(frame, 4 * q16 + e);
      }
    }
#pragma unroll
    for (int u = 0; u < NS / 2; ++u) {
      const int n = n0 + wn * 16 * NS + 32 * u, plane = (n >= p.n_split) + (n >= 2 * p.n_split);
      if (plane > 1) continue;
      const bf16x8 g8 = *reinterpret_cast<const bf16x8 *>((plane ? p.gk : p.gq) + 8 * q16);
      const bf16x8 b8 = *reinterpret_cast<const bf16x8 *>((plane ? p.bk : p.bq) + 8 * q16);
#pragma unroll
      for (int a = 0; a < MS; ++a) {
        float v[8], s = 0.0f, ss = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = acc[a][2 * u + (e >> 2)][e & 3];
          s += v[e];
        }
        const float mean = across(s) * (1.0f / 32);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] -= mean;
          ss += v[e] * v[e];
        }
        const float rstd = 1.0f / sqrtf(across(ss) * (1.0f / 32) + p.eps);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] * rstd * (float)g8[e] + (float)b8[e];
        if (p.rope) {
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const f32x2 f = turn[a][e / 2];
            const float x = v[e], y = v[e + 1];
            v[e] = x * f[0] - y * f[1];
            v[e + 1] = x * f[1] + y * f[0];
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[a][2 * u + (e >> 2)][e & 3] = v[e];
      }
    }
  }

  // ---- activation, stores: 16 tokens x SEG features at a time through 2 KB per wavefront (the ring is free) ----
  if (KG == 1) __syncthreads();
  constexpr int CPR = SEG / 8, RPI = 64 / CPR;           // chunks per row segment, rows per store instruction
  auto xpos = [](int row, int q) { return SEG == 64 ? q ^ gemm_swizzle(row) : q ^ ((row >> 2) & 2); };
  const unsigned xs = lds0 + 2048 * wave;
  const int mw = m0 + wm * 16 * MS;
#pragma unroll
  for (int h = 0; h < 16 * NS / SEG; ++h) {
    const int fw = n0 + wn * 16 * NS + SEG * h;          // first feature of the segment
    const int n = fw + 8 * (lane % CPR), plane = n / p.n_split;
    bf16_t *dst = C + plane * p.plane_stride + (n - plane * p.n_split);
#pragma unroll
    for (int a = 0; a < MS; ++a) {
#pragma unroll
      for (int u = 0; u < SEG / 32; ++u) {
        bf16x8 y;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = acc[a][SEG / 16 * h + 2 * u + (e >> 2)][e & 3];
          y[e] = (bf16_t)(EPI == GEMM_GELU ? gelu(x) : x);
        }
        lds_write8(xs + 2 * SEG * l16 + 16 * xpos(l16, 4 * u + q16), y);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int i = 0; i < 16 / RPI; ++i) {
        const int row = RPI * i + lane / CPR, m = mw + 16 * a + row;
        const bf16x8 r = lds_read8(xs + 2 * SEG * row + 16 * xpos(row, lane % CPR));
        if (m < M && n + 8 <= N) {
          *reinterpret_cast<bf16x8 *>(dst + m * p.ldc) = r;
        } else if (m < M && n < N) {   // N is a multiple of 4: the last chunk of a row may be half
          bf16x4 lo;
          lo[0] = r[0]; lo[1] = r[1]; lo[2] = r[2]; lo[3] = r[3];
          *reinterpret_cast<bf16x4 *>(dst + m * p.ldc) = lo;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
}

}  // namespace pab
