// Projection kernel for problems that fill the chip: one persistent workgroup
// of 8 wavefronts per CU works through tiles of 256 tokens x 32 NS features,
// 4 wavefronts along the tokens x 2 along the features, 4 x NS sub-tiles each.
//
// What bounds it: at full rate a 256 x 256 x 64 step needs 1.07 us of matrix
// pipe (random operands, power limit; 0.87 us on zeros) and 64 KB from L2,
// which delivers about 60 GB/s per CU when all CUs ask (1.07 us); it takes 1.42.
// Against the former 128 x 256 tiles (two workgroups per CU, 32-column stages)
// L2 traffic per multiply-add is down by a third, LDS operand reads by 40%.
// Tried and slower: four wavefronts of 128 x 128 (one per SIMD, nothing to cover
// a wait: 2.4 us per step), two co-resident workgroups of 128 x 192 (901 TFLOP/s
// at 25440 x 3456 x 1152 against 1065), 32-column stages in a deeper ring.
//
// The K slices of all tiles of a workgroup form one stream through two LDS
// stages.  Inside a slice (2 NS steps of one weight sub-tile x 4 token sub-tiles)
// operands are read RING - 1 steps ahead of their MFMAs.  RING - 1 steps before the
// end everything of the slice has been read: there one barrier frees its stage
// and publishes the other, so that the first operands of the next slice are read
// behind the last MFMAs of this one, and the copy of the slice after that starts,
// one round per step (issued together they held up the wavefront's MFMAs).  The
// copies run across tile borders: a tile's first two slices arrive during the
// end of the previous tile and its stores.
//
// Tiles: full ones of 256 tokens first; the remaining token rows are cut into
// tiles of 64, 128, 192 or 256 rows, whichever evens out the last round best
// (25440 x 3456 x 1152: 1200 tiles of 256 x 288 are 4.7 rounds of 256 workgroups, that is 5;
// 85 x 12 full ones and 20 x 12 tail tiles of 192 rows take 4 + 0.82).  The last tile of either axis is moved back to end
// at the matrix edge: rows that two tiles compute are written twice with the same
// bits, and nothing needs a bounds check.
//
// GEMM_NORM (NS = 9): the query / key / value projection finishes the paper's "layernorm2" and "pos emb" on its
// accumulators: a wavefront's 144 features are two whole heads of 72.  The separate pass read and wrote q and k once
// more: 46 us at 25440 tokens, 52 us at 17408 with the rotation, where the epilogue adds about 10 and 20 us.
//
// NS = 8 (256 features): tiles start on cache lines.  NS = 9 (288): fits hidden
// sizes that are multiples of 288 (72-element heads in fours) without padding; the
// odd sub-tile of wave column 1 lies before its pairs, so that all pairs are
// stored from 64-byte boundaries.
#pragma once
#include <type_traits>
#include "gemm_common.hpp"
#include "rope_table.hpp"

namespace pab {

template <int NS, int RING, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_stream_kernel(const GemmParams p) {
  constexpr int BM = 256, BN = 32 * NS, BK = 64;
  constexpr int STAGE = 128 * (BM + BN);         // bytes: token rows, pair rows of the weights, odd sub-tiles
  constexpr int NPAIR = NS / 2;
  constexpr bool ODD = NS % 2 != 0;
  constexpr int W0 = 128 * BM, W1 = W0 + 128 * 64 * NPAIR;   // byte offsets of the pair rows / odd rows in a stage
  constexpr int SHIFT1 = ODD ? 16 : 0;           // features of wave column 1 before its pairs
  constexpr int NDMA = 4 + NPAIR + (ODD ? 1 : 0);   // copy rounds of a wavefront per slice (the last: wavefronts 0-3)
  constexpr int NJ = 2 * NS, AHEAD = RING - 1, JB = NJ - AHEAD;   // steps per slice, operand distance, barrier step
  static_assert(NPAIR % 2 == 0, "pairs are stored two at a time");
  static_assert(NJ % RING == 0 && NDMA <= NJ, "the operand ring continues across slices");
  constexpr int BIAS = 2 * STAGE, XPOSE = BIAS + 2048;   // byte offsets: two bias rows, 2 KB per wavefront
  constexpr bool NORM = EPI == GEMM_NORM;
  constexpr int HD = 72, ROPE = HD / 2 * 8;      // head dim of GEMM_NORM, bytes of one frame's rotary factors
  constexpr int GB = XPOSE + 8 * 2048, FACT = GB + 4 * 2 * HD;   // gamma / beta of q, k; two frames' factors per wavefront
  static_assert(!NORM || NS == 9, "a wavefront's features are two heads of 72");

  __shared__ __attribute__((aligned(16))) unsigned char smem[NORM ? FACT + 8 * 2 * ROPE : GB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, q16 = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char *)smem);
  const int M = p.M, N = p.N, K = p.K, nk = (K + BK - 1) / BK;

  // ---- the workgroup's tiles: unit i of it is number wg + i * gridDim.x; a round of a full grid gives each XCD 32
  //      consecutive units, which are 4 token tiles x 8 feature tiles ----
  struct Tile { int m0, n0, ms; bool second; };
  constexpr bool PAIR = EPI == GEMM_PLAIN;       // the tiles of a second problem come last, where the last round has room
  constexpr int GM = 4;
  const int n_full = p.n_mt * p.n_nt;
  auto unit = [&](int u) __attribute__((always_inline)) {
    Tile t;
    t.second = PAIR && u >= p.n_units - p.n_units2;
    if (t.second) {
      const int r = u - (p.n_units - p.n_units2);
      t.ms = __builtin_amdgcn_readfirstlane(p.ms2);
      t.m0 = __builtin_amdgcn_readfirstlane(min(r / p.n_nt2 * 64 * p.ms2, p.M2 - 64 * p.ms2));
      t.n0 = __builtin_amdgcn_readfirstlane(min(r % p.n_nt2 * BN, p.N2 - BN));
      return t;
    }
    if (u < n_full) {
      const int g = u / (GM * p.n_nt), r = u % (GM * p.n_nt), gm = min(GM, p.n_mt - g * GM);   // the last group may be smaller
      t.m0 = (g * GM + r % gm) * BM; t.n0 = (r / gm) * BN; t.ms = 4;
    } else {
      const int r = u - n_full;
      t.ms = p.ms_tail;
      t.m0 = min(p.n_mt * BM + (r / p.n_nt) * 64 * t.ms, M - 64 * t.ms); t.n0 = (r % p.n_nt) * BN;
    }
    t.n0 = min(t.n0, N - BN);
    t.m0 = __builtin_amdgcn_readfirstlane(t.m0);
    t.n0 = __builtin_amdgcn_readfirstlane(t.n0);
    t.ms = __builtin_amdgcn_readfirstlane(t.ms);
    return t;
  };
  const int wg = gridDim.x == 256 ? (blockIdx.x & 7) * 32 + (blockIdx.x >> 3) : blockIdx.x;
  const int n_mine = (p.n_units - wg + (int)gridDim.x - 1) / (int)gridDim.x;

  // ---- copies: wavefront w moves rows 8 w .. 8 w + 7 of every 64 rows; its lane row lane >> 3, position lane & 7 ----
  const int crow = 8 * wave + (lane >> 3);
  const int cq = (lane & 7) ^ gemm_swizzle(crow);
  const unsigned vfull_a = (unsigned)(2 * (crow * (long long)K + 8 * cq));
  // a round of pair rows: 32 of each wave column; row i: sub-tile i >> 4, operand row i & 15
  const unsigned vfull_w = (unsigned)(2 * (((crow >> 5) * (16 * NS + SHIFT1) + 8 * ((crow & 15) >> 2) + 4 * ((crow >> 4) & 1) +
                                           (crow & 3)) * (long long)K + 8 * cq));
  // odd sub-tiles: the last 16 features of wave column 0, the first 16 of column 1
  const unsigned vfull_s = (unsigned)(2 * (((crow >> 4 ? 16 * NS : 32 * NPAIR) + (crow & 15)) * (long long)K + 8 * cq));
  int s_tile = 0, s_kt = 0, s_ms = 0;            // the copy stream: tile, slice, its token rows / 64
  unsigned voff_a = vfull_a, voff_w = vfull_w, voff_s = vfull_s;   // lane offsets of the slice: a half slice repeats columns 0-31
  bool s_live = false;
  const bf16_t *s_a = p.A, *s_w = p.W, *s_b = p.bias;
  auto stream_tile = [&](int i) __attribute__((always_inline)) {
    const Tile t = unit(wg + i * (int)gridDim.x);
    s_ms = t.ms;
    s_a = (t.second ? p.A2 : p.A) + (long long)t.m0 * K;
    s_w = (t.second ? p.W2 : p.W) + (long long)t.n0 * K;
    s_b = t.second ? p.bias2 : p.bias;
    if (s_b) s_b += t.n0;
  };
  auto copy_round = [&](int stage, int i) __attribute__((always_inline)) {   // round i of the stream's current slice
    if (!s_live) return;
    const unsigned lds = lds0 + STAGE * stage + 1024 * wave;
    if (i < 4) {
      if (i < s_ms) dma16_to_lds(s_a + (long long)64 * i * K, voff_a, lds + 8192 * i);
    } else if (i < 4 + NPAIR) {
      dma16_to_lds(s_w + (long long)32 * (i - 4) * K, voff_w, lds + W0 + 8192 * (i - 4));
    } else if (wave < 4) {
      dma16_to_lds(s_w, voff_s, lds + W1);
    }
  };
  auto next_slice = [&]() __attribute__((always_inline)) {
    if (!s_live) return;
    if (s_kt == 0 && s_b && wave == 7) dma16_to_lds(s_b, 16 * min(lane, BN / 8 - 1), lds0 + BIAS + 1024 * (s_tile & 1));
    s_a += BK;
    s_w += BK;
    if (++s_kt == nk) {
      s_kt = 0;
      if (++s_tile < n_mine) stream_tile(s_tile);
    }
    if (K & 32) {
      const unsigned back = s_kt == nk - 1 && cq >= 4 ? 64 : 0;
      voff_a = vfull_a - back; voff_w = vfull_w - back; voff_s = vfull_s - back;
    }
  };

  if (NORM && tid < 4 * HD) {
    const int which = tid / HD, i = tid % HD;
    const bf16_t *src = which == 0 ? p.gq : which == 1 ? p.bq : which == 2 ? p.gk : p.bk;
    reinterpret_cast<bf16_t *>(smem + GB)[tid] = src[i];
  }
  stream_tile(0);
  for (int stage = 0; stage < 2; ++stage) {      // the first two slices
    s_live = s_tile < n_mine;
#pragma unroll
    for (int i = 0; i < NDMA; ++i) copy_round(stage, i);
    next_slice();
  }
  s_live = false;
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  const int sw = gemm_swizzle(l16);
  const unsigned op = 128 * l16 + 16 * (q16 ^ sw);        // operand address inside 16 rows; columns 32.. : ^ 64
  int stage = 0;

  // ---- GEMM_NORM: bias, then layernorm over the two heads of the wavefront's 144 features and the rotation, on the
  //      accumulators of a tile of plane 0 (q) or 1 (k); plane 2 (v) takes the bias only.  A lane holds chunks of 8 (the
  //      odd sub-tile: 4) consecutive features, each inside one head, and the four lanes of a token hold all of it. ----
  auto norm_heads = [&](auto &acc, const bf16_t *bs, int plane, int m0) __attribute__((always_inline)) {
    // A token that two tiles compute goes through two instantiations of this code (tiles of 64 .. 256 rows): which products
    // are fused is written out, or the compiler chose differently in them and the last bits depended on the tile.
#pragma clang fp contract(off)
    constexpr int MS = sizeof(acc) / sizeof(acc[0]), NCH = NPAIR + 1;
    const int shift = wn ? SHIFT1 : 0, odd = wn ? 0 : 32 * NPAIR;
    auto feature = [&](int c) { return c < NPAIR ? shift + 32 * c + 8 * q16 : odd + 4 * q16; };   // of the 144
    auto value = [&](int a, int c, int e) { return c < NPAIR ? acc[a][2 * c + (e >> 2)][e & 3] : acc[a][NS - 1][e]; };
    auto set = [&](int a, int c, int e, float x) {
      if (c < NPAIR) acc[a][2 * c + (e >> 2)][e & 3] = x;
      else acc[a][NS - 1][e] = x;
    };
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int n = c < NPAIR ? 8 : 4;
      if (p.bias) {
#pragma unroll
        for (int e = 0; e < n; ++e) {
          const float b = (float)bs[feature(c) + e];
#pragma unroll
          for (int a = 0; a < MS; ++a) set(a, c, e, value(a, c, e) + b);
        }
      }
    }
    if (plane > 1) return;
    float mean[MS][2], rstd[MS][2];
    auto across = [](float x) {   // over the four lanes of a token
      x += __shfl_xor(x, 16);
      return x + __shfl_xor(x, 32);
    };
#pragma unroll
    for (int a = 0; a < MS; ++a) {
      float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        float s = 0.0f;
#pragma unroll
        for (int e = 0; e < (c < NPAIR ? 8 : 4); ++e) s += value(a, c, e);
        const bool second = feature(c) >= HD;
        s0 += second ? 0.0f : s;
        s1 += second ? s : 0.0f;
      }
      mean[a][0] = across(s0) * (1.0f / HD);
      mean[a][1] = across(s1) * (1.0f / HD);
      s0 = s1 = 0.0f;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const bool second = feature(c) >= HD;
        const float m = second ? mean[a][1] : mean[a][0];
        float s = 0.0f;
#pragma unroll
        for (int e = 0; e < (c < NPAIR ? 8 : 4); ++e) {
          const float d = value(a, c, e) - m;
          set(a, c, e, d);
          s = __builtin_fmaf(d, d, s);
        }
        s0 += second ? 0.0f : s;
        s1 += second ? s : 0.0f;
      }
      rstd[a][0] = 1.0f / sqrtf(__builtin_fmaf(across(s0), 1.0f / HD, p.eps));
      rstd[a][1] = 1.0f / sqrtf(__builtin_fmaf(across(s1), 1.0f / HD, p.eps));
      __builtin_amdgcn_sched_barrier(0);
    }
    // rotary factors of the one or two frames that the wavefront's (at most 64) tokens lie in: frames have 64 or more
    const int frame0 = m0 / p.S, frame1 = (m0 + 16 * MS - 1) / p.S;
    const unsigned fact = lds0 + FACT + 2 * ROPE * wave;
    if (p.rope) {
#pragma unroll
      for (int i = lane; i < HD; i += 64) {
        const f32x2 f = rope_factor<HD>(i < HD / 2 ? frame0 : frame1, i % (HD / 2));
        *(__attribute__((address_space(3))) f32x2 *)(size_t)(fact + 8 * i) = f;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    const bf16_t *gamma = reinterpret_cast<const bf16_t *>(smem + GB) + 2 * HD * plane, *beta = gamma + HD;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int n = c < NPAIR ? 8 : 4;
      const bool second = feature(c) >= HD;
      const int d0 = feature(c) - (second ? HD : 0);          // inside the head
      float g[8], b[8];
#pragma unroll
      for (int e = 0; e < n; ++e) {
        g[e] = (float)gamma[d0 + e];
        b[e] = (float)beta[d0 + e];
      }
#pragma unroll
      for (int a = 0; a < MS; ++a) {
        const float r = second ? rstd[a][1] : rstd[a][0];
#pragma unroll
        for (int e = 0; e < n; ++e) set(a, c, e, __builtin_fmaf(value(a, c, e) * r, g[e], b[e]));
      }
      if (p.rope) {
        auto factors = [&](unsigned frame, f32x4 *f) {
#pragma unroll
          for (int i = 0; i < n / 4; ++i) f[i] = *(const __attribute__((address_space(3))) f32x4 *)(size_t)(fact + frame + 4 * d0 + 16 * i);
        };
        auto rotate = [&](int a, const f32x4 *f) {
#pragma unroll
          for (int i = 0; i < n / 2; ++i) {
            const float x = value(a, c, 2 * i), y = value(a, c, 2 * i + 1), cs = f[i / 2][2 * (i & 1)], sn = f[i / 2][2 * (i & 1) + 1];
            set(a, c, 2 * i, __builtin_fmaf(x, cs, -(y * sn)));
            set(a, c, 2 * i + 1, __builtin_fmaf(x, sn, y * cs));
          }
        };
        f32x4 f[2];
        factors(0, f);
        if (frame0 == frame1) {
#pragma unroll
          for (int a = 0; a < MS; ++a) rotate(a, f);
        } else {
#pragma unroll
          for (int a = 0; a < MS; ++a) {
            factors(m0 + 16 * a + l16 >= frame1 * p.S ? ROPE : 0, f);
            rotate(a, f);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  auto run_tile = [&](auto ms_tag, const Tile t, int parity) __attribute__((always_inline)) {
    constexpr int MS = decltype(ms_tag)::value;            // token sub-tiles of a wavefront
    f32x4 acc[MS][NS];
    bf16x8 tf[2][MS], wf[RING];                            // token operands of both column halves, ring of weight operands
    unsigned tb, wb;
    auto use_stage = [&](int s) __attribute__((always_inline)) {
      tb = lds0 + STAGE * s + 2048 * MS * wm + op;
      wb = lds0 + STAGE * s + W0 + 4096 * wn + op;
    };
    auto rd_t = [&](int ks, int a) __attribute__((always_inline)) { tf[ks][a] = lds_read8((ks ? tb ^ 64 : tb) + 2048 * a); };
    auto rd_w = [&](int j) __attribute__((always_inline)) {
      const int b = j % NS;
      const unsigned off = b < 2 * NPAIR ? 8192 * (b >> 1) + 2048 * (b & 1) : W1 - W0 - 2048 * wn;
      return lds_read8((j / NS ? wb ^ 64 : wb) + off);
    };
    use_stage(stage);
#pragma unroll
    for (int a = 0; a < MS; ++a) rd_t(0, a);
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) wf[j] = rd_w(j);
#pragma unroll
    for (int a = 0; a < MS; ++a)
#pragma unroll
      for (int b = 0; b < NS; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[a][b][e] = 0.0f;

    // one slice; HALF: the last one of an odd multiple of 32 columns, whose columns 32-63 do not exist and are not computed
    auto slice = [&](auto half_tag) __attribute__((always_inline)) {
      constexpr bool HALF = decltype(half_tag)::value;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j == JB) {   // this slice has been read, the next one has arrived
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
          s_live = s_tile < n_mine;
          stage ^= 1;
          use_stage(stage);
#pragma unroll
          for (int a = 0; a < MS; ++a) rd_t(0, a);
        }
        const int d = (j - JB + NJ) % NJ;   // steps since the barrier
        if (d < NDMA) copy_round(stage ^ 1, d);
        if (d == NDMA - 1) next_slice();
        if (!HALF || j + AHEAD < NS || j + AHEAD >= NJ) wf[(j + AHEAD) % RING] = rd_w((j + AHEAD) % NJ);
        if (!HALF && j >= 1 && j <= MS) rd_t(1, j - 1);
        if (!HALF || j < NS) {
#pragma unroll
          for (int a = 0; a < MS; ++a) acc[a][j % NS] = mfma16(wf[j % RING], tf[j / NS][a], acc[a][j % NS]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    for (int kt = 0; kt < K / BK; ++kt) slice(std::false_type{});
    if (K & 32) slice(std::true_type{});

    const int shift = wn ? SHIFT1 : 0, odd = wn ? 0 : 32 * NPAIR;   // where the pairs / the odd sub-tile start
    const bf16_t *bs = reinterpret_cast<const bf16_t *>(smem + BIAS + 1024 * parity) + wn * 16 * NS;
    const int f0 = t.n0 + wn * 16 * NS, m0 = t.m0 + wm * 16 * MS;
    const bool bias = (t.second ? p.bias2 : p.bias) != nullptr;
    bf16_t *const C = t.second ? p.C2 : p.C;
    if constexpr (NORM) norm_heads(acc, bs, t.n0 / p.n_split, m0);
    // ---- bias, activation, stores: 16 tokens x 64 features at a time through the wavefront's 2 KB ----
    const unsigned xs = lds0 + XPOSE + 2048 * wave;
    const unsigned xw = xs + 128 * l16, xr = xs + 128 * (lane >> 3) + 16 * ((lane & 7) ^ gemm_swizzle(lane >> 3));
#pragma unroll
    for (int h = 0; h < NPAIR / 2; ++h) {
      float bv[2][8];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8 b8 = zero8();
        if (!NORM && bias) b8 = *reinterpret_cast<const bf16x8 *>(bs + shift + 64 * h + 32 * u + 8 * q16);
#pragma unroll
        for (int e = 0; e < 8; ++e) bv[u][e] = (float)b8[e];
      }
      const int n = f0 + shift + 64 * h + 8 * (lane & 7), plane = n / p.n_split;
      bf16_t *dst = C + plane * p.plane_stride + (n - plane * p.n_split) + (long long)(m0 + (lane >> 3)) * p.ldc;
#pragma unroll
      for (int a = 0; a < MS; ++a) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          bf16x8 y;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = acc[a][4 * h + 2 * u + (e >> 2)][e & 3] + bv[u][e];
            y[e] = (bf16_t)(EPI == GEMM_GELU ? gelu(x) : x);
          }
          lds_write8(xw + 16 * ((4 * u + q16) ^ sw), y);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const bf16x8 r0 = lds_read8(xr), r1 = lds_read8((xr ^ 64) + 1024);   // rows 8 further: swizzle ^ 4
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        *reinterpret_cast<bf16x8 *>(dst) = r0;
        *reinterpret_cast<bf16x8 *>(dst + 8 * p.ldc) = r1;
        dst += 16 * p.ldc;
      }
    }
    if (ODD) {
      bf16x4 b4;
#pragma unroll
      for (int e = 0; e < 4; ++e) b4[e] = (bf16_t)0.0f;
      if (!NORM && bias) b4 = *reinterpret_cast<const bf16x4 *>(bs + odd + 4 * q16);
      const int n = f0 + odd + 8 * (lane & 1), plane = n / p.n_split;
      bf16_t *dst = C + plane * p.plane_stride + (n - plane * p.n_split) + (long long)(m0 + (lane >> 1)) * p.ldc;
#pragma unroll
      for (int a = 0; a < MS; ++a) {
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = acc[a][NS - 1][e] + (float)b4[e];
          y[e] = (bf16_t)(EPI == GEMM_GELU ? gelu(x) : x);
        }
        lds_write4(xs + 32 * (16 * a + l16) + 8 * q16, y);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int a = 0; a < (MS + 1) / 2; ++a) {
        const bf16x8 r = lds_read8(xs + 1024 * a + 16 * lane);
        if (2 * a + 1 < MS || lane < 32) *reinterpret_cast<bf16x8 *>(dst + 32 * a * p.ldc) = r;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  };

  for (int i = 0; i < n_mine; ++i) {
    const Tile t = unit(wg + i * (int)gridDim.x);
    if (t.ms == 4) run_tile(std::integral_constant<int, 4>{}, t, i & 1);
    else if (t.ms == 3) run_tile(std::integral_constant<int, 3>{}, t, i & 1);
    else if (t.ms == 2) run_tile(std::integral_constant<int, 2>{}, t, i & 1);
    else run_tile(std::integral_constant<int, 1>{}, t, i & 1);
  }
}

}  // namespace pab
