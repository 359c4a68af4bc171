// Attention of small launches: o = softmax(q k^T / sqrt(D)) v per (batch, head), the same operation as attn_tile16.hpp with its
// sub-tiles, operand layouts and lazy running maximum, for launches whose time is latency and not work.
//
// What bounds such a launch there is the chain that one workgroup goes through: 2 us of address arithmetic before its first
// request, a barrier per step of the ring, and a combination in which one wavefront in four does the work (5 frames of 252
// tokens and 8 heads, 10.3 us per launch: set-up 2.0, two steps 3.5, combination 1.7, stores 0.8, all of 8.9 us that a
// workgroup lives).  Here a wavefront is on its own until the end: it has a 32-query tile and every G-th 32-key tile, copies
// its K and V tiles into LDS of its own (the next K while the softmax runs, the next V at the end of the step) and meets the
// other key groups of its query tile at one barrier, behind which all of them take a share of the rows: partial sums with the
// denominator and the maximum beside them, read, weighed, added and stored 16 bytes per lane in row order.
// 10.3 -> 6.9 us there; 4 frames of 128 tokens and 8 heads 7.0 -> 4.1, 4 of 500 and 8 13.1 -> 9.5, 4 of 64 and 4 (heads of
// 32, fp32) 4.3 -> 2.8, 48 frames at 1590 positions, 16 heads 350 -> 166, cross attention of 1000 tokens and 8 heads to 300 keys
// 16.3 -> 6.1.
//
// The price is that a K/V tile serves 32 queries instead of 256: with many query tiles the copies take longer than the arithmetic.
// 64 rows of 144 bytes are 129 cache lines as counted; 9 frames of 462 tokens and 8 heads (17.2 us) draw 61 GB/s per CU, all that L2
// gives when every CU asks, 5 of 252 only 26.  plan_short and plan_short_cross in launch_plan.hpp have the lines.
#pragma once
#include "attn_short_layout.hpp"
#include "mfma_util.hpp"

namespace pab {

struct ShortParams {
  const void *q, *k, *v;
  void *o;
  int sq, sk, n_head;
  int n_blk;                     // workgroups of a problem
  int n_work;                    // ... of all (batch, head) problems
  unsigned blk_magic, head_magic;  // ceil(2^32 / n_blk), ceil(2^32 / n_head): quotients by a high product
  long long q_bs, kv_bs;         // batch strides of q / o and of k / v, elements
  int q_ss, kv_ss;               // sequence strides, elements
  float c;                       // log2(e) / sqrt(D)
};

typedef __attribute__((ext_vector_type(2))) float f32x2_t;

template <typename T> struct Chunk;   // 8 elements as loaded
template <> struct Chunk<bf16_t> {
  bf16x8 x;
  __device__ __forceinline__ void load(const bf16_t *p) { x = *reinterpret_cast<const bf16x8 *>(p); }
  __device__ __forceinline__ bf16x8 get() const { return x; }
};
template <> struct Chunk<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float *p) {
    a = *reinterpret_cast<const f32x4 *>(p);
    b = *reinterpret_cast<const f32x4 *>(p + 4);
  }
  __device__ __forceinline__ bf16x8 get() const {
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = (bf16_t)a[e];
      v[4 + e] = (bf16_t)b[e];
    }
    return v;
  }
};

// maximum over the four lanes that share a query (lane bits 4 and 5), without the LDS crossbar
__device__ __forceinline__ float max_quad16(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// NW wavefronts: NW / G query tiles with G key groups each.  ZERO: V rows past the last key are zeros, as in the cross kernels, whose
// small launches these are; else copies of that key's row, as in the tile kernel
template <typename T, int D, int NW, int G, bool ZERO>
__global__ __launch_bounds__(64 * NW, sizeof(T) == 4 ? 2 : 4) void attn_short_kernel(const ShortParams p) {
  constexpr int CH = D / 8;                  // 8-element chunks of a row
  constexpr int QT = NW / G;                 // query tiles of a workgroup
  constexpr int RP = SHORT_PITCH<D>;         // pitch of K and V rows in LDS
  constexpr int DT16 = (D + 1 + 15) / 16;
  constexpr int OP = D + 4;                  // floats of a partial row: D sums, denominator, maximum, two unused
  constexpr int KV_BYTES = 2 * 32 * RP * 2, O_BYTES = 32 * OP * 4;
  constexpr int REGION = KV_BYTES > O_BYTES ? KV_BYTES : O_BYTES;   // of a wavefront: K tile and V tile, later its partial O
  constexpr int REM = D % 32;
  constexpr bool REM16 = REM > 0 && REM <= 16;
  constexpr int KS = D / 32;
  constexpr bool DIRECT = sizeof(T) == 2;
  static_assert(REM == 0 || REM == 8, "head dim");
  constexpr int RPL = 64 / (CH + 1), NL = (32 + RPL - 1) / RPL;   // rows per copy, copies per tile
  __shared__ __attribute__((aligned(16))) unsigned char smem[NW * REGION];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int qt = wave / G, kg = wave % G;
  // workgroup ids go round-robin over the 8 XCDs: each takes a contiguous eighth of the blocks, so that the blocks of a problem
  // share an L2 copy of its keys and no XCD has more to do than another (against every eighth problem 0.94 of the time over 274
  // shapes, 0.6 where problems are few and not a multiple of 8)
  const unsigned per = gridDim.x >> 3, id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (id >= (unsigned)p.n_work) return;
  const unsigned bh = p.n_blk == 1 ? id : __umulhi(id, p.blk_magic), blk = id - bh * p.n_blk;
  const unsigned batch = p.n_head == 1 ? bh : __umulhi(bh, p.head_magic), head = bh - batch * p.n_head;
  const T *qb = reinterpret_cast<const T *>(p.q) + batch * p.q_bs + head * D;
  const T *kb = reinterpret_cast<const T *>(p.k) + batch * p.kv_bs + head * D;
  const T *vb = reinterpret_cast<const T *>(p.v) + batch * p.kv_bs + head * D;
  T *ob = reinterpret_cast<T *>(p.o) + batch * p.q_bs + head * D;
  const int sq = p.sq, sk = p.sk, q_ss = p.q_ss, kv_ss = p.kv_ss;
  const int q0 = (blk * QT + qt) * 32;
  const int ntile = (sk + 31) >> 5;
  bf16_t *kt = reinterpret_cast<bf16_t *>(smem + wave * REGION), *vt = kt + 32 * RP;
  const unsigned lds_kv = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char *)smem) + wave * REGION;

  // copy i of a tile: rows RPL i + lane / (CH + 1), CH chunks each; the lane behind them idles
  const int crow = lane / (CH + 1), ccol = lane % (CH + 1);
  const bool clive = ccol < CH && crow < RPL;
  // bf16 rows go straight to LDS.  fp32 rows are rounded on the way: those of K come in operand layout and stay in registers,
  // those of V pass through registers
  Chunk<T> kc[2][KS], vc[NL];
  f32x4 kc4[2];
  auto request = [&](const T *base, int t, bool is_v) __attribute__((always_inline)) {
    if constexpr (DIRECT) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int row = RPL * i + crow;
        if (clive && (RPL * (i + 1) <= 32 || row < 32))
          dma16_to_lds(base, 2u * (unsigned)(min(32 * t + row, sk - 1) * kv_ss + 8 * ccol), lds_kv + (is_v ? 64 * RP : 0) + 2 * RPL * RP * i);
      }
    } else if (is_v) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int row = RPL * i + crow;
        if (clive && (RPL * (i + 1) <= 32 || row < 32)) vc[i].load(base + (unsigned)(min(32 * t + row, sk - 1) * kv_ss + 8 * ccol));
      }
    } else {
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        const T *src = base + (unsigned)(min(32 * t + 16 * kh + l16, sk - 1) * kv_ss);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kc[kh][ks].load(src + 32 * ks + 8 * g4);
        kc4[kh] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (REM16 && g4 < 2) kc4[kh] = *reinterpret_cast<const f32x4 *>(src + 32 * KS + 4 * g4);
      }
    }
  };
  if (kg < ntile) request(kb, kg, false);

  bf16x8 qf[2][KS];
  bf16x4 qr[2];
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const T *src = qb + (unsigned)(min(q0 + 16 * qh + l16, sq - 1) * q_ss);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[qh][ks] = Io<T>::load8(src + 32 * ks + 8 * g4);
#pragma unroll
    for (int e = 0; e < 4; ++e) qr[qh][e] = (bf16_t)0.0f;
    if (REM16 && g4 < 2) qr[qh] = Io<T>::load4(src + 32 * KS + 4 * g4);
  }
  if (kg < ntile) request(vb, kg, true);
  // what lies behind the rows: zeros (K, columns that the 16-column step covers), the constant chunk (V).  No copy touches it
  if (lane < 32) {
    bf16x8 one = zero8();
    *reinterpret_cast<bf16x8 *>(kt + lane * RP + D) = one;
    one[0] = (bf16_t)1.0f;
    *reinterpret_cast<bf16x8 *>(vt + lane * RP + D) = one;
  }
  f32x4 oacc[DT16][2];
  float m_run[2], m_thr[2], m_negc[2];
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    m_run[qh] = -INFINITY;
    m_thr[qh] = -INFINITY;
    m_negc[qh] = 0.0f;
#pragma unroll
    for (int dt = 0; dt < DT16; ++dt)
#pragma unroll
      for (int r = 0; r < 4; ++r) oacc[dt][qh][r] = 0.0f;
  }
  const float c = p.c, thr = 8.0f / c;
  const bf16_t *k_src = kt + l16 * RP + 8 * g4, *kr_src = kt + l16 * RP + 32 * KS + 4 * g4;
  const bf16_t *v_row = vt + (4 * g4 + (l16 >> 2)) * RP;

  for (int t = kg; t < ntile; t += G) {
    // what was requested has landed (the copies are invisible to the compiler)
    if constexpr (DIRECT) {
      __builtin_amdgcn_s_waitcnt(0x0F70);
    } else {
#pragma unroll
      for (int i = 0; i < NL; ++i)
        if (clive && (RPL * (i + 1) <= 32 || RPL * i + crow < 32))
          *reinterpret_cast<bf16x8 *>(vt + (RPL * i + crow) * RP + 8 * ccol) = vc[i].get();
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // ---- S^T = K Q^T ----
    f32x4 S[2][2];
    bf16x8 kf[2][KS];
    bf16x4 kr[2];
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[kh][ks] = DIRECT ? *reinterpret_cast<const bf16x8 *>(k_src + 16 * kh * RP + 32 * ks) : kc[kh][ks].get();
      if (REM16) {
        if (DIRECT) kr[kh] = *reinterpret_cast<const bf16x4 *>(kr_src + 16 * kh * RP);
        else
#pragma unroll
          for (int e = 0; e < 4; ++e) kr[kh][e] = (bf16_t)kc4[kh][e];
      }
    }
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
#pragma unroll
        for (int r = 0; r < 4; ++r) S[kh][qh][r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) S[kh][qh] = mfma16(kf[kh][ks], qf[qh][ks], S[kh][qh]);
      }
    if (REM16) {
      mfma_shape_change(S[0][0], S[0][1], S[1][0], S[1][1]);
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int qh = 0; qh < 2; ++qh) S[kh][qh] = mfma16_k16(kr[kh], qr[qh], S[kh][qh]);
    }
    if (DIRECT) __builtin_amdgcn_s_waitcnt(0xC07F);   // the reads of K are done before a copy may overwrite it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (t + G < ntile) request(kb, t + G, false);
    if (32 * t + 32 > sk) {
      // rows past the last key are copies of it and weigh 0: zeros, or an infinity of that key would become NaN.  Two lanes per
      // row, the chunk in the middle twice.  0.1 us of a launch
      if (ZERO && 32 * t + (lane >> 1) >= sk) {
#pragma unroll
        for (int i = 0; i < (CH + 1) / 2; ++i) *reinterpret_cast<bf16x8 *>(vt + (lane >> 1) * RP + 8 * (i + (lane & 1) * (CH / 2))) = zero8();
      }
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (32 * t + 16 * kh + 4 * g4 + r >= sk) {
            S[kh][0][r] = -INFINITY;
            S[kh][1][r] = -INFINITY;
          }
    }
    float mx[2];
    bool grow = false;
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) {
      float a = fmaxf(fmaxf(S[0][qh][0], S[0][qh][1]), S[0][qh][2]);
      a = fmaxf(fmaxf(a, S[0][qh][3]), S[1][qh][0]);
      a = fmaxf(fmaxf(a, S[1][qh][1]), S[1][qh][2]);
      mx[qh] = fmaxf(a, S[1][qh][3]);
      grow |= mx[qh] > m_thr[qh];
    }
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        const float m_new = fmaxf(m_run[qh], max_quad16(mx[qh]));
        // another query of the wavefront grows; this one may have seen no key but of score -inf: it weighs nothing and stays 0
        const bool none = m_new == -INFINITY;
        const float alpha = none ? 1.0f : __builtin_amdgcn_exp2f((m_run[qh] - m_new) * c);
        m_run[qh] = m_new;
        m_thr[qh] = m_new + thr;
        m_negc[qh] = none ? 0.0f : -m_new * c;
#pragma unroll
        for (int dt = 0; dt < DT16; ++dt)
#pragma unroll
          for (int r = 0; r < 4; ++r) oacc[dt][qh][r] *= alpha;
      }
    }
    bf16x8 pf[2];
#pragma unroll
    for (int qh = 0; qh < 2; ++qh)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          pf[qh][4 * kh + r] = (bf16_t)__builtin_amdgcn_exp2f(__builtin_fmaf(S[kh][qh][r], c, m_negc[qh]));
#pragma unroll
    for (int dt = 0; dt < DT16; ++dt) {
      const bf16_t *v_src = v_row + short_v_column<D>(dt, l16 & 3);
      const bf16x4 lo = lds_read_tr4(v_src), hi = lds_read_tr4(v_src + 16 * RP);
      bf16x8 vf;
      vf[0] = lo[0]; vf[1] = lo[1]; vf[2] = lo[2]; vf[3] = lo[3];
      vf[4] = hi[0]; vf[5] = hi[1]; vf[6] = hi[2]; vf[7] = hi[3];
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) oacc[dt][qh] = mfma16(vf, pf[qh], oacc[dt][qh]);
    }
    if (DIRECT) __builtin_amdgcn_s_waitcnt(0xC07F);   // ... and those of V
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (t + G < ntile) request(vb, t + G, true);
  }

  // ---- partial rows to LDS: D sums, denominator, maximum ----
  float *part = reinterpret_cast<float *>(smem + wave * REGION);
#pragma unroll
  for (int qh = 0; qh < 2; ++qh)
#pragma unroll
    for (int dt = 0; dt < DT16; ++dt)
      if (16 * dt + 4 * g4 <= D) {
        f32x4 y = oacc[dt][qh];
        if (dt == D / 16 && g4 == D % 16 / 4) y[1] = m_run[qh];   // behind the denominator
        *reinterpret_cast<f32x4 *>(part + (16 * qh + l16) * OP + 16 * dt + 4 * g4) = y;
      }
  if (G > 1) __syncthreads();
  else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const float *first = reinterpret_cast<const float *>(smem + qt * G * REGION);
#pragma unroll
  for (int pass = 0; pass < (32 * CH + 64 * G - 1) / (64 * G); ++pass) {
    const int i = 64 * (G * pass + kg) + lane;
    const int row = i / CH, ch = i - row * CH;
    if (i < 32 * CH && q0 + row < sq) {
      const float *src = first + row * OP;
      f32x2_t lm[G];
      f32x4 xa[G], xb[G];
      float m_all = -INFINITY;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        lm[g] = *reinterpret_cast<const f32x2_t *>(src + g * (REGION / 4) + D);
        xa[g] = *reinterpret_cast<const f32x4 *>(src + g * (REGION / 4) + 8 * ch);
        xb[g] = *reinterpret_cast<const f32x4 *>(src + g * (REGION / 4) + 8 * ch + 4);
        m_all = fmaxf(m_all, lm[g][1]);
      }
      float den = 0.0f;
      f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f}, b = a;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        // a group that saw no key (or only keys of score -inf) has m = -inf and nothing accumulated: its factor is 0, not NaN
        const float s = G == 1 ? 1.0f : lm[g][1] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((lm[g][1] - m_all) * c);
        den += lm[g][0] * s;
        a += xa[g] * s;
        b += xb[g] * s;
      }
      const float inv = 1.0f / den;
      T *dst = ob + (unsigned)((q0 + row) * q_ss) + 8 * ch;
      if (sizeof(T) == 2) {
        bf16x8 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) { y[e] = (bf16_t)(a[e] * inv); y[4 + e] = (bf16_t)(b[e] * inv); }
        *reinterpret_cast<bf16x8 *>(dst) = y;
      } else {
        *reinterpret_cast<f32x4 *>(dst) = a * inv;
        *reinterpret_cast<f32x4 *>(dst + 4) = b * inv;
      }
    }
  }
}

}  // namespace pab
