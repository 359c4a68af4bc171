// Rotary factors (cos, sin)(pos * theta_i), theta_i = 10000^(-2i / D), as constant data of the library: tables of
// the digits of pos in base 64, (cos, sin)(digit * 64^k * theta_i) for k = 0 .. 4, computed in double by the compiler
// (one exponential series for theta_1 / theta_0, powers by multiplication, one sine / cosine series per pair, digits and
// 64-fold angles by complex multiplication) and rounded once to fp32.  A factor is the product of the
// entries of its nonzero digits; calling sincosf for every element instead made the rotary pass 20 us longer than its memory traffic.
#pragma once
#include "mfma_util.hpp"

namespace pab {

constexpr int ROPE_BASE = 64, ROPE_DIGITS = 5;   // positions below 64^5

template <int D> struct RopeTable {
  float v[ROPE_DIGITS][ROPE_BASE][D / 2][2];
};

template <int D> constexpr RopeTable<D> make_rope_table() {
  RopeTable<D> t{};
  const double x = -2.0 * 9.210340371976182736 / D;   // ln(10000)
  double ratio = 1.0, term = 1.0;
  for (int n = 1; n < 25; ++n) {
    term *= x / n;
    ratio += term;
  }
  double theta = 1.0;                                  // at most 1: the series below converge fast
  for (int i = 0; i < D / 2; ++i) {
    double c = 1.0, s = theta, tc = 1.0, ts = theta;
    for (int n = 1; n < 12; ++n) {
      tc *= -theta * theta / ((2 * n - 1) * (2 * n));
      ts *= -theta * theta / ((2 * n) * (2 * n + 1));
      c += tc;
      s += ts;
    }
    for (int k = 0; k < ROPE_DIGITS; ++k) {
      double pc = 1.0, ps = 0.0;
      for (int d = 0; d < ROPE_BASE; ++d) {
        t.v[k][d][i][0] = (float)pc;
        t.v[k][d][i][1] = (float)ps;
        const double nc = pc * c - ps * s;
        ps = pc * s + ps * c;
        pc = nc;
      }
      c = pc;                                          // 64 times the angle
      s = ps;
    }
    theta *= ratio;
  }
  return t;
}

template <int D> __device__ constexpr RopeTable<D> rope_table = make_rope_table<D>();

typedef __attribute__((ext_vector_type(2))) float f32x2;

// factor of position pos >= 0 and feature pair i; the fused products are written out, so that it has the same bits wherever it is inlined
template <int D> __device__ __forceinline__ f32x2 rope_factor(int pos, int i) {
#pragma clang fp contract(off)
  const RopeTable<D> &t = rope_table<D>;
  f32x2 f = {t.v[0][pos % ROPE_BASE][i][0], t.v[0][pos % ROPE_BASE][i][1]};
  for (int k = 1; k < ROPE_DIGITS; ++k) {
    pos /= ROPE_BASE;
    if (pos == 0) break;
    const float c = t.v[k][pos % ROPE_BASE][i][0], s = t.v[k][pos % ROPE_BASE][i][1];
    f = f32x2{__builtin_fmaf(f[0], c, -(f[1] * s)), __builtin_fmaf(f[0], s, f[1] * c)};
  }
  return f;
}

}  // namespace pab
