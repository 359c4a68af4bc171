// How a call is cut into launches: which problems of the tile kernel are split, which projection kernel and tile.  Plain
// arithmetic on sizes without any device code, so that a host program can ask which way a shape takes.
#pragma once
#include <algorithm>

namespace pab {

constexpr int TILE_NWV = 8;       // wavefronts per workgroup: 256 queries share each staged K/V tile (4: 1.5-2% slower)
constexpr int TILE_SPLIT_G = 4;   // key groups of a split item
constexpr int TILE_CUS = 32;      // CUs of an XCD; a CU holds two workgroups (16 wavefronts)

struct ItemPlan {
  int n_item;            // workgroups of a plain problem
  long long bh_plain;    // the first problems, run as plain items; the others are split
  long long n_split;     // workgroups of a split problem (0: none is split)
};

// Split items (a quarter of the queries, four key groups: a quarter of the steps) for some problems, or for all.  An XCD
// takes every eighth (batch, head) problem and has TILE_CUS CUs; workgroups take about the same time, so an XCD's time
// steps up where its workgroups pass a multiple of TILE_CUS, by half with the second workgroup of a CU (S = 1024, 16 heads:
// 29.0 us with 24 per XCD, 43.3 with 36), by a whole one with the third.  The problems beyond the last multiple are split,
// all of them if there is none (most of those launches are plan_short's, which is asked first), where the XCD with the most of their
// items has no more than
//   one per CU (72 problems of 1024 tokens 44.1 -> 32.8 us, 66 of 788 35.4 -> 26.0, 84 of 700 32.0 -> 25.0, 16 of 1024 with fp32 rows
//     40.0 -> 25.1), from 8 key tiles: with fewer the combination costs more than the steps that it saves;
//   after an even multiple, where they would wait for a whole round: two per CU for long sequences (6 of 3600 79.6 -> 50.1, 136 of
//     1000 67.6 -> 58.4, 40 of 3600 204 -> 193, 16 of 1100 with fp32 rows 40.5 -> 34.5; but 48 of 512, from before there was the short
//     kernel, 17.0 -> 17.6);
//   after an odd one, where they would run beside the others: two or three per CU for longer ones still, whose items are
//     cheaper (24 of 2871, 45 items per XCD, 101 -> 77, 10 of 4640, 73 items, 157 -> 136; but 84 of 912, 45 items, 39.8 -> 47.3,
//     110 of 677 34.0 -> 40.0); with fp32 rows, which are converted on the way in by four times as many items, fewer (heads of
//     32: 33 of 2481, 80 items, 80 -> 84; of 72: 32 of 1984, 50 items, 82 -> 89).
// Failing that, those over the last full round of two workgroups per CU, if that is at most a quarter round (91 of 3066, fp32:
// 499 -> 472; but 224 of 562 with 160 workgroups over 41.0 -> 45.8).
// More items than that only lose: 10 of 6103 queries and 448 keys (fp32) 33 -> 50 with 96 on an XCD.  752 shapes (heads of 32 and 72, both types, 1 .. 2800 problems): 0.89 of the time of
// the former rule (a rest of at most a quarter of the last round, 16 key tiles); none that is split is slower by more than 3 %.
inline ItemPlan plan_items(long long n_bh, int sq, int sk, int head_dim, int elem_size) {
  constexpr int QBLK = 32 * TILE_NWV;
  ItemPlan p{(sq + QBLK - 1) / QBLK, n_bh, 0};
  const int ntile = (sk + 31) / 32;
  const long long n_split = (sq + QBLK / TILE_SPLIT_G - 1) / (QBLK / TILE_SPLIT_G);
  const long long per_xcd = (n_bh + 7) / 8 * p.n_item, multiple = per_xcd / TILE_CUS;
  auto items_xcd = [&](long long plain) { return (n_bh - plain + 7) / 8 * n_split; };   // split items of the fullest XCD
  const long long beyond = per_xcd % TILE_CUS ? multiple * TILE_CUS / p.n_item * 8 : n_bh;
  const long long rest = n_bh * p.n_item % (16 * TILE_CUS), round = n_bh - rest / p.n_item;
  int most = ntile >= 8 ? TILE_CUS : 0;
  if (multiple % 2 == 0) most = ntile >= 32 ? 2 * TILE_CUS : most;
  else if (elem_size == 2 && ntile >= 64) most = 3 * TILE_CUS;
  else if (elem_size == 2 || head_dim == 32) most = ntile >= 40 ? 2 * TILE_CUS : ntile >= 32 ? 3 * TILE_CUS / 2 : most;
  else most = ntile >= 64 ? 3 * TILE_CUS / 2 : most;
  if (beyond < n_bh && items_xcd(beyond) <= most) p.bh_plain = beyond;
  else if (per_xcd > 2 * TILE_CUS && ntile >= 16 && rest <= 4 * TILE_CUS && items_xcd(round) <= 2 * TILE_CUS) p.bh_plain = round;
  if (p.bh_plain < n_bh) p.n_split = n_split;
  return p;
}

// Small launches take attn_short.hpp: 10 times its wavefronts plus its key groups, or 0 for another kernel.
//
// Key groups: what a wavefront does one after the other is ntile / groups steps, the more groups the shorter, while the chip is
// not full of wavefronts; then blocks in pairs of wavefronts, two blocks with two groups each, four blocks without groups.  us,
// heads of 72: 15 tiles, 360 blocks 22: 10.2, 44: 9.2; 8 tiles, 1040 blocks 22: 10.5, 42: 10.8, 44: 11.6; 9 blocks of a problem,
// 1440 in all 22: 13.4, 42: 11.5; 256 problems of 225 tokens 22: 16.5, 42: 16.3, 41: 14.0.  fp32 rows of heads of 72 leave registers for
// two wavefronts per SIMD, so that a 513th block of four waits for a second round: 128 of 133 tokens (640) 44: 14.6, 22: 10.4.
inline int short_groups(long long n_blocks, long long blk, int ntile, int head_dim, int elem_size) {
  if (ntile <= 2) return n_blocks <= 256 || ntile == 1 ? 22 : 42;
  const long long four = elem_size == 4 && head_dim == 72 && ntile < 16 ? 512 : 650;
  if (n_blocks <= 256 || (ntile >= 5 && n_blocks <= four) || (head_dim == 32 && ntile >= 16)) return 44;
  if (n_blocks > 1450 && (blk % 4 == 0 || blk >= 32)) return 41;
  if (ntile == 4 || ntile >= 16 || (n_blocks > 1200 && (blk % 2 == 0 || blk >= 9))) return 42;
  return 22;
}

// A 32-query block there loads the keys for itself, so its time goes with the number of blocks; the tile kernel's with the key
// tiles of a workgroup, the rounds of workgroups on the fullest XCD and, where problems are split, the split items.  The line is a
// number of blocks, lower for what the tile kernel does well.  us, tile kernel -> short:
//   bf16, heads of 72: 96 problems of 256 tokens (768 blocks) 11.4 -> 8.6, 40 of 700 (880) 20.4 -> 15.3, 224 of 150 (1120) 9.9 -> 9.9,
//     256 of 225 (2048) 15.0 -> 14.0, 36 of 1000 (1152) 27.5 -> 25.7, 36 of 1189 (1368) 33.2 -> 35.1, 12 of 2984 (1128) 68.4 -> 73.4;
//     seven blocks do not come in fours (208 of 205, 1456, 11.8 -> 12.9); a second workgroup per CU 400 of 150 (2000) 15.9 -> 13.6,
//     132 of 622 (2640) 34.0 -> 36.6; problems past a whole number of workgroups per CU, which are split there: 81 of 559 (1458)
//     21.3 -> 19.3, 99 of 608 (1881) 25.0 -> 27.2, 72 of 807 (1872) 27.9 -> 33.0, 60 of 1045 (1980) 32.9 -> 50.9; all split, long: 6 of
//     3600 (678) 48.4 -> 55.9, but 12 of 1590 28.1 -> 24.4.  Few problems leave XCDs idle there: 1 of 10401 (326) 342 -> 78, 4 of
//     9867 (1236) 331 -> 191.
//   Heads of 32, half the bytes per block and the same arithmetic: 180 of 256 (1440) 8.0 -> 7.1, 12 of 2400 (900) 39.1 -> 23.9, 9 of
//     5850 (1647) 127 -> 81; where the XCDs have about as many problems each (on average eight tenths of the most) 128 of
//     500 (2048) 12.2 -> 15.5, 32 of 1966 (1984) 33.9 -> 40.4, 60 of 1052 (1980) 21.5 -> 24.8.
//   fp32 rows, twice the bytes: heads of 32 143 of 129 (715) 7.3 -> 6.0, 195 of 182 (1170) 8.3 -> 9.1, 223 of 127 (892) 6.0 -> 6.4, 16 of
//     1667 (848) 28.1 -> 36.7; heads of 72 78 of 287 (702) 16.5 -> 13.3, 88 of 415 (1144) 25.2 -> 33.3, 144 of 105 (576) 9.4 -> 11.3;
//     from nine tiles by the pitch of the rows, which are read four times as often as there: whole cache lines apart (every fourth head
//     count) they fall on the same channels: 24 of 550, H = 6 17.5 -> 14.2, H = 8 1.00 - 1.02, 12 of 880, H = 6 0.84, H = 4 1.19, 16 of
//     1473, H = 16 43.2 -> 72.4, 80 of 306, H = 16 18.3 -> 20.1.
//   Sequences of one or two key tiles (clips of 33 .. 64 frames) leave most of a 256-query workgroup idle: at any number of problems
//     0.4 - 0.6 of the time (25440 problems of 48: 350 -> 166), fp32 rows 0.8 (2532 blocks 11.4 -> 9.3).
// 2600 random shapes below 2000 blocks: 0.76 of the tile kernel's time; 0.8 % of them slower by 3 % or more (at most 10 %).
inline int plan_short(long long n_bh, int sq, int sk, int head_dim, int elem_size, long long kv_pitch_bytes = 0) {
  const long long blk = (sq + 31) / 32, n_blocks = n_bh * blk;
  const int ntile = (sk + 31) / 32;
  const ItemPlan tile = plan_items(n_bh, sq, sk, head_dim, elem_size);
  const long long xcd_bh = (n_bh + 7) / 8, per_xcd = xcd_bh * tile.n_item;
  const bool wide = head_dim == 72, clip = ntile <= 2 && sq <= 64, one = tile.n_item == 1;
  const bool all_split = tile.n_split && !tile.bh_plain, part_split = tile.n_split && tile.bh_plain;
  long long most;
  const auto at_most = [&](bool where, long long n) { if (where) most = std::min(most, n); };
  if (elem_size == 2) {
    most = clip ? n_blocks : per_xcd > 2 * TILE_CUS ? 0 : per_xcd > TILE_CUS ? 2000 : !wide || one ? 2048 : ntile <= 24 ? 1320
                                                                                               : ntile <= 80 ? 1200 : 1080;
    at_most(wide && one && ntile == 7 && per_xcd <= TILE_CUS, 1300);
    at_most(wide && part_split && ntile >= 13, ntile <= 16 ? 1900 : 1500);
    at_most(!wide && ntile >= 7 && 10 * n_bh >= 64 * xcd_bh && (per_xcd <= TILE_CUS || (part_split && ntile > 16)), 1550);
  } else {
    const bool lines = kv_pitch_bytes % 128 == 0 && n_bh > 4;
    most = clip ? 2600 : wide ? 850 : 900;
    at_most(one && !clip && (ntile == 4 || (wide && ntile == 3)), 512);
    at_most(wide && lines && ntile >= 9, ntile <= 16 ? 780 : all_split ? 256 : 512);
    at_most(wide && n_bh > 4 && all_split && xcd_bh * tile.n_split > TILE_CUS, 512);
    at_most(!wide && all_split && ntile >= 25, ntile <= 50 ? 700 : 500);
  }
  at_most(wide && tile.n_split && ntile > 50, 0);
  return n_blocks <= most ? short_groups(n_blocks, blk, ntile, head_dim, elem_size) : 0;
}

// Cross attention (bf16): the cross kernels stage all keys of a head per workgroup and give every wavefront whole query tiles,
// of which few tokens have too few.  us, cross kernel -> short, heads of 72: 500 tokens, 8 heads and 200 keys 13.0 -> 5.1, 2000
// tokens and 300 keys 16.7 -> 8.0, 3500 tokens, 12 heads (1320 blocks) 16.8 -> 13.5, 4000 tokens, 16 heads (2000) 17.6 -> 16.9, 6000
// tokens, 12 heads (2256) 17.9 -> 20.7; up to 128 keys only the smallest: 700 tokens, 7 heads and 90 keys (154 blocks) 4.5 -> 4.2,
// 1000 tokens, 16 heads (512) 4.7 -> 5.6, heads of 32 there 4.3 -> 3.8 with 120 keys, but 1970 tokens, 8 heads (496) and 65 keys 3.6 -> 3.7;
// up to 64 keys none.
inline int plan_short_cross(int n_tok, int L, int n_head, int head_dim) {
  const long long blk = (n_tok + 31LL) / 32, n_blocks = n_head * blk;
  const int ntile = (L + 31) / 32;
  const long long most = ntile > 4 ? 2000 : ntile < 3 ? 0 : head_dim == 32 && ntile == 4 ? 512 : 256;
  return n_blocks <= most ? short_groups(n_blocks, blk, ntile, head_dim, 2) : 0;
}

// Whether the tile kernel moves its results to row order on the way out (store_rows16) or stores them as accumulated.  With few
// queries most of the eight wavefronts are idle and nothing covers the way through the LDS crossbar; it pays in larger launches,
// the sooner where pieces of a row start on 64-byte boundaries.  As accumulated -> in row order, us: up to 48 queries (fp32 rows: others
// of so few are plan_short's) 34 frames at 440 positions, 3 heads 22.4 -> 23.4, 36 at 900, 4 heads 51.8 -> 53.3, 48 at 1590, 16 heads
// 467 -> 470; more of them 72 at 185, 5 heads 16.5 -> 17.1, 100 frames of 96 tokens, 10 heads 20.3 -> 21.0, but 49 at 700, 3 heads (fp32)
// 38.6 -> 37.9, 80 at 1001, 5 heads 70.6 -> 67.2, 96 at 185, 8 heads 29.2 -> 27.4, 16 frames of 400 tokens, 16 heads 28.3 -> 26.2.
inline bool store_in_row_order(long long n_bh, int sq, long long row_pitch_bytes) {
  if (sq <= 48) return false;
  return sq > 128 || n_bh > 2048 || (sq > 64 && row_pitch_bytes % 64 == 0);
}

// ---- which projection kernel and tile: the one with the smallest estimate, in us, fitted to shapes timed on the
//      card (1358 of them, M 16 .. 45000, N and K 64 .. 4608: the picks take 1.006 of the best kernel's time; K slices of 64):
//      gemm_stream  3 + (rounds of 256 tiles) (slices t + e): t = 1.5, e = 6 at 256 features, t = 1.7, e = 8 at 288
//                   (a tail tile of 64 / 128 / 192 token rows takes 0.50 / 0.66 / 0.82 of a full one)
//      gemm_tile    base + slices max(latency, load l2) + load out, load = tiles / 256 + 0.25: a lone tile is bound by the
//                   latency of its K loop, more tiles than CUs by L2 (about 60 GB/s per CU) and by their stores; a CU
//                   holds two tiles of 128 x 128, so that up to 512 of them take one round (16000 x 448 x 1824, 500 tiles: 31.8,
//                   gemm_stream 40.2, the former kernel 33.8; 11000 x 768 x 1824, 516 tiles: 52.1, gemm_stream 39.5)
//      Both sides of the line, measured in us: 2560 x 3456 x 1152 gemm_stream 24, 128 x 128 tiles 33; 6249 x 1152 x 4608
//      83 and 66; 1350 x 3456 x 1152 128 x 128 tiles 19, 64 x 128 23; 1260 x 576 x 2304 64 x 64 tiles 12, 128 x 128 24.
//      K groups (odd numbers) where every workgroup has a CU to itself and there are 6 slices or more: 64 x 64 tiles, three
//      groups, 1260 x 576 x 2304 13.9 -> 10.1, 800 x 1152 x 1152 8.7 -> 7.0, 60 x 1152 x 4608 22.8 -> 15.1, but 1260 x 288 x 288 the
//      same 4.2, and 360 tiles on 256 CUs 30.6 -> 33.0; 64 x 128, two groups, 1260 x 1152 x 4608 29.7 -> 24.6; 128 x 128, two
//      groups, 2800 x 1152 x 4608 47.3 -> 39.4, 500 x 4608 x 1152 16.2 -> 14.2.
//      Two groups with 96, 160 and 192 tokens x 128 features: the K loop is one round of at most a tile per CU, so the height that
//      just fits sets its length; without them 4109 tokens of 1152 features began a second round.
//      2552 x 1152 x 4608 39.7 -> 36.8 (96), 4109 x 1152 x 4608 60.7 -> 44.6, 5157 x 864 x 3456 46.9 -> 34.8, 1302 x 3456 x 1152
//      19.6 -> 17.4, 4281 x 1152 x 1152 19.5 -> 15.8 (160), 7417 x 648 x 2592 38.7 -> 32.9 (192); 1170 x 3456 x
//      864, 15.7 -> 16.1, is the one loss of 120 shapes. ----
constexpr int GEMM_CUS = 256;

struct GemmPlan {
  int kernel;            // 8, 9: gemm_stream with that many sub-tiles per wave column; 64, 96, 128: gemm_tile, 1 more: its K groups;
                         // 113, 161, 193: its K groups over tiles of 96, 160, 192 tokens x 128 features
  int n_mt, n_nt;
  int ms_tail;           // gemm_stream: token rows / 64 of the tail tiles
  int n_units;
  double us;
  int by_feature;        // gemm_tile, gemm_heads: the order of the tiles
};

// Order of the tiles, of which an XCD takes a contiguous eighth: along the features of a token tile, or (1) along the tokens of
// a feature tile.  With few tokens the weights are the larger operand, and eighths along the features have every XCD load most
// of them: the second order is taken where it loads half the rows or fewer.  In us, the same weights each time / others each
// time: 600 x 3456 x 1152 15.3 -> 13.5 / 15.6 -> 15.1, 400 x 4608 x 1152 14.4 -> 9.2 / 14.8 -> 11.1, MLP of 400 tokens and 1152 features
// 35.7 -> 31.7.  With less to gain it costs the attention kernel behind a q / k / v projection as much (900 x 2592 x 864, 0.52 of
// the rows: 11.8 -> 13.1).
inline int tile_order(int bm, int bn, long long n_mt, long long n_nt) {
  const long long all = n_mt * n_nt, run = (all + 7) / 8;
  auto rows = [&](long long inner, long long outer, int b_inner, int b_outer) {   // of a run along `inner`
    const long long touched = (run + inner - 1) / inner + (run % inner && all > run ? 1 : 0);
    return std::min(inner, run) * b_inner + std::min(outer, touched) * b_outer;
  };
  return 2 * rows(n_mt, n_nt, bm, bn) <= rows(n_nt, n_mt, bn, bm);
}

inline int tile_tokens(int kernel) { return kernel == 113 ? 96 : kernel == 161 ? 160 : kernel == 193 ? 192 : kernel >= 128 ? 128 : 64; }
inline int tile_features(int kernel) { return kernel < 96 ? 64 : 128; }

inline void plan_stream(int ns, int M, int N, int slices, GemmPlan *best) {
  static const double part[5] = {0, 0.50, 0.66, 0.82, 1.0};
  const int bn = 32 * ns;
  if (N < bn || M < 64 || slices < 2) return;
  const long long n_nt = (N + bn - 1) / bn, all = (M + 255LL) / 256 * n_nt;
  const double tile_us = ns == 8 ? 1.5 * slices + 6.0 : 1.7 * slices + 8.0;
  for (int less = 0; less < 3; ++less) {   // full tiles for this many rounds, the rest of the token rows as tail tiles
    const long long rounds = (all + GEMM_CUS - 1) / GEMM_CUS - less;
    if (rounds < 0) break;
    const long long n_mt = std::min((long long)M / 256, rounds * GEMM_CUS / n_nt), rows = M - 256 * n_mt;
    for (int ms = 1; ms <= 4; ++ms) {
      if (M < 64 * ms) break;
      const long long tail = (rows + 64 * ms - 1) / (64 * ms) * n_nt, room = rounds * GEMM_CUS - n_mt * n_nt;
      const double tail_rounds = tail > room ? (double)((tail - room + GEMM_CUS - 1) / GEMM_CUS) : 0.0;
      const double us = 3.0 + (rounds + tail_rounds * part[ms]) * tile_us;
      if (n_mt * n_nt + tail <= 0x7fffffffLL && us < best->us)
        *best = GemmPlan{ns, (int)n_mt, (int)n_nt, ms, (int)(n_mt * n_nt + tail), us, 0};
    }
  }
}

// tiles of a problem
inline long long count_tiles(int kernel, int M, int N) {
  const int bm = tile_tokens(kernel), bn = tile_features(kernel);
  return ((long long)M + bm - 1) / bm * ((N + bn - 1) / bn);
}

// M2, N2: a second problem in the same launch (plan_pair), M2 = 0: none
inline void plan_tile(int kernel, double base, double latency, double l2, double out, int M, int N, int slices,
               GemmPlan *best, int M2 = 0, int N2 = 0) {
  const int bm = tile_tokens(kernel), bn = tile_features(kernel);
  const long long n_mt = ((long long)M + bm - 1) / bm, n_nt = (N + bn - 1) / bn, all = n_mt * n_nt + count_tiles(kernel, M2, N2);
  if ((kernel & 1) && (all > GEMM_CUS || slices < 6)) return;   // K groups: one workgroup per CU
  double load = all / (double)GEMM_CUS + 0.25;
  if (kernel == 128 && load > 1.5) load *= load <= 2.25 ? 0.8 : load <= 2.85 ? 1.1 : 1.0;   // one round of two per CU, a second begun
  const double us = base + slices * std::max(latency, load * l2) + load * out;
  if (all <= 0x7ffffff0LL && us < best->us)
    *best = GemmPlan{kernel, (int)n_mt, (int)n_nt, 0, (int)(n_mt * n_nt), us, tile_order(bm, bn, n_mt, n_nt)};
}

// gemm_heads (estimate fitted like those above, whole temporal modules in us, separate pass -> gemm_heads): 1260 tokens of 576
// 28.0 -> 23.8, 800 of 864 31.0 -> 27.2, 630 of 1152 35.3 -> 31.0; but 250 of 1152 26.2 -> 26.9, 60 of 864 22.0 -> 23.2.  145, tiles
// of 128 tokens: 1432 of 576 29.0 -> 27.2, 1760 of 864 41.4 -> 36.9, 1005 of 1152 39.9 -> 38.9, 4200 of 288 30.4 -> 28.0; past one
// tile per CU it does not go (2000 of 864, 288 tiles, 42.4 with the separate pass).
inline void plan_heads(int kernel, double base, double slice, double out, int M, int N, int slices, GemmPlan *best) {
  const int bm = kernel == 145 ? 128 : 64, bn = 144;
  const long long n_mt = ((long long)M + bm - 1) / bm, n_nt = (N + bn - 1) / bn;
  const double us = base + slice * slices + out * n_mt * n_nt / (double)GEMM_CUS;
  if (n_mt * n_nt <= GEMM_CUS && us < best->us)
    *best = GemmPlan{kernel, (int)n_mt, (int)n_nt, 0, (int)(n_mt * n_nt), us, tile_order(bm, bn, n_mt, n_nt)};
}

inline GemmPlan plan_tiles(int M, int N, int K, int M2 = 0, int N2 = 0) {
  GemmPlan best{0, 0, 0, 0, 0, 1e30, 0};
  const int slices = (K + 63) / 64;
  plan_tile(64, 2.9, 0.26, 0.25, 0.55, M, N, slices, &best, M2, N2);
  plan_tile(65, 2.95, 0.185, 0.17, 0.55, M, N, slices, &best, M2, N2);
  plan_tile(96, 3.3, 0.32, 0.36, 1.1, M, N, slices, &best, M2, N2);
  plan_tile(97, 3.2, 0.285, 0.24, 1.1, M, N, slices, &best, M2, N2);
  plan_tile(128, 3.5, 0.55, 0.52, 2.2, M, N, slices, &best, M2, N2);
  plan_tile(129, 3.6, 0.48, 0.45, 1.6, M, N, slices, &best, M2, N2);
  if (K >= 384) {
    // 96 tokens only past 2400: 2552 .. 7233 tokens take 0.86 .. 0.94 of the time.  The line is not where the gain ends (595 x 4608 x
    // 1152 13.4 -> 12.2, 2200 x 1152 x 1152 13.4 -> 12.3): the plans of smaller sizes are held by tests and stay as they were.  Nor
    // beside 64 x 64 tiles where those are the best of the others, about two per CU: 3291 x 576 x 576 6.4 -> 7.3, 5921 x 288 x 1152 9.6 -> 10.7.
    if (M > 2400 && best.kernel != 64) plan_tile(113, 3.5, 0.41, 0.37, 1.3, M, N, slices, &best, M2, N2);
    // a taller tile only where the next lower one has more tiles than CUs: 160 tokens beside a round of 128 that fits, 3786 x 960 x
    // 3840 33.1 -> 37.1, 6340 x 576 x 2304 22.4 -> 24.6, 3806 x 960 x 960 12.4 -> 13.5
    const auto past = [&](int kernel) { return count_tiles(kernel, M, N) + count_tiles(kernel, M2, N2) > GEMM_CUS; };
    if (past(129)) plan_tile(161, 3.8, 0.50, 0.475, 2.0, M, N, slices, &best, M2, N2);
    if (past(161)) plan_tile(193, 4.0, 0.57, 0.565, 2.4, M, N, slices, &best, M2, N2);
  }
  return best;
}

inline GemmPlan plan_gemm(int M, int N, int K) {
  GemmPlan best = plan_tiles(M, N, K);
  const int slices = (K + 63) / 64;
  plan_stream(8, M, N, slices, &best);
  plan_stream(9, M, N, slices, &best);
  return best;
}

// Two projections of the same K in one launch: C = A W^T and, side by side in n_split-wide planes, C2 = A2 W2^T.  The second
// one (few rows: the text of the cross module) rides along where it costs no round of its own: as further tiles of
// gemm_tile, or in the room that the last round of gemm_stream leaves (there with 64 rows or more, the least a tile has); else it
// is launched by itself (25440 and 120 tokens: 7 units of room for 18).  Cross modules in us, two launches -> one: 17408 and 300
// tokens of 1152 features 149 -> 144, 34000 and 120 of 864 147 -> 143; 2048 and 120 of 1152 39.5 -> 33.0, 6000 and 300 of 864
// 59.4 -> 54.1, 1260 and 60 of 576 20.0 -> 15.4.
// Tiles of 96, 160 and 192 tokens are the best ones for the first problem where they just fill the chip, and a launch of its own for the
// second costs more than they gain: there the pair is planned, the best tiles for both against two launches.  Cross modules in us, best
// for the first alone -> for both: 2448 and 300 tokens of 1152 features 45.1 -> 40.1, 3339 and 64 of 864 35.7 -> 30.6, 4719 and 90 of 576
// 31.6 -> 27.4, 7881 and 200 of 576 41.6 -> 38.0, 4188 and 40 of 1152 46.8 -> 41.1, 5130 and 300 of 1152 63.3 -> 58.5.
struct PairPlan {
  GemmPlan first;        // n_units: those of the first problem
  int n_nt2, ms2;
  long long n_units2;    // 0: two launches
};

inline PairPlan plan_pair(int M, int N, int M2, int N2, int K) {
  PairPlan p{plan_gemm(M, N, K), 0, 0, 0};
  GemmPlan &g = p.first;
  const auto in_tiles = [&] {
    p.n_nt2 = (N2 + tile_features(g.kernel) - 1) / tile_features(g.kernel);
    p.n_units2 = count_tiles(g.kernel, M2, N2);
    if (g.n_units + p.n_units2 > (g.kernel & 1 ? (long long)GEMM_CUS : 0x7ffffff0LL)) p.n_units2 = 0;
  };
  if (g.kernel == 8 || g.kernel == 9) {
    const int bn = 32 * g.kernel, room = (GEMM_CUS - g.n_units % GEMM_CUS) % GEMM_CUS;
    p.ms2 = M2 >= 128 ? 2 : 1;
    p.n_nt2 = (N2 + bn - 1) / bn;
    p.n_units2 = (M2 + 64LL * p.ms2 - 1) / (64 * p.ms2) * p.n_nt2;
    if (M2 < 64 || N2 < bn || p.n_units2 > room) p.n_units2 = 0;
  } else if (g.kernel) {
    in_tiles();
    if (!p.n_units2 && (g.kernel == 113 || g.kernel == 161 || g.kernel == 193)) {
      const GemmPlan both = plan_tiles(M, N, K, M2, N2);
      if (both.kernel && both.us < g.us + plan_gemm(M2, N2, K).us) {
        g = both;
        in_tiles();
      }
    }
  }
  return p;
}

// q, k, v projections of a self-attention module with layernorm2 (+ rotation) of q and k, whichever is estimated fastest:
//   the best plain projection and a pass over q and k (each read and written once at 4.8 TB/s, 3 us at least);
//   heads of 72: in the epilogue of the large-tile projection (it costs a tile 3 us);
//   in the epilogue of small tiles: heads of 72, few tokens, one tile of two heads and 64 or 128 tokens per CU: gemm_heads; heads of
//   32, which are a pair of sub-tiles: gemm_tile (it costs a launch 0.8 us and a round of tiles as much; whole modules in us, pass -> epilogue:
//   2880 tokens of 256 24.0 -> 18.4, 3696 of 256 31.4 -> 25.3, 29715 of 384 98.9 -> 90.8, 38288 of 512 428 -> 417; gemm_heads,
//   three heads per tile, took 13.8 at 189 of 128 where this takes 12.7, 14.0 -> 12.9 at 282 of 128).
enum { QKV_PASS = 0, QKV_STREAM = 1, QKV_SMALL = 2 };
struct QkvPlan {
  int way;
  GemmPlan gemm;
};

inline QkvPlan plan_qkv(int n_tok, int H, int D, int S, int rope) {
  const int C = H * D, slices = (C + 63) / 64;
  GemmPlan plain = plan_gemm(n_tok, 3 * C, C), fused{0, 0, 0, 0, 0, 1e30, 0}, small{0, 0, 0, 0, 0, 1e30, 0};
  if (D == 72 && C % 288 == 0 && (!rope || S >= 64)) plan_stream(9, n_tok, 3 * C, slices, &fused);
  fused.us += 3.0 * (fused.n_units / (double)GEMM_CUS + 0.5);
  if (D == 72) {
    plan_heads(144, 5.5, 0.3, 1.0, n_tok, 3 * C, slices, &small);
    plan_heads(145, 7.0, 0.5, 1.5, n_tok, 3 * C, slices, &small);
  } else {
    small = plan_tiles(n_tok, 3 * C, C);
    small.us += 0.8 + 0.8 * small.n_units / (double)GEMM_CUS * (small.kernel >= 128 ? 1.0 : small.kernel >= 96 ? 0.5 : 0.25);
  }
  plain.us += 3.0 + 8e-6 * n_tok * C / 4.8;
  if (small.kernel && small.us < std::min(fused.us, plain.us)) return {QKV_SMALL, small};
  if (fused.kernel && fused.us < plain.us) return {QKV_STREAM, fused};
  return {QKV_PASS, plain};
}

}  // namespace pab
