"""Which kernel, tile and item a shape takes: the library's planning header, compiled by itself for the host.  The GPU
tests of the kernels choose their shapes for the path that they run; here that choice is held, so that a change of a
planner's constant cannot silently empty one of them."""
import os
import re
import subprocess

import pytest

import test_gpu_gemm as G
import test_gpu_parity as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
QUERY = r'''
#include <cstdio>
#include <cstring>
#include "launch_plan.hpp"
int main() {
  char what[16];
  while (scanf("%15s", what) == 1) {
    if (!strcmp(what, "gemm")) {
      int M, N, K;
      if (scanf("%d %d %d", &M, &N, &K) != 3) return 1;
      const pab::GemmPlan g = pab::plan_gemm(M, N, K);
      printf("%d %d %d %d %d %d\n", g.kernel, g.n_mt, g.n_nt, g.ms_tail, g.n_units, g.by_feature);
    } else if (!strcmp(what, "pair")) {
      int M, N, M2, N2, K;
      if (scanf("%d %d %d %d %d", &M, &N, &M2, &N2, &K) != 5) return 1;
      const pab::PairPlan p = pab::plan_pair(M, N, M2, N2, K);
      printf("%d %d %d %lld\n", p.first.kernel, p.first.n_units, p.ms2, p.n_units2);
    } else if (!strcmp(what, "qkv")) {
      int n, H, D, S, rope;
      if (scanf("%d %d %d %d %d", &n, &H, &D, &S, &rope) != 5) return 1;
      const pab::QkvPlan p = pab::plan_qkv(n, H, D, S, rope);
      printf("%d %d %d %d %d %d\n", p.way, p.gemm.n_mt, p.gemm.ms_tail, p.gemm.n_units, p.gemm.by_feature, p.gemm.kernel);
    } else if (!strcmp(what, "rows")) {
      long long n_bh, pitch; int sq;
      if (scanf("%lld %d %lld", &n_bh, &sq, &pitch) != 3) return 1;
      printf("%d\n", pab::store_in_row_order(n_bh, sq, pitch));
    } else if (!strcmp(what, "short")) {
      long long n_bh; int sq, sk, D, size;
      if (scanf("%lld %d %d %d %d", &n_bh, &sq, &sk, &D, &size) != 5) return 1;
      printf("%d\n", pab::plan_short(n_bh, sq, sk, D, size));
    } else if (!strcmp(what, "pitched")) {
      long long n_bh, pitch; int sq, sk, D, size;
      if (scanf("%lld %d %d %d %d %lld", &n_bh, &sq, &sk, &D, &size, &pitch) != 6) return 1;
      printf("%d\n", pab::plan_short(n_bh, sq, sk, D, size, pitch));
    } else if (!strcmp(what, "cross")) {
      int n, L, H, D;
      if (scanf("%d %d %d %d", &n, &L, &H, &D) != 4) return 1;
      printf("%d\n", pab::plan_short_cross(n, L, H, D));
    } else {
      long long n_bh; int sq, sk, D, size;
      if (scanf("%lld %d %d %d %d", &n_bh, &sq, &sk, &D, &size) != 5) return 1;
      const pab::ItemPlan p = pab::plan_items(n_bh, sq, sk, D, size);
      printf("%d %lld %lld\n", p.n_item, p.bh_plain, p.n_split);
    }
    fflush(stdout);
  }
}
'''


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "query.cpp").write_text(QUERY)
    exe = str(d / "query")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2408_12588_amd", "csrc"), "-o", exe,
                    str(d / "query.cpp")], check=True, timeout=120)

    def ask(what, rows):
        text = "".join("%s %s\n" % (what, " ".join(str(int(x)) for x in r)) for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        got = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
        assert len(got) == len(rows)
        return got

    return ask


def items_of(shape):
    """(problems, queries, keys, head dim, bytes per element) of a call that the short or the tile kernel takes."""
    kind, T, S, L, H, D, dtype = shape
    return {0: (T * H, S, S), 1: (S * H, T, T), 2: (H, T * S, L)}[kind] + (D, 2 if dtype == "bf16" else 4)


def test_projection_shapes_take_the_kernels_they_are_chosen_for(plan):
    got = plan("gemm", G.SHAPES)
    assert [g[0] for g in got] == [8, 8, 8, 8, 9, 9, 128, 128, 96, 64, 64, 96]
    tails = [g[3] for g in got[:6]]
    assert (tails[0], tails[1], tails[4], tails[5]) == (3, 1, 2, 1)
    assert [g[1] > 0 for g in got[:6]] == [False, True, True, False, False, True]    # full tiles beside the tail tiles
    assert all(g[4] > 256 for g in got[:1] + got[2:3] + got[5:6])                    # more than one tile per CU
    groups = plan("gemm", G.K_GROUPS)
    assert [g[0] for g in groups] == [65, 65, 65, 65, 97, 97, 129, 65, 97, 129]
    assert got[-1][5] == 1 and [g[5] for g in groups[-3:]] == [1, 1, 1]     # order of the tiles
    assert plan("gemm", [(200, 2016, 2016)])[0][5] == 1                     # ... of a query + text projection
    assert [g[0] for g in plan("gemm", G.HALF_SLICES)] == [8, 9, 8, 65, 64]


def test_tile_heights_are_those_meant(plan):
    assert [g[0] for g in plan("gemm", [s[1:] for s in G.TILE_HEIGHTS])] == [s[0] for s in G.TILE_HEIGHTS]


def test_every_planned_projection_kernel_is_launched(plan):
    """Each number that the planners give has a case in launch_gemm_kernel (those of large tiles only without the norm), and any
    other one is an error, not a call without a launch."""
    source = open(os.path.join(ROOT, "paper_2408_12588_amd", "csrc", "pab_api.hip")).read()
    body = source[source.index("launch_gemm_kernel(const GemmPlan"):]
    body = body[:body.index("\n}\n")]
    cases = {int(n) for n in re.findall(r"case (\d+): hipLaunch", body)}
    assert re.search(r"default: return fail\(", body)
    sizes = sorted({int(round(16 * 1.17 ** i)) for i in range(51)})
    gemm = {g[0] for g in plan("gemm", [(m, n, k) for m in sizes for n in (64, 288, 576, 1152, 3456, 4608) for k in (32, 288, 576, 1152, 4608)])}
    assert gemm <= cases | {8, 9} and {8, 9, 64, 97, 129, 161, 193} <= gemm, gemm
    qkv = plan("qkv", [(m, h, 32, 64, 1) for m in sizes for h in (1, 3, 4, 9, 16, 25, 36)])
    assert {q[5] for q in qkv if q[0] == 2} <= cases


def test_tiles_of_96_tokens_leave_what_two_small_tiles_per_cu_do_faster(plan):
    small, tall = [(3291, 576, 576), (3459, 576, 576), (5921, 288, 1152), (6080, 288, 1152)], [(3680, 576, 576), (6120, 288, 1152)]
    assert [g[0] for g in plan("gemm", small + tall)] == [64] * 4 + [113] * 2
    assert plan("pair", [(3419, 576, 16, 1152, 576)])[0][0] == 64


def test_module_shapes_take_the_ways_they_are_chosen_for(plan):
    qkv = lambda shapes: plan("qkv", [(T * S, H, D, S, kind == 1) for kind, T, S, H, D in shapes])
    assert [q[0] for q in qkv([m + (72,) for m in G.MODULES])] == [1, 1, 1, 1, 0]
    few = qkv(G.FEW_TOKENS)
    assert [q[0] for q in few] == [2] * 6 and {q[4] for q in few} == {0, 1}      # both orders of the tiles
    # moved tokens: in the epilogue of the large tiles, with tail tiles of which most reach back over rows of another
    moved = qkv([m + (72,) for m in G.MOVED])
    assert all(way == 1 and ms < 4 for way, n_mt, ms, *_ in moved)
    assert sum((T * S - 256 * n_mt) % (64 * ms) > 0 for (kind, T, S, H), (way, n_mt, ms, *_) in zip(G.MOVED, moved)) >= 4


def test_heads_of_32_are_normalised_in_the_tiles_meant_for_them(plan):
    got = plan("qkv", [(T * S, H, 32, S, kind == 1) for _, kind, T, S, H in G.HEADS_OF_32])
    assert [(g[0], g[5]) for g in got] == [(2, shape[0]) for shape in G.HEADS_OF_32]
    got = plan("qkv", [(T * S, H, 72, S, kind == 1) for kind, T, S, H in G.HEADS_128])
    assert [(g[0], g[5]) for g in got] == [(2, 145)] * len(got)
    assert {g[5] for g in plan("qkv", [(T * S, H, D, S, kind == 1) for kind, T, S, H, D in G.FEW_TOKENS if D == 72])} == {144}


def test_text_projection_rides_where_it_is_meant_to(plan):
    got = plan("pair", [(T * S, 72 * H, L, 144 * H, 72 * H) for T, S, L, H in G.CROSS_PAIRS])
    for shape, want, (kernel, units, ms2, units2) in zip(G.CROSS_PAIRS, G.CROSS_PAIR_PATHS, got, strict=True):
        assert (kernel, ms2 if units2 and kernel < 16 else 0, units2 > 0) == want, shape
        if units2 and kernel in (8, 9):       # no round of its own
            assert units % 256 + units2 <= 256


def test_text_projection_rides_beside_the_tile_heights_too(plan):
    """Tiles that just fill the chip with the queries do not push the text into a launch of its own: bands of sizes, and both sides of them."""
    got = plan("pair", [(T * S, 72 * H, L, 144 * H, 72 * H) for _, T, S, L, H in G.HEIGHT_PAIRS])
    assert [(g[0], g[3] > 0) for g in got] == [(s[0], True) for s in G.HEIGHT_PAIRS]
    alone = {g[0] for g in plan("gemm", [(T * S, 72 * H, 72 * H) for _, T, S, L, H in G.HEIGHT_PAIRS])}
    assert alone == {113, 161, 193}
    bands = [(m, 1152, 120) for m in range(2446, 2630, 20)] + [(m, 864, 120) for m in range(3300, 3423, 20)] + [
        (m, 576, 120) for m in range(4764, 4887, 20)] + [(m, 384, 120) for m in range(7997, 8120, 20)] + [(m, 1152, 120) for m in range(4215, 4460, 20)] + [
        (m, 864, L) for m in range(2690, 3423, 50) for L in (200, 300)]
    for shape, (kernel, units, _, units2) in zip(bands, plan("pair", [(m, C, L, 2 * C, C) for m, C, L in bands])):
        assert units2 > 0 and (kernel % 2 == 0 or units + units2 <= 256), shape


def test_split_shapes_are_split(plan):
    part = {(0, 7, 700, 0, 12, 72, "bf16"): 4, (0, 9, 513, 0, 11, 32, "f32"): 19, (0, 5, 1124, 0, 12, 32, "bf16"): 12, (0, 4, 2866, 0, 6, 32, "bf16"): 8}
    calls = [items_of(shape) for shape in P.SPLIT_SHAPES]
    assert [r[0] for r in plan("short", calls)] == [0] * len(calls)      # the dispatch asks this first
    for shape, (n_bh, sq, *_), (n_item, bh_plain, n_split) in zip(P.SPLIT_SHAPES, calls, plan("items", calls)):
        assert n_bh - bh_plain == part.get(shape, n_bh) and n_split == -(-sq // 64), shape
    assert all(r[0] for r in plan("short", [items_of(shape) for shape in P.SHORT_SPLITS]))


# problems, queries, keys, head dim, bytes per element: calls that split items make slower, and such that they make faster
# (the figures are at the rule)
PLAIN = [(117, 755, 755, 72, 2), (84, 912, 912, 72, 2), (110, 677, 677, 72, 2), (13, 6045, 600, 72, 2), (32, 1590, 1590, 72, 4),
         (10, 6103, 448, 72, 4), (9, 7273, 7273, 72, 4), (10, 11634, 11634, 72, 4), (42, 1600, 1600, 72, 4), (224, 562, 562, 72, 2), (340, 229, 229, 32, 2),
         (9, 6384, 274, 32, 4), (33, 2481, 2481, 32, 4), (256, 1024, 1024, 72, 2), (256, 1590, 1590, 72, 2), (256, 3600, 3600, 72, 2)]
SPLIT = [(16, 1024, 1024, 72, 4), (6, 3600, 3600, 72, 2), (72, 1024, 1024, 72, 2), (66, 788, 788, 72, 2), (136, 1000, 1000, 72, 2),
         (84, 700, 700, 72, 2), (40, 3600, 3600, 72, 2), (204, 1024, 1024, 72, 2), (91, 3066, 3066, 72, 4), (272, 1024, 1024, 72, 2),
         (24, 2871, 2871, 72, 2), (10, 4640, 4640, 72, 2), (24, 2866, 2866, 32, 2), (60, 1124, 1124, 32, 2), (42, 1711, 1711, 72, 2)]
# ... and such that the short kernel takes before the rule is asked
PLAIN_SHORT = [(208, 284, 284, 72, 2), (48, 512, 512, 72, 2), (16, 128, 128, 72, 2), (1, 10401, 10401, 72, 4), (210, 271, 271, 32, 2)]
SPLIT_SHORT = [(16, 1024, 1024, 72, 2), (16, 300, 300, 72, 2), (40, 252, 252, 72, 2), (32, 1024, 1024, 72, 2)]


def test_split_items_where_they_pay(plan):
    assert [p[2] for p in plan("items", PLAIN + PLAIN_SHORT)] == [0] * len(PLAIN + PLAIN_SHORT)
    assert all(p[2] > 0 for p in plan("items", SPLIT + SPLIT_SHORT))
    assert [p[0] for p in plan("short", PLAIN + SPLIT)] == [0] * len(PLAIN + SPLIT)
    assert all(p[0] for p in plan("short", PLAIN_SHORT + SPLIT_SHORT))
    # never more than three split items per CU on any of the eight XCDs, which take every eighth problem each
    shapes = [(n, s, k, D, size) for n in list(range(1, 40)) + [64, 91, 105, 256, 999] for s in (1, 64, 225, 300, 1000, 4000, 20000)
              for k in (1, 200, 500, 1024, 9000) for D in (32, 72) for size in (2, 4)]
    for (n, s, *rest), (n_item, bh_plain, n_split) in zip(shapes, plan("items", shapes)):
        assert 0 <= bh_plain <= n and n_item == -(-s // 256)
        assert -(-(n - bh_plain) // 8) * n_split <= 96, (n, s, rest)


def test_short_launches(plan):
    """Each way of the short kernel at the shapes that are meant for it, and the tile kernel's own ways beside it."""
    got = [r[0] for r in plan("short", [items_of(shape) for shape in P.SHORT_SHAPES])]
    assert got == [22] * 7 + [44] * 8 + [42] * 6 + [41]
    calls = [items_of(shape) for shape in P.TILE_SHAPES]
    assert [r[0] for r in plan("short", calls)] == [0] * len(calls)
    assert [bh_plain > 0 for _, bh_plain, _ in plan("items", calls)] == [True, False] + [True] * (len(calls) - 2)
    # both sides of the line: problems, queries, keys, head dim, bytes per element
    short = [(96, 256, 256, 72, 2), (40, 700, 700, 72, 2), (192, 290, 290, 72, 2), (256, 225, 225, 72, 2), (72, 462, 462, 72, 2),
             (400, 150, 150, 72, 2), (12, 1590, 1590, 72, 2), (180, 256, 256, 32, 2), (12, 2400, 2400, 32, 2), (143, 129, 129, 32, 4),
             (60, 217, 217, 72, 4), (25440, 48, 48, 72, 2), (1266, 56, 56, 32, 4)]
    tile = [(132, 622, 622, 72, 2), (6, 3600, 3600, 72, 2), (195, 182, 182, 32, 4), (88, 415, 415, 72, 4), (128, 500, 500, 72, 2),
            (256, 400, 400, 72, 2), (256, 1024, 1024, 72, 2), (256, 1590, 1590, 72, 2)]
    assert all(r[0] for r in plan("short", short)) and not any(r[0] for r in plan("short", tile))


def test_long_sequences_stay_with_the_tile_kernel_where_it_is_faster(plan):
    """Problems, queries, keys, head dim, bytes per element that the short kernel makes slower (figures at the rule), and neighbours that it
    makes faster."""
    tile = [(60, 1045, 1045, 72, 2), (50, 1164, 1164, 72, 2), (72, 807, 807, 72, 2), (99, 608, 608, 72, 2), (208, 205, 205, 72, 2), (12, 2984, 2984, 72, 2),
            (128, 500, 500, 32, 2), (32, 1966, 1966, 32, 2), (60, 1052, 1052, 32, 2), (16, 1473, 1473, 72, 4), (20, 1180, 1180, 72, 4),
            (8, 1401, 1401, 72, 4), (8, 1111, 1111, 72, 4), (80, 306, 306, 72, 4), (144, 105, 105, 72, 4), (32, 516, 516, 72, 4), (16, 1667, 1667, 32, 4),
            (223, 127, 127, 32, 4)]
    short = [(1, 10401, 10401, 72, 2), (4, 9867, 9867, 72, 2), (81, 559, 559, 72, 2), (140, 398, 398, 72, 2), (176, 205, 205, 72, 2), (238, 240, 240, 72, 2),
             (20, 1523, 1523, 72, 2), (12, 5109, 521, 72, 2), (84, 551, 551, 32, 2), (18, 2711, 2711, 32, 2), (9, 5850, 5850, 32, 2), (6, 910, 910, 72, 4),
             (78, 287, 287, 72, 4), (126, 107, 107, 72, 4), (128, 133, 133, 72, 4), (3, 8976, 91, 72, 4), (22, 968, 968, 32, 4)]
    assert [r[0] for r in plan("short", tile)] == [0] * len(tile)
    assert all(r[0] for r in plan("short", short))
    # long sequences of fp32 rows of 72: also by the heads, four of which are a whole number of cache lines
    by_heads = lambda H: [r[0] > 0 for r in plan("pitched", [(24, 551, 551, 72, 4, 288 * H), (20, 560, 560, 72, 4, 288 * H), (32, 657, 657, 72, 4, 288 * H),
                                                             (16, 680, 680, 72, 4, 288 * H)])]
    assert by_heads(6) == by_heads(1) == [True] * 4 and by_heads(8) == by_heads(16) == [False] * 4
    assert [r[0] for r in plan("short", [items_of(s) for s in P.SHORT_F32_GROUPS])] == [22] * len(P.SHORT_F32_GROUPS)
    assert [r[0] for r in plan("cross", [(1970, 65, 8, 32), (504, 65, 8, 32)])] == [0, 44]


def test_cross_attention_of_few_tokens(plan):
    ask = lambda shapes: [r[0] for r in plan("cross", [(T * S, L, H, D) for T, S, L, H, D in shapes])]
    assert ask([s[1:] for s in P.SHORT_CROSS]) == [s[0] for s in P.SHORT_CROSS]
    assert ask(P.LONG_CROSS) == [0] * len(P.LONG_CROSS)
    full = [(16, 1590, 120, 16, 72), (17, 1024, 300, 16, 72), (1, 1000, 120, 16, 72), (1, 100, 64, 2, 72), (1, 700, 120, 30, 32), (12, 500, 300, 12, 72)]
    assert ask(full) == [0] * len(full)


def test_extreme_inputs_of_the_short_kernel_take_every_way_of_it(plan):
    assert [r[0] for r in plan("short", [items_of(s[1:]) for s in P.SHORT_EXTREMES])] == [s[0] for s in P.SHORT_EXTREMES]
    extremes = P.SHORT_CROSS_EXTREMES + P.SHORT_CROSS_RAGGED
    assert [r[0] for r in plan("cross", [(T * S, L, H, D) for _, _, T, S, L, H, D, _ in extremes])] == [s[0] for s in extremes]


def test_order_of_stores(plan):
    accumulated = [(1600, 34, 230400), (925, 50, 133200), (925, 72, 133200), (1000, 96, 1440), (10 ** 6, 48, 2304)]
    in_rows = [(5005, 80, 720720), (1480, 96, 213120), (256, 400, 2304), (2100, 49, 302400), (4, 129, 720)]
    assert [r[0] for r in plan("rows", accumulated + in_rows)] == [0] * 5 + [1] * 5
    # the GPU test has both orders for either type and head dim, on the tile kernel
    calls = [items_of(s[:7]) for s in P.FEW_QUERIES]
    assert [r[0] for r in plan("short", calls)] == [0] * len(calls)
    pitches = [s[4] * (s[2] if s[0] == 1 else 1) * D * size for s, (*_, D, size) in zip(P.FEW_QUERIES, calls)]
    assert [r[0] for r in plan("rows", [(n, sq, pitch) for (n, sq, *_), pitch in zip(calls, pitches)])] == [s[7] for s in P.FEW_QUERIES]
    assert {s[5:] for s in P.FEW_QUERIES} == {(D, t, o) for D in (72, 32) for t in ("bf16", "f32") for o in (False, True)}
    assert all(r[0] for r in plan("short", [items_of(s) for s in P.SHORT_FEW_QUERIES]))


def test_one_round_of_large_small_tiles(plan):
    """Two 128 x 128 tiles share a CU: preferred up to 512 of them, not for the few more that begin a second round."""
    shapes = [(16000, 448, 1824), (13838, 512, 1824), (16000, 448, 4608), (4000, 1728, 1152), (11000, 768, 1824)]
    assert [(g[0], g[4] <= 512) for g in plan("gemm", shapes)] == [(128, True)] * 4 + [(8, True)]


def rows_loaded(n_mt, n_nt, bm, bn, by_feature):
    """Token and weight rows that the eight XCDs load for their contiguous runs of tiles."""
    total = n_mt * n_nt
    run = -(-total // 8)
    rows = 0
    for xcd in range(8):
        ids = range(run * xcd, min(run * (xcd + 1), total))
        tiles = [(i % n_mt, i // n_mt) if by_feature else (i // n_nt, i % n_nt) for i in ids]
        rows += bm * len({m for m, n in tiles}) + bn * len({n for m, n in tiles})
    return rows


def test_order_of_small_tiles_loads_fewer_rows(plan):
    """By feature (few tokens, many features) only where that halves the rows, or nearly so in the runs as they fall."""
    by_feature = [(600, 3456, 1152), (640, 3456, 864), (512, 4608, 1152), (480, 4608, 864), (400, 4608, 1152), (400, 3456, 864), (548, 3968, 2624)]
    by_token = [(2400, 864, 1152), (1647, 1532, 224), (1260, 2304, 576), (900, 2592, 864), (1260, 576, 576), (60, 4608, 1152), (4097, 1156, 160)]
    for shape, (kernel, n_mt, n_nt, _, units, order) in zip(by_feature + by_token, plan("gemm", by_feature + by_token)):
        assert kernel in (64, 65, 96, 97, 128, 129) and order == (shape in by_feature), shape
        bm, bn = 128 if kernel >= 128 else 64, 128 if kernel >= 96 else 64
        tokens, features = (rows_loaded(n_mt, n_nt, bm, bn, f) for f in (0, 1))
        assert features <= 0.55 * tokens if order else features >= 0.45 * tokens, (shape, tokens, features)
