"""GPU parity of the projection kernels at the edges of their tiles (the plain shapes are in test_gpu_module.py)."""
import math

import numpy as np
import pytest
import torch

from oracle import pab_module_oracle as mo

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [
    # M, N, K: what the shape is chosen for (kernel as picked by the size rule)
    (9001, 2304, 160),    # large tiles, 256 features: token tiles of 192 rows, more than one per CU, the last moved back; half slice
    (8200, 1728, 288),    # ... full tiles and 64-row tail tiles, last feature tile moved back, K = 4.5 slices
    (17000, 1444, 160),   # ... N = 4 mod 8: overlapping feature tiles start off 16-byte boundaries
    (9000, 1152, 128),    # ... two K slices, the fewest it takes
    (30000, 288, 224),    # large tiles, 288 features: one feature tile, 128-row tail tiles, half slice
    (12001, 2596, 160),   # ... full and 64-row tail tiles, N = 9.01 tiles
    (4097, 1156, 160),    # 128 x 128 tiles: one token row and four features in the last tiles
    (5000, 1152, 96),     # ... K = 1.5 slices
    (1647, 1532, 224),    # 64 x 128 tiles, ragged; K = 3.5 slices
    (700, 68, 96),        # 64 x 64 tiles: four features in the last, K = 1.5 slices
    (65, 64, 32),         # ... half a slice in all
    (601, 3460, 352),     # 64 x 128 tiles, consecutive tiles along the tokens; 25 token rows and four features in the last tiles
]


def rand(shape, seed, scale=1.0):
    g = np.random.Generator(np.random.Philox(key=seed))
    return torch.from_numpy(g.standard_normal(shape, dtype=np.float32) * np.float32(scale)).to(torch.bfloat16)


K_GROUPS = [
    # M, N, K: small tiles whose K slices are dealt to groups of wavefronts (kernel as picked by the size rule)
    (65, 68, 384),        # 64 x 64, three groups: two slices each, the fewest; one token row and four features in the last tiles
    (100, 64, 416),       # ... 6.5 slices: one group has a third, half a slice
    (1260, 576, 480),     # ... the half slice with the second group
    (33, 1152, 2304),     # ... 36 slices
    (1300, 1156, 480),    # 64 x 128, two groups: 7.5 slices
    (1300, 1152, 448),    # ... an odd number of them
    (2500, 1156, 1120),   # 128 x 128, two groups: 17.5 slices, ragged tiles
    (250, 3460, 480),     # 64 x 64, three groups, consecutive tiles along the tokens; ragged tiles
    (401, 4484, 480),     # 64 x 128, two groups, ...
    (481, 4612, 864),     # 128 x 128, two groups, ...
]


@pytest.mark.parametrize("M,N,K", SHAPES + K_GROUPS)
def test_projection_tiles(M, N, K):
    from paper_2408_12588_amd import pab
    print("projection", M, N, K, flush=True)
    a, w, b = rand((M, K), 1 + M), rand((N, K), 2 + N, 1.0 / math.sqrt(K)), rand((N,), 3 + K, 0.5)
    pad = 8                                   # columns behind the result that must stay as they are
    buf = torch.full((M, N + pad), 7.0, device=DEV, dtype=torch.bfloat16)
    pab.pab_linear(a.to(DEV), w.to(DEV), b.to(DEV), out=buf[:, :N])
    torch.cuda.synchronize()
    assert bool((buf[:, N:] == 7.0).all())
    got = buf[:, :N].cpu().double().numpy()
    want = mo.linear(a.double().numpy(), w.double().numpy(), b.double().numpy())
    # an fp32 sum rounded once to bf16, 2^-9 |y|; twice that, and as much of the typical |y| for results near zero
    bound = 2.0 ** -8 * np.abs(want) + 2.0 ** -8 * np.abs(want).mean()
    err = np.abs(got - want)
    assert (err <= bound).all(), "max excess %.3e at %s" % ((err - bound).max(), np.unravel_index((err - bound).argmax(), err.shape))


TILE_HEIGHTS = [
    # kernel, M, N, K: two K groups over tiles of 96, 160 and 192 tokens, ragged tiles, four features (mod 8) in the last ones
    (113, 2816, 892, 480),      # 7.5 slices; tiles of 32 token rows at the end
    (113, 3962, 676, 800),
    (161, 4962, 908, 544),      # 8.5 slices: the half slice with the first group
    (161, 1048, 3644, 1376),    # 21.5 slices
    (193, 2860, 2140, 800),     # 12.5 slices
    (193, 1300, 4596, 1120),
]


@pytest.mark.parametrize("M,N,K", [s[1:] for s in TILE_HEIGHTS])
def test_projection_tile_heights(M, N, K):
    test_projection_tiles(M, N, K)


HALF_SLICES = [
    # M, N, K: odd multiples of 32, the last K slice has 32 columns (kernel as picked by the size rule)
    (9001, 2304, 160),    # large tiles, 256 features
    (12001, 2596, 160),   # ... 288 features
    (8200, 1728, 288),    # ... full and tail tiles
    (1260, 576, 480),     # 64 x 64 tiles, K groups
    (700, 68, 96),        # ... without
]


@pytest.mark.parametrize("M,N,K", HALF_SLICES)
def test_infinite_weights_of_a_half_slice(M, N, K):
    """An infinite weight gives infinities with the sign of its token's element, never NaN, and only in its own feature."""
    from paper_2408_12588_amd import pab
    print("infinite weights", M, N, K, flush=True)
    a, w = rand((M, K), 1 + M), rand((N, K), 2 + N, 1.0 / math.sqrt(K))
    a[a == 0] = 1.0
    hit = {3: K - 32, 5: K - 1, N - 1: K - 7, 9: K - 33}     # feature: column of the half slice (the last: in the slice before it)
    for n, k in hit.items():
        w[n, k] = float("inf") if n != 5 else float("-inf")
    got = pab.pab_linear(a.to(DEV), w.to(DEV)).cpu()
    for n, k in hit.items():
        assert torch.equal(got[:, n].float(), (a[:, k].float() * w[n, k].float())), n
    rest = [n for n in range(N) if n not in hit]
    assert bool(torch.isfinite(got[:, rest].float()).all())


MODULES = [
    # kind, T, S, heads (of 72): sizes at which the projection normalises and rotates q and k itself, unless noted
    (0, 5, 1999, 4),     # no rotation, ragged token tail
    (1, 70, 130, 4),     # wavefronts whose tokens lie in two frames; frame indices beyond 63 (two digits of the table)
    (1, 160, 64, 4),     # shortest frames it takes: one per wavefront
    (1, 33, 301, 8),     # hidden size 576
    (1, 171, 60, 4),     # shorter frames: separate pass over q and k
]


@pytest.mark.parametrize("kind,T,S,heads", MODULES)
def test_norm_and_rotation(kind, T, S, heads):
    """Modules are independent per frame (spatial) or position (temporal): some of them against the oracle, held to
    1e-2 of the largest output as the modules are elsewhere (bf16 planes in between)."""
    from paper_2408_12588_amd import pab, workloads as W
    print("module", W.KIND_NAMES[kind], T, S, heads, flush=True)
    wl = W.Workload("norm", 1, T, S, 0, heads, 72, "bf16", 1, (1, 1, 0), 0, 0, seed=77 + T)
    x, w = W.make_module_input(wl, 0, kind, 0), W.make_module_weights(wl, 0, kind)
    wd = pab.module_weights(**{n: t.to(DEV) for n, t in w.items()})
    out = pab.pab_module_compute(kind, x.to(DEV), None, wd, heads).cpu()
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    f64 = lambda t: t.double().numpy()
    for i in (0, 2, T - 1) if kind == 0 else (0, 1, 63 % S, S // 2, S - 1):
        xi, got = (x[i:i + 1], out[i:i + 1]) if kind == 0 else (x[:, i:i + 1].contiguous(), out[:, i:i + 1])
        want = mo.self_attention_module(kind, f64(xi), f64(w["shift"]), f64(w["scale"]), f64(w["w_qkv"]), f64(w["b_qkv"]),
                                        f64(w["gamma_q"]), f64(w["beta_q"]), f64(w["gamma_k"]), f64(w["beta_k"]),
                                        f64(w["w_o"]), f64(w["b_o"]), heads)
        err = np.abs(f64(got) - want).max()
        assert err <= 1e-2 * np.abs(want).max(), (i, err, np.abs(want).max())


MOVED = [
    # kind, T, S, heads (of 72): tail tiles beside full ones, the last of most reaching back over rows of the one before it
    (1, 8, 1601, 16),
    (1, 17, 1024, 16),
    (1, 16, 1589, 16),
    (1, 8, 1100, 12),
    (1, 33, 301, 8),
    (0, 5, 1999, 4),
]


@pytest.mark.parametrize("kind,T,S,heads", MOVED)
def test_tokens_have_the_same_bits_in_every_tile(kind, T, S, heads):
    """Frames (spatial) and positions (temporal) are independent: moved to other rows of x, hence to other tiles of the
    projections, they give the same bits.  Rows that two tiles compute are stored by both, in either order."""
    from paper_2408_12588_amd import pab, workloads as W
    print("moved", W.KIND_NAMES[kind], T, S, heads, flush=True)
    wl = W.Workload("moved", 1, T, S, 0, heads, 72, "bf16", 1, (1, 1, 0), 0, 0, seed=31 + S)
    x = W.make_module_input(wl, 0, kind, 0).to(DEV)
    w = pab.module_weights(**{n: t.to(DEV) for n, t in W.make_module_weights(wl, 0, kind).items()})
    out = pab.pab_module_compute(kind, x, None, w, heads)
    for by in (1, S // 5, S // 2) if kind == 1 else (1, 2):
        moved = pab.pab_module_compute(kind, torch.roll(x, by, kind).contiguous(), None, w, heads)
        differ = int((moved != torch.roll(out, by, kind)).any(-1).sum())
        assert differ == 0, "moved by %d: %d tokens differ" % (by, differ)


@pytest.mark.parametrize("tokens,hidden", [(9001, 1152), (17001, 384), (12345, 864)])
def test_tokens_have_the_same_bits_in_every_tile_of_the_mlp(tokens, hidden):
    from paper_2408_12588_amd import pab
    print("moved mlp", tokens, hidden, flush=True)
    inner, dev = 4 * hidden, lambda *a: rand(*a).to(DEV)
    w = pab.mlp_weights(shift=dev((hidden,), 1, 0.3), scale=dev((hidden,), 2, 0.3), w1=dev((inner, hidden), 3, hidden ** -0.5),
                        b1=dev((inner,), 4, 0.1), w2=dev((hidden, inner), 5, inner ** -0.5), b2=dev((hidden,), 6, 0.1))
    x = dev((tokens, hidden), 7)
    out = pab.pab_mlp_compute(x, w, inner)
    for by in (1, 333, 1700):
        assert torch.equal(pab.pab_mlp_compute(torch.roll(x, by, 0).contiguous(), w, inner), torch.roll(out, by, 0))


CROSS_PAIRS = [
    # T, S, L, heads (of 72): the text's k / v projection in the launch of the query projection, as ...
    (5, 252, 60, 8),        # ... 64 x 64 tiles with K groups, ragged in the text
    (1, 1, 1, 4),           # ... one token, one text token
    (12, 500, 300, 12),     # ... more tiles than CUs
    (1, 900, 250, 16),      # ... the last of the K groups' 256 workgroups
    (1, 200, 100, 28),      # ... consecutive tiles along the tokens, of both problems
    (17, 1024, 64, 16),     # ... tiles of the last round of gemm_stream, 256 features: one of 64 rows
    (17, 1024, 100, 16),    # ... two of 64 rows, the second moved back
    (17, 1024, 131, 16),    # ... two of 128 rows, the second moved back
    (20, 1700, 64, 12),     # ... 288 features: one of 64 rows
    (20, 1700, 131, 12),    # ... two of 128 rows, the second moved back
    # ... or in one of its own:
    (8, 1590, 64, 16),      # no room in the last round
    (16, 1590, 131, 16),
    (16, 1590, 500, 16),    # long text
    (17, 1024, 63, 16),     # fewer than 64 text tokens: less than a tile of gemm_stream
    (16, 1590, 63, 16),     # ... and no room
    (1, 1300, 250, 16),     # K groups, more tiles than CUs in all
]
# of each: kernel of the query projection; rows / 64 of gemm_stream's tiles for the text; whether the text rides along
CROSS_PAIR_PATHS = [(65, 0, True), (64, 0, True), (128, 0, True), (97, 0, True), (65, 0, True), (8, 1, True), (8, 1, True), (8, 2, True),
                    (9, 1, True), (9, 2, True), (8, 0, False), (8, 0, False), (8, 0, False), (8, 0, False), (8, 0, False), (97, 0, False)]


HEIGHT_PAIRS = [
    # kernel, T, S, L, heads: sizes where tiles of 96, 160 or 192 tokens are the best ones for the queries alone.  Without room for the text:
    (129, 1, 2448, 300, 16), (129, 1, 3339, 64, 12), (129, 1, 4719, 90, 8), (128, 1, 7881, 200, 8), (193, 1, 4188, 40, 16), (128, 1, 5130, 300, 16),
    (113, 1, 3762, 40, 8), (161, 1, 3899, 16, 16), (193, 1, 8169, 64, 8),   # with room
]


@pytest.mark.parametrize("T,S,L,heads", [s[1:] for s in HEIGHT_PAIRS])
def test_query_and_text_projection_of_tile_heights(T, S, L, heads):
    test_query_and_text_projection(T, S, L, heads)


@pytest.mark.parametrize("T,S,L,heads", CROSS_PAIRS)
def test_query_and_text_projection(T, S, L, heads):
    """Cross modules are independent per token: some against the oracle, 1e-2 of the largest output as elsewhere."""
    from paper_2408_12588_amd import pab, workloads as W
    print("cross pair", T, S, L, heads, flush=True)
    wl = W.Workload("pair", 1, T, S, L, heads, 72, "bf16", 1, (0, 0, 1), 0, 0, seed=55 + L)
    x, text, w = W.make_module_input(wl, 0, W.CROSS, 0), W.make_text(wl), W.make_module_weights(wl, 0, W.CROSS)
    out = pab.pab_module_compute(W.CROSS, x.to(DEV), text.to(DEV), pab.module_weights(**{n: t.to(DEV) for n, t in w.items()}), heads)
    out = out.cpu().view(T * S, -1)
    assert torch.isfinite(out.float()).all()
    f64 = lambda t: t.double().numpy()
    rows = sorted({0, T * S // 3, T * S // 2, T * S - 65, T * S - 1} & set(range(T * S)))
    want = mo.cross_attention_module(f64(x.view(1, T * S, -1)[:, rows]), f64(text), *(f64(w[k]) for k in (
        "w_qkv", "b_qkv", "w_kv", "b_kv", "w_o", "b_o")), heads)[0]
    err = np.abs(f64(out[rows]) - want).max()
    assert err <= 1e-2 * np.abs(want).max(), (err, np.abs(want).max())


FEW_TOKENS = [
    # kind, T, S, heads, head dim: sizes at which q and k are normalised (and rotated) in the epilogue of gemm_heads
    (0, 1, 705, 8, 72),      # one token in the last token tile
    (1, 70, 3, 4, 72),       # several frames per tile, frame indices beyond 63; hidden size 288 = 4.5 slices: the second group ends early
    (1, 5, 90, 12, 72),      # hidden size 864 = 13.5 slices: the half slice with the second group
    (0, 1, 449, 16, 72),
    (1, 9, 21, 4, 32),       # heads of 32, three per tile: tiles across the q / k / v planes
    (0, 1, 1, 1, 32),        # one token, half a slice: the second group has none
]


HEADS_OF_32 = [
    # kernel, kind, T, S, heads: sizes at which gemm_tile normalises (and rotates) q and k, by its tile and K groups
    (64, 1, 7, 5, 3),        # planes that begin inside a tile, half a slice, frames shorter than a sub-tile
    (64, 1, 70, 1, 5),       # one token per frame, frame indices beyond 63
    (64, 0, 1, 700, 8),
    (65, 1, 11, 30, 16),
    (96, 1, 2, 679, 16),
    (97, 1, 20, 37, 16),
    (128, 1, 16, 351, 12),
    (129, 0, 3, 667, 16),
    (113, 1, 6, 407, 12),
    (161, 1, 17, 153, 19),   # planes that begin inside a tile
    (193, 1, 7, 354, 25),
]


HEADS_128 = [
    # kind, T, S, heads (of 72): gemm_heads with tiles of 128 tokens
    (0, 1, 1025, 16),        # one token in the last tile
    (1, 70, 45, 4),          # several frames per tile, frame indices beyond 63; 4.5 slices
    (1, 13, 117, 12),        # 13.5 slices: the half slice with the second group
    (1, 4, 358, 8),
]


@pytest.mark.parametrize("kind,T,S,heads", HEADS_128)
def test_norm_and_rotation_of_128_token_tiles(kind, T, S, heads):
    test_norm_and_rotation_few_tokens(kind, T, S, heads, 72)


@pytest.mark.parametrize("kind,T,S,heads,D", [s[1:] + (32,) for s in HEADS_OF_32])
def test_norm_and_rotation_of_heads_of_32(kind, T, S, heads, D):
    test_norm_and_rotation_few_tokens(kind, T, S, heads, D)


@pytest.mark.parametrize("kind,T,S,heads,D", FEW_TOKENS)
def test_norm_and_rotation_few_tokens(kind, T, S, heads, D):
    """Whole outputs against the oracle, 1e-2 of the largest output as for the modules elsewhere."""
    from paper_2408_12588_amd import pab, workloads as W
    print("few tokens", kind, T, S, heads, D, flush=True)
    f64 = lambda t: t.double().numpy()
    wl = W.Workload("few", 1, T, S, 0, heads, D, "bf16", 1, (1, 1, 0), 0, 0, seed=91 + S)
    x, w = W.make_module_input(wl, 0, kind, 0), W.make_module_weights(wl, 0, kind)
    out = pab.pab_module_compute(kind, x.to(DEV), None, pab.module_weights(**{k: t.to(DEV) for k, t in w.items()}), heads)
    want = mo.self_attention_module(kind, f64(x), *(f64(w[k]) for k in ("shift", "scale", "w_qkv", "b_qkv", "gamma_q", "beta_q",
                                                                        "gamma_k", "beta_k", "w_o", "b_o")), heads)
    err = np.abs(f64(out.cpu()) - want).max()
    assert err <= 1e-2 * np.abs(want).max(), (err, np.abs(want).max())
