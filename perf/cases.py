"""Cases that stand for what a program does with this library, through its public entry points.

Five forms of work, each with a range of sizes:

  video     a whole denoising run through ``PabContext.pab_attention``: every (block, kind, step) cell is computed into
            its cache slot or reused, as the broadcast schedule says
  op        one attention operation, ``pab_attention_compute``
  module    one attention module, ``pab_module_compute``: layernorm + modulate, projections, q / k layernorm (+ rotary),
            attention, output projection
  mlp       one MLP module, ``pab_mlp_compute``
  blocks    a denoising run of whole transformer blocks: attention modules and MLPs through ``PabContext`` and
            ``MlpContext``, both broadcast

Sizes are those of ``paper_2408_12588_amd.workloads`` (Tiny, 480p, 512 x 512, 512 x 512 long clip, 720p) and of the
tests.  Inputs are N(0,1) in the storage type and weights have rows of about unit norm, as everywhere in this repository;
``peaked`` scales one query token in twenty by 8, the stress recipe.
"""
import math

import torch

from paper_2408_12588_amd import pab, workloads

DEV = "cuda:0"
SPATIAL, TEMPORAL, CROSS = workloads.SPATIAL, workloads.TEMPORAL, workloads.CROSS
KINDS = {"spatial": SPATIAL, "temporal": TEMPORAL, "cross": CROSS}


def listed():
    return [
        # The Tiny configuration, end to end: 60 calls of a few microseconds each, fp32, head dim 32.  Launches and host
        # work are all there is: what a smoke test, an unpatched first run or a very small model pays.
        dict(name="video_tiny", form="video", dtype="f32", blocks=2, T=4, S=64, L=16, heads=4, head_dim=32, steps=10,
             spatial=2, temporal=4, cross=6, lo=2, hi=8, pool=4),
        # The 480p configuration, end to end: 30 steps of 28 blocks, the run that bench.py times.
        dict(name="video_480p", form="video", dtype="bf16", blocks=28, T=16, S=1590, L=120, heads=16, head_dim=72, steps=30,
             spatial=2, temporal=4, cross=6, lo=3, hi=27, pool=4),
        # A small clip at module level (a preview): attention modules and MLPs of three blocks over ten steps, about a
        # thousand tokens, where every projection is too small to fill the chip.
        dict(name="blocks_small", form="blocks", blocks=3, T=5, S=252, L=60, heads=8, head_dim=72, steps=10, spatial=2,
             temporal=4, cross=6, lo=2, hi=8, mlp_range=2),
        # Single operations at the sizes of the other configurations: a frame of 32 x 32 tokens (whole key tiles), ...
        dict(name="spatial_512", form="op", kind="spatial", dtype="bf16", T=16, S=1024, L=0, heads=16, head_dim=72, peaked=False),
        # ... of 45 x 80 tokens with a peaked softmax, the longest sequence, ...
        dict(name="spatial_720p", form="op", kind="spatial", dtype="bf16", T=16, S=3600, L=0, heads=16, head_dim=72, peaked=True),
        # ... temporal attention over 16 frames (a stream of rows through HBM), ...
        dict(name="temporal_480p", form="op", kind="temporal", dtype="bf16", T=16, S=1590, L=0, heads=16, head_dim=72, peaked=False),
        # ... cross attention to a short text and, on the 17-frame clip, to a long one.
        dict(name="cross_480p", form="op", kind="cross", dtype="bf16", T=16, S=1590, L=120, heads=16, head_dim=72, peaked=False),
        dict(name="cross_512_long", form="op", kind="cross", dtype="bf16", T=17, S=1024, L=300, heads=16, head_dim=72, peaked=False),
        # Modules: what is broadcast when the whole attention module is the cached object, one per kind.
        dict(name="module_spatial_480p", form="module", kind="spatial", T=16, S=1590, L=0, heads=16, head_dim=72),
        dict(name="module_temporal_512_long", form="module", kind="temporal", T=17, S=1024, L=0, heads=16, head_dim=72),
        dict(name="module_cross_480p", form="module", kind="cross", T=16, S=1590, L=120, heads=16, head_dim=72),
        # The MLP of a block: two projections, hidden size 1152 to 4608 and back.
        dict(name="mlp_480p", form="mlp", tokens=25440, hidden=1152, inner=4608),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    form = rng.choice(["video", "op", "op", "op", "module", "module", "mlp", "blocks"])
    if form == "video":
        dtype = rng.choice(["f32", "bf16"])
        steps = rng.randint(4, 10)
        return dict(form=form, dtype=dtype, blocks=rng.randint(1, 4), T=rng.randint(1, 16), S=_log_int(rng, 16, 400),
                    L=_log_int(rng, 4, 140), heads=rng.randint(1, 8), head_dim=rng.choice([32, 72]), steps=steps,
                    spatial=rng.randint(1, 3), temporal=rng.randint(1, 4), cross=rng.randint(1, 6), lo=1, hi=steps - 2, pool=2)
    if form == "op":
        kind = rng.choice(["spatial", "temporal", "cross"])
        return dict(form=form, kind=kind, dtype="bf16", T=rng.randint(4, 32 if kind == "temporal" else 17),
                    S=_log_int(rng, 128, 3600), L=_log_int(rng, 8, 512) if kind == "cross" else 0, heads=rng.randint(6, 16),
                    head_dim=rng.choice([72, 72, 72, 32]), peaked=kind != "temporal" and rng.random() < 0.25)
    if form == "module":   # the hidden size heads * head_dim is a multiple of 32
        kind = rng.choice(["spatial", "temporal", "cross"])
        return dict(form=form, kind=kind, T=rng.randint(2, 17), S=_log_int(rng, 64, 2400),
                    L=_log_int(rng, 8, 300) if kind == "cross" else 0, heads=4 * rng.randint(1, 4), head_dim=rng.choice([72, 72, 32]))
    if form == "mlp":
        hidden = rng.choice([288, 384, 576, 768, 864, 1152, 1152])
        return dict(form=form, tokens=_log_int(rng, 300, 40000), hidden=hidden, inner=4 * hidden)
    steps = rng.randint(4, 8)
    return dict(form=form, blocks=rng.randint(1, 4), T=rng.randint(2, 12), S=_log_int(rng, 32, 600), L=_log_int(rng, 8, 140),
                heads=rng.choice([4, 8, 12, 16]), head_dim=72, steps=steps, spatial=rng.randint(1, 3), temporal=rng.randint(1, 4),
                cross=rng.randint(1, 6), lo=1, hi=steps - 2, mlp_range=2)


# ---- inputs ------------------------------------------------------------------------------------------------------------
class _Source:
    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)

    def randn(self, shape, scale=1.0, offset=0.0, dtype=torch.bfloat16):
        x = torch.randn(shape, generator=self.gen, device=DEV, dtype=torch.float32)
        return x.mul_(scale).add_(offset).to(dtype)

    def qkv(self, case, kind, dtype, peaked=False):
        T, S, H, D = case["T"], case["S"], case["heads"], case["head_dim"]
        kv = (case["L"], H, D) if kind == CROSS else (T, S, H, D)
        q = self.randn((T, S, H, D), dtype=dtype)
        if peaked:
            rows = torch.randperm(T * S, generator=self.gen, device=DEV)[:T * S // 20]
            q.view(T * S, H, D)[rows] *= 8.0
        return q, self.randn(kv, dtype=dtype), self.randn(kv, dtype=dtype)

    def module_weights(self, kind, C, D):
        unit = 1.0 / math.sqrt(C)
        w = dict(w_o=self.randn((C, C), unit), b_o=self.randn((C,), 0.1))
        if kind == CROSS:
            w.update(w_qkv=self.randn((C, C), unit), b_qkv=self.randn((C,), 0.1), w_kv=self.randn((2 * C, C), unit),
                     b_kv=self.randn((2 * C,), 0.1))
        else:
            w.update(shift=self.randn((C,), 0.3), scale=self.randn((C,), 0.3), w_qkv=self.randn((3 * C, C), unit),
                     b_qkv=self.randn((3 * C,), 0.1), gamma_q=self.randn((D,), 0.2, 1.0), beta_q=self.randn((D,), 0.2),
                     gamma_k=self.randn((D,), 0.2, 1.0), beta_k=self.randn((D,), 0.2))
        return pab.module_weights(**w)

    def mlp_weights(self, C, F):
        return pab.mlp_weights(shift=self.randn((C,), 0.3), scale=self.randn((C,), 0.3), w1=self.randn((F, C), 1.0 / math.sqrt(C)),
                               b1=self.randn((F,), 0.1), w2=self.randn((C, F), 1.0 / math.sqrt(F)), b2=self.randn((C,), 0.1))


def _context(case, dtype):
    """The run's context over a cleared cache (slots are rounded up in size; what lies between them is defined)."""
    cfg = pab.make_config(case["blocks"], case["T"], case["S"], case["L"], case["heads"], case["head_dim"], dtype,
                          case["steps"], (case["spatial"], case["temporal"], case["cross"]), case["lo"], case["hi"])
    return pab.PabContext(cfg, DEV, workspace=torch.zeros(pab.pab_workspace_bytes(cfg), dtype=torch.uint8, device=DEV))


def _mlp_starts(case):
    return list(range(case["lo"], case["hi"], case["mlp_range"] + 1))


def prepare(case, seed):
    src = _Source(seed)
    form = case["form"]
    if form == "video":
        dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        pool = [[src.qkv(case, kind, dtype) for kind in (SPATIAL, TEMPORAL, CROSS)] for _ in range(case["pool"])]
        return dict(case=case, ctx=_context(case, pab.BF16 if case["dtype"] == "bf16" else pab.F32), pool=pool, dtype=dtype)
    if form == "op":
        dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        q, k, v = src.qkv(case, KINDS[case["kind"]], dtype, case["peaked"])
        return dict(case=case, q=q, k=k, v=v, out=torch.empty_like(q))
    if form == "mlp":
        n, C, F = case["tokens"], case["hidden"], case["inner"]
        x = src.randn((n, C))
        return dict(case=case, x=x, w=src.mlp_weights(C, F), scratch=pab.mlp_scratch(n, C, F, DEV), out=torch.empty_like(x))
    T, S, L, H, D = case["T"], case["S"], case["L"], case["heads"], case["head_dim"]
    C = H * D
    scratch = pab.module_scratch(T, S, L, H, D, DEV)
    text = src.randn((L, C)) if L else None
    if form == "module":
        x = src.randn((T, S, C))
        return dict(case=case, x=x, text=text, w=src.module_weights(KINDS[case["kind"]], C, D), scratch=scratch, out=torch.empty_like(x))
    # blocks: one hidden state per step and call site, one weight set per (block, module)
    n, F = T * S, 4 * C
    mlp = pab.MlpContext(case["blocks"], case["steps"], n, C, F, _mlp_starts(case), case["mlp_range"], 0, case["blocks"] - 1, DEV)
    mlp.workspace.zero_()
    return dict(case=case, ctx=_context(case, pab.BF16), mlp=mlp, text=text, scratch=scratch, mlp_scratch=pab.mlp_scratch(n, C, F, DEV),
                xs=[src.randn((T, S, C)) for _ in range(4)],
                ws=[[src.module_weights(kind, C, D) for kind in (SPATIAL, TEMPORAL, CROSS)] for _ in range(case["blocks"])],
                mlp_ws=[src.mlp_weights(C, F) for _ in range(case["blocks"])])


# ---- one pass ----------------------------------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    form = case["form"]
    if form == "op":
        return pab.pab_attention_compute(KINDS[case["kind"]], state["q"], state["k"], state["v"], out=state["out"])
    if form == "module":
        return pab.pab_module_compute(KINDS[case["kind"]], state["x"], state["text"], state["w"], case["heads"],
                                      scratch=state["scratch"], out=state["out"])
    if form == "mlp":
        return pab.pab_mlp_compute(state["x"], state["w"], case["inner"], scratch=state["scratch"], out=state["out"])
    ctx = state["ctx"]
    ctx.pab_reset()
    if form == "video":
        pool, i = state["pool"], 0
        for step in range(case["steps"]):
            for block in range(case["blocks"]):
                for kind in (SPATIAL, TEMPORAL, CROSS):
                    q, k, v = pool[i % len(pool)][kind]
                    ctx.pab_attention(block, kind, step, q, k, v)
                    i += 1
        return ctx.workspace.view(state["dtype"])
    mlp = state["mlp"]
    mlp.pab_mlp_reset()
    xs, i = state["xs"], 0
    for step in range(case["steps"]):
        for block in range(case["blocks"]):
            for kind in (SPATIAL, TEMPORAL, CROSS):
                ctx.pab_module_attention(block, kind, step, xs[i % len(xs)], state["text"], state["ws"][block][kind], state["scratch"])
                i += 1
            mlp.pab_mlp(block, step, xs[i % len(xs)], state["mlp_ws"][block], state["mlp_scratch"])
            i += 1
    return ctx.workspace.view(torch.bfloat16), mlp.workspace.view(torch.bfloat16)


# ---- what a pass cannot do without -------------------------------------------------------------------------------------
def _op_work(case, kind, size):
    T, S, L, H, D = case["T"], case["S"], case["L"], case["heads"], case["head_dim"]
    n = T * S
    keys = S if kind == SPATIAL else T if kind == TEMPORAL else L
    rows = 2 * n + 2 * (L if kind == CROSS else n)
    return rows * H * D * size, 4.0 * n * H * keys * D


def _module_work(case, kind):
    """x and the weights read, the output written; projections and attention."""
    n, L, C, D = case["T"] * case["S"], case["L"], case["heads"] * case["head_dim"], case["head_dim"]
    flops = _op_work(case, kind, 2)[1] + 2.0 * n * C * C
    if kind == CROSS:
        return 2.0 * (2 * n * C + L * C + 4 * C * C + 4 * C), flops + 2.0 * (n + 2 * L) * C * C
    return 2.0 * (2 * n * C + 4 * C * C + 6 * C + 4 * D), flops + 6.0 * n * C * C


def _mlp_work(n, C, F):
    return 2.0 * (2 * n * C + 2 * C * F + F + 3 * C), 4.0 * n * C * F


def work(case):
    form = case["form"]
    if form == "op":
        b, f = _op_work(case, KINDS[case["kind"]], 2 if case["dtype"] == "bf16" else 4)
        return {"bytes": b, "flops": f}
    if form == "module":
        b, f = _module_work(case, KINDS[case["kind"]])
        return {"bytes": b, "flops": f}
    if form == "mlp":
        b, f = _mlp_work(case["tokens"], case["hidden"], case["inner"])
        return {"bytes": b, "flops": f}
    total_b = total_f = 0.0
    for kind, name in ((SPATIAL, "spatial"), (TEMPORAL, "temporal"), (CROSS, "cross")):
        computed = sum(pab.pab_schedule(kind, s, case["lo"], case["hi"], case[name]) == pab.COMPUTE for s in range(case["steps"]))
        if form == "video":
            b, f = _op_work(case, kind, 2 if case["dtype"] == "bf16" else 4)
        else:
            b, f = _module_work(case, kind)
        total_b, total_f = total_b + computed * case["blocks"] * b, total_f + computed * case["blocks"] * f
    if form == "blocks":
        C = case["heads"] * case["head_dim"]
        b, f = _mlp_work(case["T"] * case["S"], C, 4 * C)
        starts, last = _mlp_starts(case), case["blocks"] - 1
        computed = sum(pab.pab_mlp_schedule(s, 0, starts, case["mlp_range"], 0, last) == pab.COMPUTE for s in range(case["steps"]))
        total_b, total_f = total_b + computed * case["blocks"] * b, total_f + computed * case["blocks"] * f
    return {"bytes": total_b, "flops": total_f}


def tolerance(case):
    # Operands, probabilities and intermediate planes are rounded to bf16 (2^-9 each), sums are fp32.  Relative error
    # against the same path in float64, measured at these sizes: operations 1.8e-3 .. 2.4e-3 (fp32 rows, which are
    # rounded on load, 2.4e-3 .. 3.2e-3), the MLP 2.9e-3, attention modules, where more roundings follow each other,
    # 2.4e-3 .. 4.0e-3.  Four times that:
    return {"rel": 0.015 if case["form"] in ("module", "blocks") else 0.01}
