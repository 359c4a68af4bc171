"""Host-side behaviour of libpab.so that needs no GPU: the library loads, exports
what include/pab.h declares, its schedule equals the oracle's bit for bit, and
argument errors come back as negative status codes."""
import ctypes
import os
import random
import re

import pytest

from oracle import pab_oracle as orc
from paper_2408_12588_amd import pab, workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_exports_match_header():
    text = open(os.path.join(ROOT, "include", "pab.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(pab_[a-z_]+)\s*\(", text))
    assert declared == set(pab.EXPORTS)
    for name in declared:
        assert hasattr(pab.lib, name), name


@pytest.mark.parametrize("wl", W.CONFIGS, ids=lambda w: w.name)
def test_schedule_equals_oracle_on_workloads(wl):
    for kind in range(3):
        n = wl.intervals[kind]
        if n == 0:
            continue
        for s in range(wl.n_steps):
            assert pab.pab_schedule(kind, s, wl.lo, wl.hi, n) == orc.schedule(s, wl.lo, wl.hi, n)
            assert pab.pab_source_step(kind, s, wl.lo, wl.hi, n) == orc.source_step(s, wl.lo, wl.hi, n)
        # the no-broadcast baseline computes every step
        assert all(pab.pab_schedule(kind, s, wl.lo, wl.hi, 1) == pab.COMPUTE for s in range(wl.n_steps))


def test_schedule_golden_rows(golden_schedule_rows):
    for name, n_steps, lo, hi, n, pattern in golden_schedule_rows:
        got = "".join("CR"[pab.pab_schedule(0, s, lo, hi, n)] for s in range(n_steps))
        assert got == pattern, name


def test_schedule_fuzz_against_oracle():
    rng = random.Random(99)
    for _ in range(20000):
        s = rng.randint(0, 400)
        lo = rng.randint(0, 300)
        hi = rng.randint(lo, 400)
        n = rng.randint(1, 16)
        kind = rng.randint(0, 2)
        assert pab.pab_schedule(kind, s, lo, hi, n) == orc.schedule(s, lo, hi, n)
        assert pab.pab_source_step(kind, s, lo, hi, n) == orc.source_step(s, lo, hi, n)


def test_schedule_errors():
    for args in [(3, 0, 0, 5, 2), (-1, 0, 0, 5, 2), (0, -1, 0, 5, 2), (0, 0, 0, 5, 0), (0, 0, 6, 5, 2),
                 (0, 0, -1, 5, 2), (0, 2**31 - 1, -2**31, 5, 2)]:   # a negative window start is refused, not wrapped
        assert pab.lib.pab_schedule(*args) == pab.EINVAL
        assert pab.lib.pab_source_step(*args) == pab.EINVAL
        assert pab.pab_last_error() != ""
        with pytest.raises(pab.PabError):
            pab.pab_schedule(*args)


def test_timestep_window_equals_oracle(golden_timestep_windows):
    windows, rows, _ = golden_timestep_windows
    for name, n_steps, first, stride, t_start, t_end, lo, hi in windows:
        ts = [first - s * stride for s in range(n_steps)]
        got = pab.pab_window_from_timesteps(ts, t_start, t_end)
        assert got == orc.window_from_timesteps(ts, t_start, t_end), name
        assert got == (None if lo < 0 else (lo, hi)), name
    # the paper's three Open-Sora settings on the first window, row by row
    name, n_steps, first, stride, t_start, t_end, lo, hi = windows[0]
    w = pab.pab_window_from_timesteps([first - s * stride for s in range(n_steps)], t_start, t_end)
    for rname, n, pattern in rows:
        assert "".join("CR"[pab.pab_schedule(0, s, w[0], w[1], n)] for s in range(n_steps)) == pattern, rname
    rng = random.Random(3)
    for _ in range(3000):
        n = rng.randint(1, 60)
        ts = sorted((rng.choice([rng.randint(0, 1000), rng.uniform(0, 1000)]) for _ in range(n)), reverse=True)
        a, b = sorted((rng.uniform(-50, 1050), rng.uniform(-50, 1050)))
        assert pab.pab_window_from_timesteps(ts, b, a) == orc.window_from_timesteps(ts, b, a)


def test_timestep_window_errors():
    lo, hi = ctypes.c_int(7), ctypes.c_int(8)
    arr = (ctypes.c_double * 3)(900.0, 500.0, 100.0)
    f = pab.lib.pab_window_from_timesteps
    assert f(None, 3, 900.0, 100.0, ctypes.byref(lo), ctypes.byref(hi)) == pab.EINVAL
    assert f(arr, 0, 900.0, 100.0, ctypes.byref(lo), ctypes.byref(hi)) == pab.EINVAL
    assert f(arr, 3, 100.0, 900.0, ctypes.byref(lo), ctypes.byref(hi)) == pab.EINVAL
    assert f(arr, 3, float("nan"), 100.0, ctypes.byref(lo), ctypes.byref(hi)) == pab.EINVAL
    up = (ctypes.c_double * 3)(100.0, 500.0, 900.0)
    assert f(up, 3, 900.0, 100.0, ctypes.byref(lo), ctypes.byref(hi)) == pab.EINVAL
    assert f(arr, 3, 900.0, 100.0, None, ctypes.byref(hi)) == pab.EINVAL
    assert (lo.value, hi.value) == (7, 8)                      # untouched by failures ...
    assert f(arr, 3, 450.0, 150.0, ctypes.byref(lo), ctypes.byref(hi)) == 0
    assert (lo.value, hi.value) == (7, 8)                      # ... and by an empty window
    assert f(arr, 3, 900.0, 500.0, ctypes.byref(lo), ctypes.byref(hi)) == 2
    assert (lo.value, hi.value) == (0, 1)


def test_presets_are_the_papers_table(golden_timestep_windows):
    _, _, presets = golden_timestep_windows
    models = {"open_sora": pab.OPEN_SORA, "open_sora_plan": pab.OPEN_SORA_PLAN, "latte": pab.LATTE}
    assert len(presets) == 9
    for model, level, ranges, t_start, t_end in presets:
        assert pab.pab_preset(models[model], level) == (ranges, t_start, t_end), (model, level)
    for model in range(3):   # the pyramid (Sec. 2.3): spatial < temporal < cross, and levels get more aggressive
        prev = (0, 0, 0)
        for level in range(3):
            r, _, _ = pab.pab_preset(model, level)
            assert r[0] < r[1] < r[2]
            assert all(a >= b for a, b in zip(r, prev)) and r != prev
            prev = r
    iv = (ctypes.c_int * 3)()
    a, b = ctypes.c_double(), ctypes.c_double()
    for model, level in ((3, 0), (-1, 0), (0, 3), (0, -1)):
        assert pab.lib.pab_preset(model, level, iv, ctypes.byref(a), ctypes.byref(b)) == pab.EINVAL
    assert pab.lib.pab_preset(0, 0, None, ctypes.byref(a), ctypes.byref(b)) == pab.EINVAL


def test_mlp_schedule_equals_oracle():
    rng = random.Random(17)
    for _ in range(4000):
        n_steps = rng.randint(1, 60)
        starts = sorted(rng.sample(range(n_steps), rng.randint(0, min(6, n_steps))))
        n = rng.randint(1, 5)
        blo = rng.randint(0, 6)
        bhi = rng.randint(blo, 10)
        step, block = rng.randint(0, n_steps + 3), rng.randint(0, 12)
        dec, src = orc.mlp_schedule(step, block, starts, n, blo, bhi)
        assert pab.pab_mlp_schedule(step, block, starts, n, blo, bhi) == dec
        assert pab.pab_mlp_source_step(step, block, starts, n, blo, bhi) == src
    # the hand-mapped rows of the fixture file
    with open(os.path.join(ROOT, "tests", "golden", "timestep_windows.txt")) as f:
        rows = [l[4:].split("|") for l in f if l.startswith("mlp ")]
    assert len(rows) == 2
    for head, steps, pattern in rows:
        h = head.split()
        first, stride, n_steps, n, blo, bhi = (int(v) for v in h[1:7])
        ts = [first - s * stride for s in range(n_steps)]
        starts = pab.pab_steps_from_timesteps(ts, [int(v) for v in h[7:]])
        assert starts == [int(v) for v in steps.split()] == orc.start_steps_from_timesteps(ts, [int(v) for v in h[7:]])
        assert "".join("CR"[pab.pab_mlp_schedule(s, blo, starts, n, blo, bhi)] for s in range(n_steps)) == pattern.strip()
    assert pab.pab_steps_from_timesteps([900, 800, 700], [950, 800, 750, 10]) == [0, 1, 2, None]
    for args in [(-1, 0, [1], 2, 0, 1), (0, -1, [1], 2, 0, 1), (0, 0, [1], 0, 0, 1), (0, 0, [-2], 2, 0, 1)]:
        with pytest.raises(pab.PabError):
            pab.pab_mlp_schedule(*args)


def test_mlp_context_errors_without_device():
    cfg = pab.pab_mlp_config(4, 10, 64, 128, 512, 1, 2, 0, 1)
    assert pab.lib.pab_mlp_workspace_bytes(ctypes.byref(cfg)) == 2 * 64 * 128 * 2
    assert pab.lib.pab_mlp_scratch_bytes(64, 128, 512) == 64 * 128 * 2 + 64 * 512 * 2
    starts = (ctypes.c_int * 1)(3)
    h = ctypes.c_void_p()
    fake = 0x10000
    assert pab.lib.pab_mlp_create(ctypes.byref(cfg), starts, fake, 100, ctypes.byref(h)) == pab.ENOMEM
    assert pab.lib.pab_mlp_create(ctypes.byref(cfg), starts, fake + 8, 1 << 20, ctypes.byref(h)) == pab.EINVAL
    bad = pab.pab_mlp_config(4, 10, 64, 100, 512, 1, 2, 0, 1)          # hidden not a multiple of 32
    assert pab.lib.pab_mlp_create(ctypes.byref(bad), starts, fake, 1 << 20, ctypes.byref(h)) == pab.EINVAL
    late = (ctypes.c_int * 1)(10)                                       # starting step outside the run
    assert pab.lib.pab_mlp_create(ctypes.byref(cfg), late, fake, 1 << 20, ctypes.byref(h)) == pab.EINVAL
    # two broadcasts that overlap (starts closer than the range) are refused; the same start twice is one broadcast
    wide = pab.pab_mlp_config(4, 10, 64, 128, 512, 2, 3, 0, 1)
    assert pab.lib.pab_mlp_create(ctypes.byref(wide), (ctypes.c_int * 2)(3, 4), fake, 1 << 20, ctypes.byref(h)) == pab.EINVAL
    assert "closer than the broadcast range" in pab.pab_last_error()
    assert pab.lib.pab_mlp_create(ctypes.byref(wide), (ctypes.c_int * 2)(5, 3), fake, 1 << 20, ctypes.byref(h)) == pab.EINVAL
    assert pab.lib.pab_mlp_create(ctypes.byref(wide), (ctypes.c_int * 2)(3, 6), fake, 1 << 20, ctypes.byref(h)) == pab.OK
    assert pab.lib.pab_mlp_destroy(h) == pab.OK
    assert pab.lib.pab_mlp_create(ctypes.byref(wide), (ctypes.c_int * 2)(3, 3), fake, 1 << 20, ctypes.byref(h)) == pab.OK
    assert pab.lib.pab_mlp_destroy(h) == pab.OK
    assert pab.lib.pab_mlp_create(ctypes.byref(cfg), starts, fake, 1 << 20, ctypes.byref(h)) == pab.OK
    # slots of the participating blocks 0 and 1, none for the others
    assert pab.lib.pab_mlp_slot_ptr(h, 0) == fake and pab.lib.pab_mlp_slot_ptr(h, 1) == fake + 64 * 128 * 2
    assert pab.lib.pab_mlp_slot_ptr(h, 2) is None and pab.lib.pab_mlp_slot_ptr(h, -1) is None
    assert pab.lib.pab_mlp_slot_ptr(None, 0) is None
    out = ctypes.c_void_p()
    w = pab.pab_mlp_weights()
    # a reuse before anything was computed, a block out of range, a computed step without inputs
    assert pab.lib.pab_mlp(h, 0, 4, None, None, None, 0, None, None, ctypes.byref(out)) == pab.ESTATE
    assert pab.lib.pab_mlp(h, 4, 0, None, None, None, 0, None, None, ctypes.byref(out)) == pab.EINVAL
    assert pab.lib.pab_mlp(h, 0, 0, None, ctypes.byref(w), None, 0, None, None, ctypes.byref(out)) == pab.EINVAL
    assert pab.lib.pab_mlp(h, 3, 0, fake, ctypes.byref(w), fake, 1 << 20, None, None, ctypes.byref(out)) == pab.EINVAL   # uncached block, no y
    assert pab.lib.pab_mlp_launch_count(h) == 0
    assert pab.lib.pab_mlp_destroy(h) == pab.OK


def test_workspace_bytes():
    cfg = pab.config_of(W.OPENSORA_480P)
    slot = 16 * 1590 * 16 * 72 * 2
    assert slot % 256 == 0
    assert pab.pab_workspace_bytes(cfg) == 28 * 3 * slot
    # alternating blocks (one kind each) get one slot per block; without the mask every block gets both kinds
    assert pab.pab_workspace_bytes(pab.config_of(W.LATTE_512)) == 28 * 16 * 1024 * 16 * 72 * 2
    wl = W.LATTE_512
    unmasked = pab.make_config(wl.n_blocks, wl.T, wl.S, wl.L, wl.heads, wl.head_dim, pab.BF16, wl.n_steps, wl.intervals,
                               wl.lo, wl.hi)
    assert pab.pab_workspace_bytes(unmasked) == 28 * 2 * 16 * 1024 * 16 * 72 * 2
    tiny = pab.config_of(W.TINY)
    assert pab.pab_workspace_bytes(tiny) == 2 * 3 * 4 * 64 * 4 * 32 * 4
    bad = pab.config_of(W.TINY)
    bad.head_dim = 48
    assert pab.lib.pab_workspace_bytes(ctypes.byref(bad)) == 0 and "head_dim" in pab.pab_last_error()
    assert pab.lib.pab_workspace_bytes(None) == 0


def _create(cfg, ptr, nbytes):
    h = ctypes.c_void_p()
    rc = pab.lib.pab_create(ctypes.byref(cfg), ptr, nbytes, ctypes.byref(h))
    return rc, h


def test_create_and_attention_errors_without_device():
    # pab_create only does pointer arithmetic on the workspace, so a made-up aligned
    # address is enough to walk the error paths; nothing here launches a kernel.
    cfg = pab.config_of(W.TINY)
    need = pab.pab_workspace_bytes(cfg)
    fake = 0x10000000
    assert _create(cfg, fake, need - 1)[0] == pab.ENOMEM
    assert _create(cfg, fake + 16, need)[0] == pab.EINVAL          # not 256-byte aligned
    assert _create(cfg, None, need)[0] == pab.EINVAL
    assert pab.lib.pab_create(ctypes.byref(cfg), fake, need, None) == pab.EINVAL
    for field, val in [("n_blocks", 0), ("T", 0), ("S", -1), ("heads", 0), ("head_dim", 64), ("dtype", 7),
                       ("n_steps", 0), ("range_lo", -1), ("range_hi", 0), ("L", 0)]:
        bad = pab.config_of(W.TINY)
        setattr(bad, field, val)
        assert _create(bad, fake, need)[0] == pab.EINVAL, field
    bad = pab.config_of(W.TINY)
    bad.interval[1] = -1
    assert _create(bad, fake, need)[0] == pab.EINVAL
    bad.interval[0] = bad.interval[1] = bad.interval[2] = 0
    assert _create(bad, fake, need)[0] == pab.EINVAL

    rc, h = _create(cfg, fake, need)
    assert rc == pab.OK and h.value
    out = ctypes.c_void_p()
    att = lambda *a: pab.lib.pab_attention(h, *a, ctypes.byref(out))
    assert att(0, 3, 0, 16, 16, 16, None) == pab.EINVAL          # bad kind
    assert att(2, 0, 0, 16, 16, 16, None) == pab.EINVAL          # block out of range
    assert att(0, 0, 10, 16, 16, 16, None) == pab.EINVAL         # step out of range
    assert att(0, 0, 0, None, 16, 16, None) == pab.EINVAL        # NULL q on a computed step
    assert att(0, 0, 0, 8, 16, 16, None) == pab.EINVAL           # misaligned q
    assert pab.lib.pab_attention(h, 0, 0, 0, 16, 16, 16, None, None) == pab.EINVAL
    assert pab.lib.pab_attention(None, 0, 0, 0, 16, 16, 16, None, ctypes.byref(out)) == pab.EINVAL
    # step 3 of the tiny spatial row is a reuse step, but nothing was computed yet
    assert att(0, 0, 3, None, None, None, None) == pab.ESTATE
    assert "needs the output of step 2" in pab.pab_last_error() and "holds step -1" in pab.pab_last_error()
    assert pab.lib.pab_launch_count(h) == 0
    # slots are laid out block-major, kind-minor
    slot = 4 * 64 * 4 * 32 * 4
    assert pab.lib.pab_slot_ptr(h, 0, 0) == fake
    assert pab.lib.pab_slot_ptr(h, 1, 2) == fake + 5 * slot
    assert pab.lib.pab_slot_ptr(h, 2, 0) is None and pab.lib.pab_slot_ptr(h, 0, 3) is None
    assert pab.lib.pab_reset(h) == pab.OK
    assert pab.lib.pab_destroy(h) == pab.OK
    assert pab.lib.pab_destroy(None) == pab.EINVAL and pab.lib.pab_reset(None) == pab.EINVAL
    assert pab.lib.pab_launch_count(None) == -1

    # a config without cross attention has no cross slot and rejects cross calls; its blocks alternate between
    # spatial and temporal attention (block_kinds), so block b owns slot b and nothing else
    latte = pab.config_of(W.LATTE_512)
    slot = 16 * 1024 * 16 * 72 * 2
    rc, h = _create(latte, fake, pab.pab_workspace_bytes(latte))
    assert rc == pab.OK
    assert pab.lib.pab_attention(h, 0, 2, 0, 16, 16, 16, None, ctypes.byref(out)) == pab.EINVAL
    assert pab.lib.pab_slot_ptr(h, 0, 2) is None
    assert pab.lib.pab_slot_ptr(h, 0, 0) == fake and pab.lib.pab_slot_ptr(h, 0, 1) is None
    assert pab.lib.pab_slot_ptr(h, 1, 1) == fake + slot and pab.lib.pab_slot_ptr(h, 1, 0) is None
    assert pab.lib.pab_slot_ptr(h, 27, 1) == fake + 27 * slot
    assert pab.lib.pab_attention(h, 1, 0, 0, 16, 16, 16, None, ctypes.byref(out)) == pab.EINVAL   # block 1 is temporal
    assert "block_kinds" in pab.pab_last_error()
    pab.lib.pab_destroy(h)
    # the mask may only name kinds that have a broadcast range, and only the three kinds
    wl = W.LATTE_512
    for mask in ([4] + [1] * 27, [8] + [1] * 27):
        bad = pab.make_config(wl.n_blocks, wl.T, wl.S, wl.L, wl.heads, wl.head_dim, pab.BF16, wl.n_steps, wl.intervals,
                              wl.lo, wl.hi, mask)
        assert _create(bad, fake, 1 << 40)[0] == pab.EINVAL and "block_kinds" in pab.pab_last_error()
    # a mixed mask: block 0 has both kinds, block 1 none, block 2 temporal only
    mixed = pab.make_config(3, wl.T, wl.S, wl.L, wl.heads, wl.head_dim, pab.BF16, wl.n_steps, wl.intervals, wl.lo, wl.hi,
                            [3, 0, 2])
    assert pab.pab_workspace_bytes(mixed) == 3 * slot
    rc, h = _create(mixed, fake, 3 * slot)
    assert rc == pab.OK
    assert [pab.lib.pab_slot_ptr(h, b, k) for b in range(3) for k in range(2)] == \
        [fake, fake + slot, None, None, None, fake + 2 * slot]
    pab.lib.pab_destroy(h)


def test_compute_argument_errors_without_device():
    f = pab.lib.pab_attention_compute
    ok = (0, pab.BF16, 2, 8, 4, 2, 72)
    assert f(*ok, None, 16, 16, 16, None) == pab.EINVAL
    assert f(*ok, 16, 16, 16, 24, None) == pab.EINVAL              # misaligned o
    assert f(0, pab.BF16, 2, 8, 4, 2, 64, 16, 16, 16, 16, None) == pab.EINVAL   # head_dim
    assert f(2, pab.BF16, 2, 8, 0, 2, 72, 16, 16, 16, 16, None) == pab.EINVAL   # cross without keys
    assert f(5, pab.BF16, 2, 8, 4, 2, 72, 16, 16, 16, 16, None) == pab.EINVAL
    assert f(0, 3, 2, 8, 4, 2, 72, 16, 16, 16, 16, None) == pab.EINVAL
    assert f(0, pab.BF16, 0, 8, 4, 2, 72, 16, 16, 16, 16, None) == pab.EINVAL


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_argument_without_torch_internals(monkeypatch, missing):
    """A torch build that lacks the raw stream functions: calls go to the current stream all the same."""
    import types
    import torch
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream" if missing == "_cuda_getDevice" else "_cuda_getDevice",
                        lambda *a: 0, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=1234))
    assert pab._stream(None) == 1234
    assert pab._stream(7) == 7


def test_native_binding_leaves_the_unusual_to_python():
    """The native binding takes plain numbers and dense device tensors and hands back everything else; errors are the same."""
    import torch
    b = pab._binding
    cfg = pab.config_of(W.TINY)
    rc, h = _create(cfg, 0x10000000, pab.pab_workspace_bytes(cfg))
    assert rc == pab.OK
    for args in [(3, 0, 0), (0, 3, 0), (2, 0, 0), (0, 0, 10), (0, 0, -1)]:     # out of range: raised, not handed back
        block, kind, step = args
        with pytest.raises(pab.PabError) as e:
            b.attention(h.value, block, kind, step, 16, 16, 16, 0)
        assert e.value.status == pab.EINVAL
    with pytest.raises(pab.PabError) as e:
        b.attention(h.value, 0, 0, 3, None, None, None, 0)
    assert e.value.status == pab.ESTATE and "needs the output of step 2" in str(e.value)
    with pytest.raises(pab.PabError) as e:
        b.attention(None, 0, 0, 0, 16, 16, 16, 0)                              # a destroyed context
    assert e.value.status == pab.EINVAL

    class Sub(torch.Tensor):
        pass
    t = torch.zeros(4, 64, 4, 32)
    for odd in (t, t.as_subclass(Sub), torch.nn.Parameter(t), torch.zeros(4, 64, 4, 32, device="meta"), 1.0, "x", 2 ** 70):
        assert b.attention(h.value, 0, 0, 0, odd, 16, 16, 0) is NotImplemented, odd
        assert b.attention_compute(0, odd, odd, odd, odd, 0) is NotImplemented, odd
    for odd in (1.0, True, None, 2 ** 70):
        assert b.attention(h.value, odd, 0, 0, 16, 16, 16, 0) is NotImplemented, odd
    assert b.attention(h.value, 0, 0, 0, 16, 16, 16, None) is NotImplemented   # no device tensor: which stream, Python decides
    assert b.attention(h.value, 0, 0, 0, 16, 16, 16, object()) is NotImplemented
    for wrong in ((), (1,) * 7, (1,) * 9):
        with pytest.raises(TypeError):
            b.attention(*wrong)
    pab.lib.pab_destroy(h)


def _package_copy(tmp_path, binding):
    """This package with libpab.so and, unless None, `binding` as the content of its native binding."""
    import shutil
    import torch
    here = os.path.dirname(pab.__file__)
    there = tmp_path / os.path.basename(here)
    there.mkdir()
    for name in os.listdir(here):
        if name.endswith(".py") or name == "libpab.so":
            shutil.copy(os.path.join(here, name), there / name)
    if binding is not None:
        (there / os.path.basename(pab.binding_path(torch.__version__))).write_bytes(binding)
    return there


@pytest.mark.parametrize("binding", [None, b"built for another machine"])
def test_package_works_without_the_native_binding(tmp_path, binding):
    """libpab.so alone is enough: without the binding, or with one that does not load, calls take the Python path."""
    import subprocess
    import sys
    code = ("from %s import pab\n"
            "import os, sys; assert pab.__file__.startswith(sys.argv[1])\n"
            "assert pab._binding.attention(0, 0, 0, 0, None, None, None, None) is NotImplemented\n"
            "assert pab._binding.attention_compute(0, None, None, None, None, None) is NotImplemented\n"
            "assert pab.pab_schedule(0, 3, 2, 8, 2) == pab.REUSE\n") % os.path.basename(os.path.dirname(pab.__file__))
    _package_copy(tmp_path, binding)
    res = subprocess.run([sys.executable, "-c", code, str(tmp_path)], cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    assert ("does not load" in res.stderr) == (binding is not None)


def test_library_builds_without_what_the_binding_needs(tmp_path, monkeypatch, capsys):
    """libpab.so needs hipcc only; a binding that cannot be built is said and not an error of its callers.  One that was built for
    another torch or Python does not count as built."""
    from paper_2408_12588_amd import build
    hipcc = tmp_path / "hipcc"
    hipcc.write_text("#!/bin/sh\nwhile [ \"$1\" != -o ]; do shift; done\ntouch \"$2\"\n")
    hipcc.chmod(0o755)
    monkeypatch.setenv("HIPCC", str(hipcc))
    monkeypatch.setenv("CXX", "false")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libpab.so"))
    assert build.build_lib() == build.LIB and os.path.exists(build.LIB)
    assert build.ensure_built() == build.LIB
    assert "binding is not built" in capsys.readouterr().err
    with pytest.raises(RuntimeError):
        build.build_binding()
    assert sorted(os.listdir(tmp_path)) == ["hipcc", "libpab.so"]
    import sysconfig
    here = build.binding_path()
    assert here.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and here != build.binding_path("2.0.0")
