"""CPU-only checks of the C-ABI library: it loads, exports every declared symbol, and its
host-side logic (budgets, compaction plan, argument validation) agrees with the oracle.
No device work is launched here."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import oracle as orc
import paper_2601_04359_amd as pk
from paper_2601_04359_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(binding.lib_path()):
        from paper_2601_04359_amd.build import build_library
        build_library()
    return binding.lib()


def test_every_declared_symbol_is_exported(L):
    with open(os.path.join(ROOT, "include", "packcache.h")) as f:
        header = f.read()
    names = set(re.findall(r"\b(pc_[a-z0-9_]+)\s*\(", header))
    assert {"pc_budget", "pc_rope3d", "pc_rebase", "pc_score", "pc_compact", "pc_frame_attn", "pc_compact_plan",
            "pc_strerror", "pc_last_error_detail", "pc_version", "pc_score_workspace_bytes",
            "pc_compact_workspace_bytes", "pc_frame_attn_workspace_bytes"} <= names
    for n in names:
        assert hasattr(L, n), n
    assert pk.pc_version() >= 100
    assert pk.pc_strerror(0) == "ok" and "NULL" in pk.pc_strerror(-1)


@pytest.mark.parametrize("gamma", [0.5, 0.7, 0.85, 0.95, 1.0, 0.3333333333333333, 1e-3])
@pytest.mark.parametrize("N,n_past,b_min", [(64, 4, 8), (4032, 47, 512), (4032, 23, 0), (4096, 60, 1), (7, 3, 0)])
def test_budget_pow_matches_oracle(L, gamma, N, n_past, b_min):
    assert pk.pc_budget(pk.PC_BUDGET_POW, N, n_past, gamma, b_min) == orc.budget_pow(N, n_past, gamma, b_min)


def test_budget_pow_config_values(L):
    assert pk.pc_budget(pk.PC_BUDGET_POW, 64, 4, 0.7, 8) == [44, 31, 21, 15]
    assert sum(pk.pc_budget(pk.PC_BUDGET_POW, 4032, 47, 0.85, 512)) == 37512
    assert pk.pc_budget(pk.PC_BUDGET_POW, 4096, 12, 0.5, 0) == [4096 >> d for d in range(1, 13)]
    assert pk.pc_budget(pk.PC_BUDGET_POW, 100, 0, 0.5, 0) == []


@pytest.mark.parametrize("rho", [0.5, 0.7, 0.85, 0.95, 1.0])
@pytest.mark.parametrize("w", [1, 2, 3, 12, 47])
@pytest.mark.parametrize("q_min", [0, 100, 512, 3000])
def test_budget_norm_and_half_match_oracle(L, rho, w, q_min):
    assert pk.pc_budget(pk.PC_BUDGET_NORM, 4084, w, rho, q_min) == orc.budget_norm(4084, w, rho, q_min)
    assert pk.pc_budget(pk.PC_BUDGET_HALF, 4084, w, 0.0, q_min) == orc.budget_half(4084, w, q_min)
    assert pk.pc_budget(pk.PC_BUDGET_SLIDE, 4084, w) == orc.budget_slide(4084, w)


def test_budgets_match_oracle_on_random_parameters(L):
    """Exact integer budgets for random decay factors (arbitrary doubles, not only short decimals),
    frame sizes, window lengths and quotas: the library's big-integer arithmetic against the
    oracle's rationals; and the invariants of Eq. 8 (fixed-budget rules add up to B_one)."""
    rng = np.random.default_rng(2024)
    for _ in range(400):
        N, w = int(rng.integers(1, 9000)), int(rng.integers(0, 100))
        gamma = float(rng.choice([rng.uniform(1e-3, 1.0), 1.0, 0.5, rng.uniform(0.9, 1.0)]))
        q = int(rng.choice([0, rng.integers(0, 50), rng.integers(0, N + 1)]))
        assert pk.pc_budget(pk.PC_BUDGET_POW, N, w, gamma, q) == orc.budget_pow(N, w, gamma, q), (N, w, gamma, q)
        norm = pk.pc_budget(pk.PC_BUDGET_NORM, N, w, gamma, q)
        half = pk.pc_budget(pk.PC_BUDGET_HALF, N, w, 0.0, q)
        assert norm == orc.budget_norm(N, w, gamma, q), (N, w, gamma, q)
        assert half == orc.budget_half(N, w, q), (N, w, q)
        if w > 0:
            assert sum(norm) == N and sum(half) == N
            assert all(a >= b for a, b in zip(norm, norm[1:])) and all(a >= b for a, b in zip(half, half[1:]))


def test_budget_half_series_from_the_paper(L):
    assert pk.pc_budget(pk.PC_BUDGET_HALF, 4096, 4) == [2048, 1024, 512, 512]
    assert pk.pc_budget(pk.PC_BUDGET_HALF, 4096, 1) == [4096]


def test_budget_errors(L):
    for args in [(9, 10, 2, 0.5, 0), (0, -1, 2, 0.5, 0), (0, 10, -2, 0.5, 0), (0, 10, 2, 0.0, 0),
                 (0, 10, 2, 1.5, 0), (1, 10, 2, -0.1, 0), (0, 10, 2, 0.5, -1)]:
        with pytest.raises(pk.PackCacheError) as e:
            pk.pc_budget(*args)
        assert e.value.status == -5
    assert L.pc_budget(0, 10, 2, 0.5, 0, None) == -1
    assert b"budget_out" in L.pc_last_error_detail()


def test_compact_plan_matches_oracle(L):
    w = synth.config1()
    b = pk.pc_budget(pk.PC_BUDGET_POW, w.n_frame, w.n_past, w.gamma, w.b_min)
    budgets = pk.segment_budgets(w.segments, b)
    assert budgets == [16, 64, 15, 21, 31, 44]
    segs, nk = pk.pc_compact_plan(w.segments, budgets)
    assert segs == orc.packed_segments(w.segments, budgets) and nk == 191
    # budget above the segment length is clamped, zero budget empties the segment
    segs, nk = pk.pc_compact_plan(w.segments, [0, 0, 1000, 0, 5, 64])
    assert [s[1] for s in segs] == [16, 64, 64, 0, 5, 64] and nk == 213


def test_compact_plan_errors(L):
    with pytest.raises(pk.PackCacheError) as e:
        pk.pc_compact_plan([(0, 4, 0, 0), (5, 4, 2, 1)], [4, 4])        # gap in the table
    assert e.value.status == -2
    with pytest.raises(pk.PackCacheError) as e:
        pk.pc_compact_plan([(0, 4, 2, 0)], [-1])
    assert e.value.status == -5
    with pytest.raises(pk.PackCacheError) as e:
        pk.pc_compact_plan([(0, 4, 7, 0)], [1])                          # unknown kind
    assert e.value.status == -2


def test_argument_validation_returns_before_any_device_work(L):
    one = C.c_void_p(16)   # non-NULL dummy; every call below must fail before touching it
    # dtype
    assert L.pc_frame_attn(one, one, one, 5, 2, 1, 4, 4, 128, 512, 512, 512, 0.1, one, None, None, 0, None) == -3
    # Hq not a multiple of Hkv
    assert L.pc_frame_attn(one, one, one, 1, 3, 2, 4, 4, 128, 512, 512, 512, 0.1, one, None, None, 0, None) == -2
    # empty key set
    assert L.pc_frame_attn(one, one, one, 1, 2, 1, 4, 0, 128, 512, 512, 512, 0.1, one, None, None, 0, None) == -2
    # NULL tensor
    assert L.pc_frame_attn(None, one, one, 1, 2, 1, 4, 4, 128, 512, 512, 512, 0.1, one, None, None, 0, None) == -1
    # bf16 tier is D = 128 only
    assert L.pc_frame_attn(one, one, one, 1, 2, 1, 4, 4, 64, 256, 256, 256, 0.1, one, None, None, 0, None) == -4
    # stride too small
    assert L.pc_frame_attn(one, one, one, 1, 2, 1, 4, 4, 128, 8, 512, 512, 0.1, one, None, None, 0, None) == -2
    # rope: sections must add up to D
    assert L.pc_rope3d(one, 1, 1, 4, 128, 512, one, 32, 48, 40, 1e4, 1.0, None) == -2
    assert L.pc_rope3d(one, 1, 1, 4, 128, 512, one, 32, 48, 48, 1e4, 0.0, None) == -2      # out_scale must be > 0
    assert L.pc_rope3d(None, 1, 1, 4, 128, 512, one, 32, 48, 48, 1e4, 1.0, None) == -1
    # rebase: sections must add up to D; a temporal section that is not whole 16-byte chunks; NULL
    assert L.pc_rebase(one, 1, 1, 128, 512, one, 1, 12, 0, 4, 4, 32, 48, 40, 1e4, None) == -2
    assert L.pc_rebase(one, 1, 1, 128, 512, one, 1, 12, 0, 4, 4, 20, 60, 48, 1e4, None) == -4
    assert L.pc_rebase(None, 1, 1, 128, 512, one, 1, 12, 0, 4, 4, 32, 48, 48, 1e4, None) == -1
    assert L.pc_rebase(one, 1, 1, 128, 512, one, 2, 12, 0, 4, 4, 32, 48, 48, 1e4, None) == -2   # Hsel > Hkv
    assert L.pc_rebase(None, 1, 1, 128, 512, None, 1, 12, 0, 0, 4, 32, 48, 48, 1e4, None) == 0   # nothing to do
    # score: workspace missing / too small
    need = L.pc_score_workspace_bytes(4, 2, 8, 100, 0)
    assert need > 0
    assert L.pc_score(one, one, 1, 4, 2, 8, 100, 128, 1024, 12800, None, 0.1, None, 0, one, 100, 0, 0, 0, None, 0, None) == -6
    assert L.pc_score(one, one, 1, 4, 2, 8, 100, 128, 1024, 12800, None, 0.1, None, 0, one, 100, 0, 0, 0, one, need - 1, None) == -6
    # key range: empty, reversed or past the end
    for kb, ke in ((5, 5), (7, 3), (0, 101), (-1, 10), (100, 0)):
        assert L.pc_score(one, one, 1, 4, 2, 8, 100, 128, 1024, 12800, None, 0.1, None, 0, one, 100, 0, kb, ke, one, need, None) == -2
    # compact: too many segments; partial aliasing of outputs
    seg = (binding.pc_segment * 2)(binding.pc_segment(0, 4, 0, 0), binding.pc_segment(4, 8, 2, 1))
    bud = (C.c_int32 * 2)(4, 3)
    assert L.pc_compact(one, one, one, 1, 1, 128, 4096, 0, one, 0, seg, 500, bud, 0, one, one, one, 4096, 0,
                        None, 0, None, None, one, 1 << 20, None) == -2
    two = C.c_void_p(4096)
    assert L.pc_compact(one, one, one, 1, 1, 128, 4096, 36, one, 12, seg, 2, bud, 0, one, two, one, 4096, 36,
                        None, 0, None, None, one, 1 << 20, None) == -2
    assert b"alias" in L.pc_last_error_detail()


def test_binding_raises_without_library(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_LIB", None)
    monkeypatch.setattr(binding, "lib_path", lambda: str(tmp_path / "libpackcache.so"))
    with pytest.raises(FileNotFoundError):
        binding.pc_version()


def test_table_helpers_agree_with_their_fallbacks(L, monkeypatch):
    """What RollingLayer and RollingStack score and move, from the compiled half and without it."""
    import torch  # noqa: F401
    if binding._NATIVE is None:
        binding._bind_native(L)
    native, rng = binding._NATIVE, np.random.default_rng(12)
    assert native
    T, C0, F, S = pk.PC_SEG_TEXT, pk.PC_SEG_COND, pk.PC_SEG_FRAME, pk.PC_SEG_SELF

    def both(f, *args):
        got = []
        for half in (native, False):
            monkeypatch.setattr(binding, "_NATIVE", half)
            try:
                got.append(f(*args))
            except (IndexError, TypeError) as e:
                got.append(type(e))
        assert got[0] == got[1], (f.__name__, args, got)
        return got[0]

    for trial in range(300):
        kinds = [int(k) for k in rng.choice([T, C0, F, F, F, S], int(rng.integers(0, 9)))]     # anchors behind frames too
        lens = [int(rng.choice([0, 1, 5, 40])) for _ in kinds]                                 # zero-length frames
        segs = [(sum(lens[:i]), n, k, i) for i, (n, k) in enumerate(zip(lens, kinds))]
        n_frames = both(binding._past_frames, segs)
        assert n_frames == kinds.count(F)
        by = [int(b) for b in rng.integers(0, 41, n_frames)]
        budgets = both(pk.segment_budgets, segs, by)
        both(pk.segment_budgets, [list(s) for s in segs], tuple(by) + (3,))
        if n_frames:
            assert both(pk.segment_budgets, segs, by[:-1]) is IndexError
        over = [i for i, s in enumerate(segs) if s[2] == F and budgets[i] < s[1]]
        want = (segs[over[0]][0], segs[over[-1]][0] + segs[over[-1]][1]) if over else None
        assert both(binding._prunable_span, segs, budgets) == want
        assert both(binding._prunable_span, segs, [s[1] for s in segs]) is None        # none is over its budget
        both(binding._prunable_span, segs, budgets[:-1])
    both(pk.segment_budgets, [(0, np.int64(4), np.int32(F), 0)], [np.int32(2)])          # not built-in: converted
    both(pk.segment_budgets, [(0, 4, F, 0)], [True])


@pytest.mark.parametrize("other", [dict(torch_version="0.0"), dict(pc_version=-1)])
def test_compiled_half_of_another_build_is_not_bound(L, monkeypatch, other):
    import torch  # noqa: F401
    from paper_2601_04359_amd import _marshal
    monkeypatch.setattr(binding, "_NATIVE", None)
    for name, value in other.items():
        monkeypatch.setattr(_marshal, name, value)
    with pytest.warns(UserWarning, match="built for"):
        binding._bind_native(L)
    assert binding._NATIVE is False
    monkeypatch.undo()
    binding._bind_native(L)
    assert binding._NATIVE is _marshal


def test_library_builds_where_the_compiled_half_cannot(monkeypatch, tmp_path):
    from paper_2601_04359_amd import build
    commands = []

    def run(cmd):
        commands.append(cmd[0])
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
        return ""

    for name in ("PKG", "LIB_DIR"):
        monkeypatch.setattr(build, name, str(tmp_path))
    monkeypatch.setattr(build, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    (tmp_path / "_marshal.so").write_bytes(b"an older build's")
    monkeypatch.setattr(build, "_run", run)
    with pytest.warns(UserWarning, match="not built"):
        assert build.build_library() == build.LIB_PATH
    assert len(commands) == len(build.SOURCES) + 2 and not (tmp_path / "_marshal.so").exists()


def test_masked_budgets_match_the_oracle():
    w = synth.midsize()
    rng = np.random.default_rng(0)
    valid = (rng.random(w.Nk) < 0.3).astype(np.uint8)
    for gamma, b_min in ((0.85, 32), (0.5, 0), (1.0, 0)):
        budgets = pk.segment_budgets(w.segments, orc.budget_pow(w.n_frame, w.n_past, gamma, b_min))
        assert pk.pc_masked_budgets(w.segments, budgets, valid) == orc.masked_budgets(w.segments, budgets, valid)
    with pytest.raises(pk.PackCacheError):
        pk.pc_masked_budgets(w.segments, [-1] * len(w.segments), valid)


def test_batched_compaction_and_mask_argument_checks(L):
    one, two = C.c_void_p(4096), C.c_void_p(8192)
    seg = (binding.pc_segment * 2)(binding.pc_segment(0, 4, 0, 0), binding.pc_segment(4, 8, 2, 1))
    bud = (C.c_int32 * 2)(4, 3)
    ws = L.pc_compact_batch_workspace_bytes(3, 2, 12, 0)
    assert ws >= L.pc_compact_workspace_bytes(2, 12, 0) > 0
    assert L.pc_compact_batch_workspace_bytes(0, 2, 12, 0) == 0

    def call(n_layers, kv_l, pos_l, sc_l, in_place=True, hkv=2):
        Ko = one if in_place else two
        return L.pc_compact_batch(n_layers, one, one, one, 1, hkv, 128, 12 * 128, kv_l, 36, pos_l, one, 12, sc_l,
                                  seg, 2, bud, 0, Ko, Ko, Ko, 12 * 128, kv_l, 36, pos_l, None, 0, 0, None, None,
                                  one, 1 << 24, None)
    # a layer stride smaller than one layer of K / pos / score
    assert call(3, 2 * 12 * 128 - 8, 72, 24) == -2
    assert call(3, 2 * 12 * 128, 71, 24) == -2
    assert call(3, 2 * 12 * 128, 72, 23) == -2
    # zero layers; too many (layer, head) pairs for the in-place tickets
    assert call(0, 0, 0, 0) == -2
    assert call(129, 2 * 12 * 128, 72, 24) == -4
    assert b"pairs" in L.pc_last_error_detail()
    # mask: NULL pointers, short stride; empty input is fine
    assert L.pc_mask_scores(None, 2, 10, 10, one, None) == -1
    assert L.pc_mask_scores(one, 2, 10, 9, one, None) == -2
    assert L.pc_mask_scores(None, 0, 10, 10, None, None) == 0
    assert L.pc_masked_budgets(seg, 2, bud, None, bud) == -1
    # status of a workspace that does not exist
    assert L.pc_compact_status(None, None) == -1
    assert L.pc_strerror(-8) not in (None, L.pc_strerror(-7))


def test_static_scratch_entry_rejects_oversized_requests_before_any_device_work(L):
    # pc_compact_static: the request is sized on the host and refused before the device is touched
    assert L.pc_compact_static_capacity() == 4 << 20
    assert L.pc_compact_workspace_bytes(4, 193_792, 0) <= L.pc_compact_static_capacity()
    one = C.c_void_p(4096)
    n = 400_000
    assert L.pc_compact_workspace_bytes(8, n, 0) > L.pc_compact_static_capacity()
    seg = (binding.pc_segment * 1)(binding.pc_segment(0, n, 1, 0))
    bud = (C.c_int32 * 1)(n)
    rc = L.pc_compact_static(one, one, one, 1, 8, 128, n * 128, n * 3, one, n, seg, 1, bud, 0, one, one, one,
                             n * 128, n * 3, None, 0, None, None, None)
    assert rc == -6 and b"scratch" in L.pc_last_error_detail()
    # malformed table: refused as a shape error, also before any device work
    assert L.pc_compact_static(one, one, one, 1, 0, 128, 0, 0, one, 0, seg, 1, bud, 0, one, one, one, 0, 0, None,
                               0, None, None, None) == -2


def test_fold_helpers_are_the_constants_the_header_names():
    import math
    assert pk.PC_SCALE_FOLDED == math.log(2.0)
    # what the kernels test for: float(ln 2) * float(log2 e), rounded to fp32, is exactly 1
    assert C.c_float(C.c_float(pk.PC_SCALE_FOLDED).value * C.c_float(1.4426950408889634).value).value == 1.0
    for s in (128 ** -0.5, 64 ** -0.5, 0.3):
        assert abs(pk.folded_q_scale(s) - s / math.log(2.0)) <= 1e-15 * s
    src = open(os.path.join(ROOT, "include", "packcache.h")).read()
    assert "#define PC_SCALE_FOLDED 0.693147180559945309f" in src


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert p.returncode != 0 and "ONE GPU" in p.stderr and p.stdout.strip() == ""


def test_tables_marshal_the_same_from_any_kind_of_number():
    # plain and numpy integers are packed in one pass, everything else is converted one by one
    plain = [(0, 4, pk.PC_SEG_TEXT, -1), (4, 9, pk.PC_SEG_COND, 0), (13, 9, pk.PC_SEG_FRAME, 1)]
    want = pk.pc_compact_plan(plain, [4, 9, 5])
    assert want == ([(0, 4, pk.PC_SEG_TEXT, -1), (4, 9, pk.PC_SEG_COND, 0), (13, 5, pk.PC_SEG_FRAME, 1)], 18)
    for conv in (lambda v: v, np.int64, np.int32, float, np.float64):
        segs = [tuple(conv(v) for v in s) for s in plain]
        assert pk.pc_compact_plan(segs, [conv(4), conv(9), conv(5)]) == want
        assert pk.pc_compact_plan([list(s) for s in segs], (conv(4), conv(9), conv(5))) == want
    assert pk.pc_compact_plan([(0, 4, pk.PC_SEG_TEXT)], [4]) == ([(0, 4, pk.PC_SEG_TEXT, 0)], 4)   # frame left out
    assert pk.pc_compact_plan([], []) == ([], 0)


@pytest.mark.parametrize("gamma", [0.5, 1.0, 0.25, 0.75, 0.85, 1 - 2.0 ** -53, float(np.nextafter(0.5, 1)), 2.0 ** -40, 5e-324])
def test_budgets_are_exact_next_to_whole_numbers(gamma):
    # products that are whole numbers, or miss one by less than extended precision resolves, settle exactly
    from fractions import Fraction
    g = Fraction(gamma)
    for n in (1, 7, 64, 4032, 4096, 2 ** 31 - 1):
        for n_past in (1, 6, 47):
            want = [min(n, max(3, int(n * g ** d))) for d in range(1, n_past + 1)]
            assert pk.pc_budget(pk.PC_BUDGET_POW, n, n_past, gamma, 3) == want
            for mode, w in ((pk.PC_BUDGET_NORM, lambda d: g ** d / sum(g ** j for j in range(1, n_past + 1))),
                            (pk.PC_BUDGET_HALF, lambda d: Fraction(1, 2 ** min(d, n_past - 1)))):
                want = [int(n * w(d)) for d in range(1, n_past + 1)]
                want[0] += n - sum(want)
                assert pk.pc_budget(mode, n, n_past, gamma, 0) == want


def test_tables_may_be_tensors_and_iterators():
    import torch
    plain = [(0, 4, pk.PC_SEG_TEXT, -1), (4, 9, pk.PC_SEG_COND, 0), (13, 9, pk.PC_SEG_FRAME, 1)]
    budgets = [4, 9, 5]
    want = pk.pc_compact_plan(plain, budgets)
    for make in (iter, lambda b: map(int, b), lambda b: (v for v in b), np.array, torch.tensor,
                 lambda b: torch.tensor(b, dtype=torch.float32), lambda b: torch.tensor(b, dtype=torch.uint8),
                 lambda b: [torch.tensor(float(v)) for v in b], lambda b: [str(v) for v in b], dict.fromkeys):
        assert pk.pc_compact_plan(plain, make(budgets)) == want
        assert pk.pc_masked_budgets(plain, make(budgets), np.ones(22, np.uint8)) == budgets
    for make in (lambda t: [iter(s) for s in t], lambda t: [map(int, s) for s in t], np.array, torch.tensor,
                 lambda t: torch.tensor(t, dtype=torch.float64), lambda t: list(torch.tensor(t, dtype=torch.float32)),
                 lambda t: [[torch.tensor(float(v)) for v in s] for s in t]):
        assert pk.pc_compact_plan(make(plain), budgets) == want
    for bad in (5, None, [4, 9, None], [4, 9, "x"], [4, 9, 5, 6]):     # refused before as now
        with pytest.raises((TypeError, ValueError, IndexError)):
            pk.pc_compact_plan(plain, bad)


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_query_falls_back_to_the_public_one(monkeypatch, missing):
    import types
    import torch
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4711))
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 12, raising=False)
    assert binding._stream() == 12
    monkeypatch.delattr(torch._C, missing)
    assert binding._stream() == 4711


def test_attention_asks_for_no_workspace_it_would_not_use(monkeypatch):
    import torch
    # full caches of frames 24 and 48, 16/4 heads: 252 row tiles fill the chip, nothing is cut in either dtype
    for nk in (97024, 193792):
        assert pk.pc_frame_attn_workspace_bytes(16, 4032, nk, 128) == 0
    # 24/8 heads: 384 row tiles, the 128 behind the first round in two shares of 512 + 8 bytes a row
    assert pk.pc_frame_attn_workspace_bytes_for(pk.PC_BF16, 24, 8, 4032, 8320, 128) <= 2 * 128 * 256 * 520 + 512
    # one query covers every dtype and number of KV heads
    rng = np.random.default_rng(1)
    for _ in range(200):
        hq, nq, nk = int(rng.choice([2, 6, 8, 16, 24])), int(rng.integers(1, 4100)), int(rng.integers(1, 60000))
        d = int(rng.choice([64, 128]))
        every = [pk.pc_frame_attn_workspace_bytes_for(t, hq, hkv, nq, nk, d) for t in (pk.PC_F32, pk.PC_BF16)
                 for hkv in range(1, hq + 1)]
        assert pk.pc_frame_attn_workspace_bytes(hq, nq, nk, d) == max(every)
    for bad in ((pk.PC_BF16, 3, 2, 10, 10, 128), (pk.PC_BF16, 2, 0, 10, 10, 128), (pk.PC_BF16, 2, 1, 10, 10, 64),
                (pk.PC_F32, 2, 1, 0, 10, 64), (pk.PC_F32, 2, 1, 10, 10, 96), (7, 2, 1, 10, 10, 128)):
        assert pk.pc_frame_attn_workspace_bytes_for(*bad) == 0
    # and a call without a workspace takes one of its own dtype's and head count's size
    class Enough(Exception):
        pass
    def stop():
        raise Enough
    taken = []
    monkeypatch.setattr(binding, "_workspace", lambda n, like: taken.append(n) or torch.empty(16, dtype=torch.uint8))
    monkeypatch.setattr(binding, "_stream", stop)      # the last thing before the library call
    for dtype, code in ((torch.float32, pk.PC_F32), (torch.bfloat16, pk.PC_BF16)):
        for hq, hkv, nq, nk in ((16, 4, 4032, 193792), (8, 2, 252, 1179), (24, 8, 2901, 2100)):
            Q, K, V = (torch.empty((h, n, 128), dtype=dtype, device="meta") for h, n in ((hq, nq), (hkv, nk), (hkv, nk)))
            taken.clear()
            with pytest.raises(Enough):
                pk.pc_frame_attn(Q, K, V, nk, 0.1)
            need = pk.pc_frame_attn_workspace_bytes_for(code, hq, hkv, nq, nk, 128)
            assert taken == ([need] if need else [])


def test_rolling_caches_give_every_attention_call_its_own_workspace(monkeypatch):
    import torch
    from paper_2601_04359_amd import rollout
    taken = []
    monkeypatch.setattr(rollout.pk, "pc_frame_attn", lambda *a, ws=None, **kw: taken.append(ws))
    kw = dict(capacity=600, n_frame=252, scale=0.1, device="cpu")
    layer, stack = rollout.RollingLayer(8, 2, 128, **kw), rollout.RollingStack(2, 8, 2, 128, **kw)
    Q = torch.empty((8, 252, 128), dtype=torch.bfloat16)
    for _ in range(2):
        layer.attend(Q)
        stack.attend(0, Q)
        stack.attend(1, Q)
    given = [w.data_ptr() for w in taken if w is not None]
    assert len(taken) == 6 and len(set(given)) == len(given)


def test_parity_shapes_take_the_forms_they_are_meant_for(L):
    """Which kernel form and how many shares the shapes of test_gpu_parity.py take, so that a change of the
    estimates does not move them off what their tests say they cover."""
    import test_gpu_parity as g
    ample, ln2 = 1 << 40, pk.PC_SCALE_FOLDED
    attn = lambda shape, ws=ample: pk.pc_frame_attn_cut(pk.PC_BF16, *shape, 128, ws)
    cuts = [attn(s) for s in g.ATTN_ACROSS_HEADS]
    assert cuts[:4] == [(32, 1, 0)] * 4 and cuts[4][0] == 32 and cuts[4][1] > 1
    assert all(c[0] == 256 and c[1] > 1 for c in cuts[5:]) and [c[2] for c in cuts[5:]] == [0, 0, 256]
    assert all(attn(s, 0) == (256, 1, 0) for s in g.ATTN_256_ROWS_UNCUT)
    # 32 rows with divided output dims (128 work-groups at most) and undivided ones
    assert all(s[1] * -(-(s[0] // s[1] * s[2]) // 32) * c[1] <= 128 for s, c in zip(g.ATTN_ACROSS_HEADS[:5], cuts))
    for *shape, shares in g.ATTN_32_ROWS_WHOLE:
        assert attn(shape) == (32, shares, 0) and shape[1] * -(-(shape[0] // shape[1] * shape[2]) // 32) * shares > 128
    # masked keys: 32 rows in two and ten shares, 256 un-split and in four shares of 1,920 keys, fp32 with 16 and 32
    assert attn((8, 2, 252, 1804)) == (32, 2, 0)
    assert attn((2, 1, 184, 5000))[:2] == (32, 10) and attn((16, 4, 4032, 2048)) == (256, 1, 0)
    assert attn((16, 4, 1008, 7455)) == (256, 4, 0)
    f32 = lambda shape, d: pk.pc_frame_attn_cut(pk.PC_F32, *shape, d, ample)
    assert f32((2, 1, 64, 336), 64)[0] == 16 and f32((8, 2, 252, 1804), 128)[0] == 32
    assert f32((3, 1, 301, 2501), 64)[0] == 16 and f32((3, 1, 301, 2501), 128)[0] == 32
    assert f32((3, 1, 17, 5000), 64)[1] > 1 and f32((3, 1, 16, 32), 64) == (16, 1, 0)
    score = lambda shape, scale=0.088, lse=False: pk.pc_score_cut(*shape, scale, lse)
    for scale in (0.088, ln2):
        cuts = [score(s, scale) for s in g.SCORE_ACROSS_HEADS]
        assert all((c[0], c[2]) == (64, 64) for c in cuts[:3])
        assert [(c[0], c[2], c[4]) for c in cuts[3:5]] == [(64, 512, 1), (64, 512, 0)]
        assert all((c[0], c[2]) == (512, 512) for c in cuts[5:])
        per_share = [-(-(-(-s[3] // 64)) // score(s, scale)[1]) for s in g.SCORE_512_FEW_KEYS]
        assert all(score(s, scale)[0] == 512 for s in g.SCORE_512_FEW_KEYS) and {1, 2, 3} <= set(per_share)
        for s in g.SCORE_512_FEW_ROWS:
            assert score(s, scale)[2:4] == (512, 1) and score(s, scale, True)[:4] == (0, 0, 512, 1)


def test_many_rows_over_few_keys_take_256_rows():
    # more than one round of 128-row tiles: 256 rows per work-group were timed 1.03 to 1.4 times as fast
    for shape in ((16, 4, 5311, 4), (28, 4, 7066, 10), (16, 16, 13805, 25), (2, 1, 35636, 42), (16, 4, 9892, 63),
                  (3, 1, 23314, 130), (28, 4, 5607, 153), (16, 4, 5936, 347), (4, 2, 21761, 465), (3, 1, 28705, 776)):
        assert pk.pc_frame_attn_cut(pk.PC_BF16, *shape, 128, 1 << 40)[0] == 256, shape
    # the last tile that is one round, and one more
    assert pk.pc_frame_attn_cut(pk.PC_BF16, 16, 4, 64 * 32, 700, 128, 0)[0] == 128
    assert pk.pc_frame_attn_cut(pk.PC_BF16, 16, 4, 64 * 32 + 1, 700, 128, 0)[0] != 128


def test_few_rows_over_many_keys_take_32_rows():
    # 64 rows per work-group in key shares were timed 1.07 to 1.19 times as long
    for shape in ((2, 1, 2527, 2601), (2, 1, 696, 6694), (1, 1, 1636, 6521), (1, 1, 1709, 6735), (8, 1, 219, 8147),
                  (2, 1, 1292, 6516), (8, 1, 411, 4214), (1, 1, 3140, 3092)):
        assert pk.pc_frame_attn_cut(pk.PC_BF16, *shape, 128, 1 << 40)[0] == 32, shape
    assert pk.pc_frame_attn_cut(pk.PC_BF16, 8, 1, 779, 5759, 128, 1 << 40)[0] != 128


def test_small_compactions_take_the_form_that_was_faster():
    import test_gpu_parity as g
    for lens, D, dtype, Hkv, share, launches in g.COMPACT_SMALL:
        segs, _, budgets = g.small_table(lens)
        for in_place in (False, True):
            cut = pk.pc_compact_cut(1, Hkv, pk.PC_BF16 if dtype == "bf16" else pk.PC_F32, D, segs, budgets, share, in_place)
            assert cut[0] == launches[in_place], (lens, Hkv, in_place)

    def cut(layers, Hkv, lens, keep, in_place, wide=False, share=False):
        segs = [(sum(lens[:i]), n, pk.PC_SEG_FRAME, i) for i, n in enumerate(lens)]
        return pk.pc_compact_cut(layers, Hkv, pk.PC_F32 if wide else pk.PC_BF16, 128, segs, keep, share, in_place)

    # timed in both forms, and with every number of slices: the faster of them is taken
    assert cut(1, 8, [600] + [221] * 12, [237] + [140] * 12, True) == (1, 2)        # 64-byte slices: 13.6 us, two launches 9.6
    assert cut(1, 8, [300] * 3, [150] * 3, False) == (1, 4) and cut(1, 4, [300] * 3, [150] * 3, True) == (1, 4)
    assert cut(4, 8, [300] * 3, [150] * 3, True) == (1, 2) and cut(7, 8, [300] * 3, [150] * 3, True) == (1, 1)
    assert cut(1, 2, [17] * 28, [10] * 28, False)[0] == 2 and cut(1, 2, [17] * 28, [10] * 28, True)[0] == 1
    assert cut(1, 2, [17] * 28, [17] * 20 + [10] * 8, False)[0] == 1
    assert cut(28, 8, [60, 40], [60, 31], True)[0] == 2 and cut(28, 8, [280, 17], [280, 9], True)[0] == 1
    # no launch, what is refused, and what the call itself refuses
    assert cut(1, 2, [40, 50], [0, 0], True) == (0, 0) and cut(1, 2, [], [], True) == (0, 0)
    for bad in (lambda: cut(0, 2, [40], [4], True), lambda: cut(1, 0, [40], [4], True), lambda: cut(257, 1, [40], [4], True),
                lambda: cut(1, 2, [40], [-1], True), lambda: pk.pc_compact_cut(1, 2, 7, 128, [(0, 4, 2, 0)], [2]),
                lambda: pk.pc_compact_cut(1, 2, pk.PC_BF16, 96, [(0, 4, 2, 0)], [2])):
        with pytest.raises(pk.PackCacheError):
            bad()
    assert cut(1 << 20, 1 << 15, [40], [4], False) == (2, 0)


def test_column_pass_takes_the_form_that_was_faster():
    # keys per work-group of the column pass where the two forms were timed 5 % or more apart, log-sum-exps given
    for shape, keys in (((16, 4, 512, 40), 512), ((16, 4, 512, 178), 512), ((16, 4, 512, 1305), 512), ((8, 2, 512, 2551), 512),
                        ((2, 1, 1000, 2948), 512), ((8, 2, 170, 11032), 512), ((16, 4, 100, 6000), 512), ((16, 4, 512, 13810), 512),
                        ((16, 4, 64, 2392), 64), ((16, 4, 100, 2516), 64), ((8, 2, 170, 578), 64), ((8, 2, 330, 108), 64)):
        assert pk.pc_score_cut(*shape, 0.088, True)[2] == keys, shape


def test_cut_queries_refuse_what_the_calls_refuse(L):
    for bad in ((pk.PC_BF16, 3, 2, 10, 10, 128), (pk.PC_BF16, 2, 1, 0, 10, 128), (pk.PC_BF16, 2, 1, 10, 10, 64), (5, 2, 1, 10, 10, 128)):
        with pytest.raises(pk.PackCacheError):
            pk.pc_frame_attn_cut(*bad, 0)
    for bad in ((3, 2, 10, 10), (2, 1, 0, 10), (2, 1, 10, 0)):
        with pytest.raises(pk.PackCacheError):
            pk.pc_score_cut(*bad, 0.1)
    assert L.pc_frame_attn_cut(pk.PC_BF16, 2, 1, 10, 10, 128, 0, None) == -1 and L.pc_score_cut(2, 1, 10, 10, 10, 0.1, 0, None) == -1
