"""GPU parity: every C-ABI call against the fp64 oracle on the same seeded inputs.

Tolerances
  * indices, moved rows, positions, segment tables: bit-exact; selected sets may differ
    from the oracle's only on keys whose oracle score is within 1e-6 of the k-th score;
  * bf16 attention (bf16 inputs, fp32 accumulation): max |err| <= 2e-2, mean |err| <= 2e-3;
  * fp32 tier: max |err| <= 1e-5 on outputs of O(1);
  * bf16 RoPE: one bf16 rounding of the fp32 rotation, |err| <= 2^-8 |x| + 1e-6.
"""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2601_04359_amd as pk
from paper_2601_04359_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BAND = 1e-6


def dev(x, dtype):
    t = torch.from_numpy(np.ascontiguousarray(x))
    if dtype == "bf16":
        return t.to(torch.bfloat16).to(DEV)
    return t.to(DEV)


def host(t):
    return t.detach().to(torch.float32).cpu().numpy() if t.is_floating_point() else t.detach().cpu().numpy()


def budgets_for(w, gamma=None, b_min=None):
    b = pk.pc_budget(pk.PC_BUDGET_POW, w.n_frame, w.n_past, w.gamma if gamma is None else gamma,
                     w.b_min if b_min is None else b_min)
    assert b == orc.budget_pow(w.n_frame, w.n_past, w.gamma if gamma is None else gamma,
                               w.b_min if b_min is None else b_min)
    return pk.segment_budgets(w.segments, b)


# The folded-scale form, written out here rather than taken from the package: queries carry
# scale * log2(e) = scale / ln 2 and the calls get ln 2 as their scale.
LN2 = float(np.log(2.0))


def q_fold(scale: float) -> float:
    return float(scale) / LN2


def check_selection(idx_gpu, sc_oracle, segments, budgets, band=BAND, other_input=None):
    """idx_gpu [Hsel][Nk_out] int; sc_oracle [Hsel][Nk] fp64.  Returns #exempted keys.
    other_input [Hsel][Nk] bool marks keys whose device input bits differ from the oracle's
    (a rotation that rounded the other way): their scores are not comparable."""
    exempted = 0
    plan = orc.packed_segments(segments, budgets)
    for h in range(sc_oracle.shape[0]):
        for (start, length, kind, _), (ps, pl, _, _) in zip(segments, plan):
            got = idx_gpu[h, ps:ps + pl].astype(np.int64)
            assert np.all(np.diff(got) > 0), "indices must be strictly ascending"
            assert got.size == 0 or (got[0] >= start and got[-1] < start + length)
            if kind != orc.SEG_FRAME or pl == length:
                assert np.array_equal(got, np.arange(start, start + length))
                continue
            if pl == 0:
                continue
            seg = sc_oracle[h, start:start + length]
            want = start + orc.select_topk(seg, pl)
            if np.array_equal(got, want):
                continue
            thr = np.sort(seg)[::-1][pl - 1]
            diff = np.setxor1d(got, want)
            ok = np.abs(seg[diff - start] - thr) <= band
            if other_input is not None:
                ok |= other_input[h, diff]
            assert np.all(ok), f"head {h} segment at {start}: selection differs outside the {band} band"
            exempted += diff.size
    return exempted


# ------------------------------------------------------------------------------- RoPE
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,H", [(1, 1), (37, 3), (252, 8), (1000, 2)])
def test_rope3d_parity(dtype, n, H):
    rng = np.random.default_rng(n * 31 + H)
    x = rng.standard_normal((H, n, 128)).astype(np.float32)
    if dtype == "bf16":
        x = synth.to_bf16(x)
    pos = np.stack([rng.integers(0, 450, n), rng.integers(0, 380, n), rng.integers(0, 670, n)], 1).astype(np.int32)
    want = orc.rope3d(x, pos, (32, 48, 48), 1e4)
    xd = dev(x, dtype)
    pk.pc_rope3d(xd, dev(pos, None), (32, 48, 48), 1e4)
    got = host(xd).astype(np.float64)
    err = np.abs(got - want)
    if dtype == "bf16":
        assert np.all(err <= 2.0 ** -8 * np.abs(want) + 1e-6)
        # the result is the correctly rounded bf16 of the exact rotation almost everywhere
        assert np.mean(got == orc.round_to_bf16(want)) > 0.999
    else:
        assert err.max() <= 2e-6


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rope3d_out_scale_is_applied_before_the_one_rounding(dtype):
    rng = np.random.default_rng(12)
    x = rng.standard_normal((3, 300, 128)).astype(np.float32)
    if dtype == "bf16":
        x = synth.to_bf16(x)
    pos = np.stack([rng.integers(0, 450, 300), rng.integers(0, 380, 300), rng.integers(0, 670, 300)], 1).astype(np.int32)
    s = q_fold(128 ** -0.5)
    want = orc.rope3d(x, pos, (32, 48, 48), 1e4) * s
    xd = dev(x, dtype)
    pk.pc_rope3d(xd, dev(pos, None), (32, 48, 48), 1e4, out_scale=s)
    got = host(xd).astype(np.float64)
    tol = 2.0 ** -8 if dtype == "bf16" else 2e-6
    assert np.all(np.abs(got - want) <= tol * np.abs(want) + 1e-6 * s)
    if dtype == "bf16":     # one rounding, not two: most elements are the nearest bf16 of the exact value
        assert (got == orc.round_to_bf16(want)).mean() > 0.99


# the whole range of the reduction: positions at both ends of int32, frequencies above one (base 0.5,
# angles beyond 2^32); tokens and heads that are no multiple of a work-group's
@pytest.mark.parametrize("base", [1e4, 0.5])
@pytest.mark.parametrize("n,H,sections", [(3, 1, (16, 24, 24)), (5, 5, (32, 48, 48)), (4, 9, (64, 0, 64))])
def test_rope3d_extreme_positions(n, H, sections, base):
    rng = np.random.default_rng(n + H)
    d = sum(sections)
    x = rng.standard_normal((H, n, d)).astype(np.float32)
    pos = rng.integers(-2 ** 31, 2 ** 31, (n, 3)).astype(np.int32)
    pos[0], pos[1], pos[2] = -2 ** 31, 2 ** 31 - 1, (0, 1, -1)
    xd = dev(x, None)
    pk.pc_rope3d(xd, dev(pos, None), sections, base)
    # frequencies of the two sides may differ in the last bit: 2^32 * 2^-52 radians, next to fp32's rounding
    assert np.abs(host(xd) - orc.rope3d(x, pos, sections, base)).max() <= 4e-6


# few tokens of many heads: the heads dealt over several work-groups per token block, the last one part-filled
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,n,sections", [(224, 3, (32, 48, 48)), (113, 64, (32, 48, 48)), (67, 1, (64, 96, 96)),
                                          (33, 30, (32, 32, 32)), (41, 260, (16, 24, 24))])
def test_rope3d_many_heads(dtype, H, n, sections):
    rng = np.random.default_rng(H + n)
    x = rng.standard_normal((H, n, sum(sections))).astype(np.float32)
    x = synth.to_bf16(x) if dtype == "bf16" else x
    pos = rng.integers(0, 700, (n, 3)).astype(np.int32)
    buf = torch.full((H, n + 2, sum(sections)), 7.0, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV)
    buf[:, :n] = dev(x, dtype)
    pk.pc_rope3d(buf[:, :n], dev(pos, None), sections, 1e4)
    want = orc.rope3d(x, pos, sections, 1e4)
    tol = 2.0 ** -8 if dtype == "bf16" else 2e-6      # as above: one rounding of the result
    assert np.all(np.abs(host(buf[:, :n]).astype(np.float64) - want) <= tol * np.abs(want) + 1e-6)
    assert (buf[:, n:] == 7).all()


def test_rope3d_negative_shift_undoes_rotation_and_head_stride():
    # a rebase by (-dt, 0, 0) (Eq. 9) is a rotation with negative position; also exercises
    # a head stride larger than n*D (capacity > rows)
    rng = np.random.default_rng(5)
    cap, n = 64, 50
    buf = torch.zeros((2, cap, 128), dtype=torch.float32, device=DEV)
    x = rng.standard_normal((2, n, 128)).astype(np.float32)
    buf[:, :n] = dev(x, "f32")
    pos = np.stack([rng.integers(0, 100, n), rng.integers(0, 100, n), rng.integers(0, 100, n)], 1).astype(np.int32)
    view = buf[:, :n]
    pk.pc_rope3d(view, dev(pos, None), (32, 48, 48), 1e4)
    np.testing.assert_allclose(host(view), orc.rope3d(x, pos, (32, 48, 48), 1e4), atol=2e-6)
    pk.pc_rope3d(view, dev(-pos, None), (32, 48, 48), 1e4)
    np.testing.assert_allclose(host(view), x, atol=4e-6)
    assert torch.all(buf[:, n:] == 0)


# ------------------------------------------------------------------------------- attention
def _attn_case(dtype, hq, hkv, nq, nk, d, seed):
    rng = np.random.default_rng(seed)
    Q = rng.standard_normal((hq, nq, d)).astype(np.float32)
    K = rng.standard_normal((hkv, nk, d)).astype(np.float32)
    V = rng.standard_normal((hkv, nk, d)).astype(np.float32)
    if dtype == "bf16":
        Q, K, V = synth.to_bf16(Q), synth.to_bf16(K), synth.to_bf16(V)
    return Q, K, V


def _fold(Q, scale):
    """Queries that carry scale * log2(e) (rounded to bf16 once, as a rotation with out_scale
    would leave them) and the scale that is left for the calls: the same softmax, and both
    sides read the same bits."""
    return synth.to_bf16((Q.astype(np.float64) * q_fold(scale)).astype(np.float32)), LN2


def _masked_reference(Q, K, V, keep, scale, rows):
    """(O rows, lse rows, importances) of the unmasked keys alone, in 64 bits on the GPU."""
    hq, hkv = Q.shape[0], K.shape[0]
    O, L = [], []
    mass = torch.zeros((hkv, int(keep.sum())), dtype=torch.float64, device=DEV)
    for h in range(hq):
        s = Q[h, rows].double() @ K[h * hkv // hq, keep].double().t() * scale
        p = torch.softmax(s, dim=1)
        O.append(p @ V[h * hkv // hq, keep].double())
        L.append(torch.logsumexp(s, dim=1))
        mass[h * hkv // hq] += p.sum(0)
    return torch.stack(O), torch.stack(L), mass


def _attn_check(dtype, Q, K, V, scale, fold=False):
    if fold:
        Q, scale = _fold(Q, scale)
    hq, nq, d = Q.shape
    nk = K.shape[1]
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(dev(Q, dtype), dev(K, dtype), dev(V, dtype), nk, scale, lse=lse)
    Ow, Lw = orc.frame_attn(Q, K, V, scale)
    err = np.abs(host(O).astype(np.float64) - Ow)
    lerr = np.abs(host(lse).astype(np.float64) - Lw)
    if dtype == "bf16":
        assert err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
        assert lerr.max() <= 1e-3
    else:
        assert err.max() <= 1e-5, err.max()
        assert lerr.max() <= 1e-5
    return err


# fold = True: the queries carry scale * log2(e) and the calls get scale = ln 2 (the kernels'
# shorter loop: scores start from minus the reference inside the matrix product)
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("nq,nk", [(1, 1), (5, 63), (64, 64), (65, 65), (256, 128), (300, 777), (513, 1000)])
def test_frame_attn_bf16_shapes(nq, nk, fold):
    Q, K, V = _attn_case("bf16", 4, 2, nq, nk, 128, nq * 1000 + nk)
    _attn_check("bf16", Q, K, V, 128 ** -0.5, fold)


@pytest.mark.parametrize("fold", [False, True])
def test_frame_attn_bf16_gqa_groups_and_large_logits(fold):
    # 3 query heads per KV head; a strong shared direction makes logits reach ~ +-40
    Q, K, V = _attn_case("bf16", 6, 2, 130, 500, 128, 77)
    Q[..., :8] += 4.0
    K[:, ::7, :8] += 4.0
    Q, K = synth.to_bf16(Q), synth.to_bf16(K)
    _attn_check("bf16", Q, K, V, 128 ** -0.5, fold)


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step", [0.05, 0.6, 40.0])
def test_frame_attn_bf16_reference_maximum_is_refreshed(step, fold):
    # logits that keep growing along the key axis: the kernel forms probabilities against a
    # reference maximum it only refreshes when a row sum runs away, so a slow drift (never
    # refreshed), a steady climb (refreshed every few tiles) and jumps of hundreds of units
    # (the stale reference overflows to inf first) must all come out right.
    rng = np.random.default_rng(9)
    hq, hkv, nq, nk, d = 4, 2, 70, 900, 128
    Q = rng.standard_normal((hq, nq, d)).astype(np.float32)
    K = rng.standard_normal((hkv, nk, d)).astype(np.float32) * 0.1
    V = rng.standard_normal((hkv, nk, d)).astype(np.float32)
    Q[..., 0] = 8.0
    ramp = step * (np.arange(nk) // 32)                     # logit contribution grows per half tile
    K[..., 0] = (ramp / (8.0 * d ** -0.5))[None, :]
    Q, K, V = synth.to_bf16(Q), synth.to_bf16(K), synth.to_bf16(V)
    _attn_check("bf16", Q, K, V, d ** -0.5, fold)


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("hq,hkv,nq,nk", [(6, 2, 300, 3000), (24, 8, 520, 2100), (3, 1, 40, 5000)])
def test_frame_attn_bf16_key_shares_and_merge(hq, hkv, nq, nk, fold):
    # shapes whose work-group count fills the chip badly: the keys are cut into shares and
    # merged (when a workspace is supplied); without one the un-split kernel must agree
    Q, K, V = _attn_case("bf16", hq, hkv, nq, nk, 128, 5)
    assert pk.pc_frame_attn_workspace_bytes(hq, nq, nk, 128) > 0
    _attn_check("bf16", Q, K, V, 128 ** -0.5, fold)                # binding supplies the workspace
    scale = 128 ** -0.5
    if fold:
        Q, scale = _fold(Q, scale)
    Qd, Kd, Vd = dev(Q, "bf16"), dev(K, "bf16"), dev(V, "bf16")
    split = pk.pc_frame_attn(Qd, Kd, Vd, nk, scale)
    whole = pk.pc_frame_attn(Qd, Kd, Vd, nk, scale, ws=torch.empty(16, dtype=torch.uint8, device=DEV))
    assert (split.float() - whole.float()).abs().max().item() <= 2 ** -6   # two roundings of values of O(1)


ATTN_ACROSS_HEADS = [(2, 1, 33, 1), (3, 1, 31, 33), (6, 2, 43, 257), (2, 1, 84, 255), (2, 1, 184, 5000),
                     (24, 8, 520, 2100), (16, 4, 2010, 2499), (24, 8, 2901, 2100)]
ATTN_256_ROWS_UNCUT = [(16, 4, 3990, nk) for nk in (1, 31, 33, 64, 65, 128, 129, 192, 193, 2499)]


# Row tiles that span query heads (nq is no multiple of the tile), steps and tiles of the keys that are
# empty, single or ragged, and both forms of the kernel: the first five shapes take 32 rows per
# work-group (four un-split, one in key shares; all with divided output dims, ATTN_32_ROWS_WHOLE has the others), the
# others 256 rows (in key shares twice; a whole round of row tiles un-split and the rest in key shares).
# test_host_abi.py pins these forms.
# step: logits climb along the key axis, as above.  Every row is computed; the oracle checks the rows
# at the tile edges and a stride of the others.
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step", [0.0, 0.6, 40.0])
@pytest.mark.parametrize("hq,hkv,nq,nk", ATTN_ACROSS_HEADS)
def test_frame_attn_bf16_row_tiles_across_heads(hq, hkv, nq, nk, step, fold):
    Q, K, V = _attn_case("bf16", hq, hkv, nq, nk, 128, nq + nk)
    scale = 128 ** -0.5
    if step:
        Q[..., 0] = 8.0
        K *= 0.1
        K[..., 0] = step * (np.arange(nk) // 32) / (8.0 * scale)
        Q, K = synth.to_bf16(Q), synth.to_bf16(K)
    if fold:
        Q, scale = _fold(Q, scale)
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(dev(Q, "bf16"), dev(K, "bf16"), dev(V, "bf16"), nk, scale, lse=lse)
    rows = sorted({0, 1, nq // 2, nq - 2, nq - 1} | set(range(0, nq, 97)))
    Ow, Lw = orc.frame_attn(np.ascontiguousarray(Q[:, rows]), K, V, scale)
    err = np.abs(host(O)[:, rows].astype(np.float64) - Ow)
    # a climb of 40 per half tile leaves all weight on the last keys: |O| reaches 4, where bf16 values
    # lie 2^-6 apart (outputs and probabilities rounded once each); else |O| < 2 as in the other tests
    tol = 2 ** -5 if step == 40.0 or nk < 40 else 2e-2
    assert err.max() <= tol and err.mean() <= 2e-3, (err.max(), err.mean())
    lw_ulp = np.maximum(1.0, np.abs(Lw)) * 2.0 ** -20     # fp32 products and logs of values up to |Lw|
    assert (np.abs(host(lse)[:, rows].astype(np.float64) - Lw) <= np.maximum(1e-3, lw_ulp)).all()


# 256 rows per work-group with all keys: walks of one, two, three and four tiles of 64, whole and ragged, a
# last half tile with no key, fewer keys than a half tile; many tiles once.  step: logits climb along the
# key axis by so much per half tile (0.05: the first reference stands throughout).
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step", [0.0, 0.05, 0.6, 40.0])
@pytest.mark.parametrize("hq,hkv,nq,nk", ATTN_256_ROWS_UNCUT)
def test_frame_attn_bf16_256_rows_and_few_keys(hq, hkv, nq, nk, step, fold):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(nk)
    Q, K, V = (torch.randn((h, n, 128), generator=gen, device=DEV) for h, n in ((hq, nq), (hkv, nk), (hkv, nk)))
    scale = 128 ** -0.5
    if step:
        Q[..., 0] = 8.0
        K *= 0.1
        K[..., 0] = step * (torch.arange(nk, device=DEV) // 32) / (8.0 * scale)
    if fold:
        Q, scale = Q * q_fold(scale), LN2
    Q, K, V = Q.bfloat16(), K.bfloat16(), V.bfloat16()
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(Q, K, V, nk, scale, lse=lse, ws=torch.empty(16, dtype=torch.uint8, device=DEV))
    rows = torch.tensor(sorted({0, 1, nq - 1} | set(range(0, nq, 61))), device=DEV)
    Ow, Lw, _ = _masked_reference(Q, K, V, torch.ones(nk, dtype=torch.bool, device=DEV), scale, rows)
    err, lerr = (O[:, rows].double() - Ow).abs(), (lse[:, rows].double() - Lw).abs()
    # tolerances as in the test above: with all weight on few keys |O| reaches 4
    assert err.max().item() <= (2 ** -5 if step == 40.0 or nk < 40 else 2e-2) and err.mean().item() <= 2e-3
    assert (lerr <= torch.clamp(Lw.abs().clamp(min=1.0) * 2.0 ** -20, min=1e-3)).all()


# 64 and 128 rows per work-group (four and two key groups): one tile of 32 keys and fewer, key groups without a tile or
# with one less than the others, ragged ends, every number of tiles modulo the LDS slots, row groups without a row, row
# tiles that span heads, key shares; climbing logits as above, and masks that leave whole tiles or key groups nothing.
ATTN_64_ROWS = [(16, 4, 581, nk) for nk in (97, 129, 257, 300, 823)] + [(6, 2, 1593, 1701), (24, 8, 481, 970), (2, 1, 1701, 8100)]
ATTN_128_ROWS = [(8, 2, 3541, nk) for nk in (1, 31, 33, 64, 65, 151, 200, 257)] + [(6, 2, 3157, 523), (24, 8, 1070, 1691)]


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step,masked", [(0.0, None), (0.6, None), (40.0, None), (0.0, slice(0, 140)), (0.0, slice(3, None, 5))])
@pytest.mark.parametrize("hq,hkv,nq,nk", ATTN_64_ROWS + ATTN_128_ROWS)
def test_frame_attn_bf16_64_and_128_rows(hq, hkv, nq, nk, step, masked, fold):
    rows_wg = 64 if (hq, hkv, nq, nk) in ATTN_64_ROWS else 128
    n_ws = pk.pc_frame_attn_workspace_bytes_for(pk.PC_BF16, hq, hkv, nq, nk, 128)
    assert pk.pc_frame_attn_cut(pk.PC_BF16, hq, hkv, nq, nk, 128, n_ws)[0] == rows_wg
    gen = torch.Generator(device=DEV)
    gen.manual_seed(nk)
    Q, K, V = (torch.randn((h, n, 128), generator=gen, device=DEV) for h, n in ((hq, nq), (hkv, nk), (hkv, nk)))
    scale = 128 ** -0.5
    keep = torch.ones(nk, dtype=torch.bool, device=DEV)
    if step:
        Q[..., 0] = 8.0
        K *= 0.1
        K[..., 0] = step * (torch.arange(nk, device=DEV) // 32) / (8.0 * scale)
    if masked is not None:
        Q[..., 0] = 4.0
        keep[masked] = False
        keep[-1] |= not keep.any()
        K[:, ~keep, 0] = float("-inf")
    if fold:
        Q, scale = Q * q_fold(scale), LN2
    Q, K, V = Q.bfloat16(), K.bfloat16(), V.bfloat16()
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    buf = torch.full((hq, nq + 3, 128), 7.0, dtype=torch.bfloat16, device=DEV)
    O = pk.pc_frame_attn(Q, K, V, nk, scale, O=buf[:, :nq], lse=lse)
    rows = torch.tensor(sorted({0, 1, 63, 64, 127, 128, nq - 1} | set(range(0, nq, 61))), device=DEV)
    Ow, Lw, _ = _masked_reference(Q, K, V, keep, scale, rows)
    err, lerr = (O[:, rows].double() - Ow).abs(), (lse[:, rows].double() - Lw).abs()
    # tolerances as in the test above: with all weight on few keys |O| reaches 4
    assert err.max().item() <= (2 ** -5 if step == 40.0 or keep.sum() < 40 else 2e-2) and err.mean().item() <= 2e-3
    assert (lerr <= torch.clamp(Lw.abs().clamp(min=1.0) * 2.0 ** -20, min=1e-3)).all() and (buf[:, nq:] == 7).all()


# 32 rows per work-group whose output's dims are divided by four, by two and not at all: the last row tile before and
# the first behind each line, key shares of both, waves without a key, ragged ends; NaN behind the last V row.
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("nq,nk,work_groups", [(1024, 1, 64), (1025, 33, 65), (2048, 257, 128), (2049, 300, 129),
                                               (1000, 255, 63), (93, 2000, 48), (184, 5000, 120)])
def test_frame_attn_bf16_output_dims_divided(nq, nk, work_groups, fold):
    cut = pk.pc_frame_attn_cut(pk.PC_BF16, 2, 1, nq, nk, 128, 1 << 40)
    assert cut[0] == 32 and -(-2 * nq // 32) * cut[1] == work_groups
    gen = torch.Generator(device=DEV)
    gen.manual_seed(nq)
    Q, K, V = (torch.randn((h, n, 128), generator=gen, device=DEV) for h, n in ((2, nq), (1, nk + 40), (1, nk + 40)))
    scale = 128 ** -0.5
    if fold:
        Q, scale = Q * q_fold(scale), LN2
    Q, K, V = Q.bfloat16(), K.bfloat16(), V.bfloat16()
    V[:, nk:] = float("nan")
    lse = torch.empty((2, nq), dtype=torch.float32, device=DEV)
    buf = torch.full((2, nq + 3, 128), 7.0, dtype=torch.bfloat16, device=DEV)
    O = pk.pc_frame_attn(Q, K, V, nk, scale, O=buf[:, :nq], lse=lse)
    rows = torch.tensor(sorted({0, 1, 31, 32, nq - 1} | set(range(0, nq, 61))), device=DEV)
    Ow, Lw, _ = _masked_reference(Q, K[:, :nk], V[:, :nk], torch.ones(nk, dtype=torch.bool, device=DEV), scale, rows)
    err, lerr = (O[:, rows].double() - Ow).abs(), (lse[:, rows].double() - Lw).abs()
    # outputs and probabilities rounded once each; with few keys |O| reaches 4, where bf16 values lie 2^-6 apart
    assert err.max().item() <= (2 ** -5 if nk < 40 else 2e-2) and err.mean().item() <= 2e-3
    assert lerr.max().item() <= 1e-3 and (buf[:, nq:] == 7).all()


# 32 rows per work-group whose output's dims are not divided (more than 128 work-groups): less than a step of keys, a
# step and a ragged one, many steps, key shares, two rounds of work-groups; climbing logits and masks as above, which
# leave steps and waves nothing or move every reference
ATTN_32_ROWS_WHOLE = [(6, 2, 691, 33, 1), (6, 2, 700, 257, 1), (16, 4, 300, 1804, 1), (6, 2, 300, 3000, 4), (28, 4, 573, 2243, 1)]


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step,masked", [(0.05, None), (0.6, None), (40.0, None), (0.0, slice(0, 140)), (0.0, slice(40, 300)),
                                         (0.0, slice(3, None, 5)), (0.0, slice(0, -3)), (0.0, slice(5, None))])
@pytest.mark.parametrize("hq,hkv,nq,nk,shares", ATTN_32_ROWS_WHOLE)
def test_frame_attn_bf16_output_dims_not_divided(hq, hkv, nq, nk, shares, step, masked, fold):
    n_ws = pk.pc_frame_attn_workspace_bytes_for(pk.PC_BF16, hq, hkv, nq, nk, 128)
    assert pk.pc_frame_attn_cut(pk.PC_BF16, hq, hkv, nq, nk, 128, n_ws)[:2] == (32, shares)
    assert hkv * -(-(hq // hkv * nq) // 32) * shares > 128
    gen = torch.Generator(device=DEV)
    gen.manual_seed(nq + nk)
    Q, K, V = (torch.randn((h, n, 128), generator=gen, device=DEV) for h, n in ((hq, nq), (hkv, nk), (hkv, nk)))
    scale = 128 ** -0.5
    keep = torch.ones(nk, dtype=torch.bool, device=DEV)
    if step:
        Q[..., 0] = 8.0
        K *= 0.1
        K[..., 0] = step * (torch.arange(nk, device=DEV) // 32) / (8.0 * scale)
    if masked is not None:
        Q[..., 0] = 4.0
        keep[masked] = False
        keep[-1] |= not keep.any()
        K[:, ~keep, 0] = float("-inf")
    if fold:
        Q, scale = Q * q_fold(scale), LN2
    Q, K, V = Q.bfloat16(), K.bfloat16(), V.bfloat16()
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(Q, K, V, nk, scale, lse=lse)
    rows = torch.tensor(sorted({0, 1, 31, 32, nq - 1} | set(range(0, nq, 37))), device=DEV)
    Ow, Lw, _ = _masked_reference(Q, K, V, keep, scale, rows)
    err, lerr = (O[:, rows].double() - Ow).abs(), (lse[:, rows].double() - Lw).abs()
    # tolerances as in the tests above: with all weight on few keys |O| reaches 4
    assert err.max().item() <= (2 ** -5 if step == 40.0 or keep.sum() < 40 else 2e-2) and err.mean().item() <= 2e-3
    assert (lerr <= torch.clamp(Lw.abs().clamp(min=1.0) * 2.0 ** -20, min=1e-3)).all()


# What lies in the spare rows behind the last key stays out of it in every form: 32, 64, 128 and 256 rows per work-group,
# a ragged last tile, key groups and shares without a whole one
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("rows_wg,hq,hkv,nq,nk", [(32, 6, 2, 691, 33), (32, 6, 2, 300, 3000), (32, 4, 2, 70, 900)] +
                         [(64, 16, 4, 581, n) for n in (97, 129, 257)] + [(64, 2, 1, 1701, 8100)] +
                         [(128, 8, 2, 3541, n) for n in (1, 33, 65, 151)] + [(128, 24, 8, 1070, 1691), (256, 16, 4, 1008, 7455)])
def test_frame_attn_bf16_spare_rows_stay_out(rows_wg, hq, hkv, nq, nk, fold):
    n_ws = pk.pc_frame_attn_workspace_bytes_for(pk.PC_BF16, hq, hkv, nq, nk, 128)
    assert pk.pc_frame_attn_cut(pk.PC_BF16, hq, hkv, nq, nk, 128, n_ws)[0] == rows_wg
    gen = torch.Generator(device=DEV)
    gen.manual_seed(nk)
    Q, K, V = (torch.randn((h, n, 128), generator=gen, device=DEV) for h, n in ((hq, nq), (hkv, nk + 600), (hkv, nk + 600)))
    scale = 128 ** -0.5
    if fold:
        Q, scale = Q * q_fold(scale), LN2
    Q, K, V = Q.bfloat16(), K.bfloat16(), V.bfloat16()
    K[:, nk:], V[:, nk:] = float("nan"), float("nan")
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(Q, K, V, nk, scale, lse=lse)
    rows = torch.tensor(sorted({0, 1, nq - 1} | set(range(0, nq, 61))), device=DEV)
    Ow, Lw, _ = _masked_reference(Q, K[:, :nk], V[:, :nk], torch.ones(nk, dtype=torch.bool, device=DEV), scale, rows)
    err, lerr = (O[:, rows].double() - Ow).abs(), (lse[:, rows].double() - Lw).abs()
    assert not O.isnan().any() and not lse.isnan().any()
    # outputs and probabilities rounded once each; with few keys |O| reaches 4, where bf16 values lie 2^-6 apart
    assert err.max().item() <= (2 ** -5 if nk < 40 else 2e-2) and err.mean().item() <= 2e-3 and lerr.max().item() <= 1e-3


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_frame_attn_bf16_error_bound_at_twice_the_workload_amplitude(seed, fold):
    """The absolute bar (max 2e-2) presumes outputs of the workloads' size, |O| < 2.  With Q and K
    at twice the amplitude the softmax is peaked and an output follows single V rows, so |O|
    reaches 2..4, where bf16 values lie 2^-6 apart.  What the arithmetic guarantees at ANY
    amplitude: the final rounding of O (at most 2^-8 |O|) plus the rounding of the probabilities
    to bf16 before the second product (at most 2^-8 sum_j p_j |v_j|; the normaliser is summed
    from the un-rounded ones) plus fp32 effects.  Checked element by element; for |V| <= 3.5
    (so |O| < 4) that is at most 0.0078 + 0.0137, which gives the documented max 2.5e-2."""
    rng = np.random.default_rng(1234 + seed)
    hq, hkv, nq, nk, d = 4, 2, 333, 2500 - 300 * seed, 128
    Q = synth.to_bf16((2.0 * rng.standard_normal((hq, nq, d))).astype(np.float32))
    K = synth.to_bf16((2.0 * rng.standard_normal((hkv, nk, d))).astype(np.float32))
    V = synth.to_bf16(np.clip(rng.standard_normal((hkv, nk, d)), -3.5, 3.5).astype(np.float32))
    scale = d ** -0.5
    if fold:
        Q, scale = _fold(Q, scale)
    O = pk.pc_frame_attn(dev(Q, "bf16"), dev(K, "bf16"), dev(V, "bf16"), nk, scale)
    Ow, _ = orc.frame_attn(Q, K, V, scale)
    Aw, _ = orc.frame_attn(Q, K, np.abs(V), scale)              # sum_j p_j |v_j|
    err = np.abs(host(O).astype(np.float64) - Ow)
    assert np.abs(Ow).max() > 2.0, "the case must reach outputs beyond the workloads' size"
    assert np.all(err <= 2.0 ** -8 * (np.abs(Ow) + Aw) + 5e-4), (err - 2.0 ** -8 * (np.abs(Ow) + Aw)).max()
    assert err.max() <= 2.5e-2 and err.mean() <= 2e-3, (err.max(), err.mean())


def test_frame_attn_bf16_closed_forms():
    Q, K, V = _attn_case("bf16", 2, 1, 70, 200, 128, 3)
    Ke = np.repeat(K[:, :1], 200, axis=1)                     # all keys equal -> mean of V
    O = host(pk.pc_frame_attn(dev(Q, "bf16"), dev(Ke, "bf16"), dev(V, "bf16"), 200, 0.1))
    np.testing.assert_allclose(O, np.broadcast_to(V.mean(1)[0], O.shape), atol=4e-3)
    O1 = host(pk.pc_frame_attn(dev(Q, "bf16"), dev(K[:, 5:6], "bf16"), dev(V[:, 5:6], "bf16"), 1, 0.1))
    assert np.array_equal(O1, np.broadcast_to(V[0, 5], O1.shape))   # one key -> that value row


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shares", [0.5, 2, 3.5])
def test_frame_attn_takes_as_many_key_shares_as_the_workspace_holds(shares, dtype):
    # the call would take about ten shares; a workspace for fewer means fewer, a misaligned one none
    hq, nq, nk, d = 2, 184, 5000, 128
    Q, K, V = _attn_case(dtype, hq, 1, nq, nk, d, 21)
    Qd, Kd, Vd = dev(Q, dtype), dev(K, dtype), dev(V, dtype)
    n = int(shares * hq * nq * (d * 4 + 8)) + 512
    buf = torch.full((n + 4096,), 255, dtype=torch.uint8, device=DEV)
    Ow, Lw = orc.frame_attn(Q, K, V, d ** -0.5)
    for off in (0, 8):
        lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
        O = pk.pc_frame_attn(Qd, Kd, Vd, nk, d ** -0.5, lse=lse, ws=buf[off:off + n])
        tol = 2e-2 if dtype == "bf16" else 1e-5
        assert np.abs(host(O).astype(np.float64) - Ow).max() <= tol
        assert np.abs(host(lse).astype(np.float64) - Lw).max() <= tol
        assert (buf[off + n:] == 255).all()     # nothing behind the workspace was written


def test_frame_attn_workspace_holds_the_rows_that_are_cut():
    # 8 x 34 row tiles: the 256 of the first round walk all keys, the last 4,095 rows are cut; a workspace
    # for 16 shares of those rows (half of what two shares of every row would take) changes nothing
    hq, hkv, nq, nk, d = 24, 8, 2901, 2100, 128
    Q, K, V = (dev(x, "bf16") for x in _attn_case("bf16", hq, hkv, nq, nk, d, 22))
    n_cut = hq * nq - (7 * 3 * nq + 18 * 256)
    n = 16 * n_cut * (d * 4 + 8) + 512
    buf = torch.full((n + 4096,), 255, dtype=torch.uint8, device=DEV)
    ample = torch.empty(4 * hq * nq * (d * 4 + 8) * 4, dtype=torch.uint8, device=DEV)
    none = torch.empty(16, dtype=torch.uint8, device=DEV)
    O, Oa, On = (pk.pc_frame_attn(Q, K, V, nk, d ** -0.5, ws=ws) for ws in (buf[:n], ample, none))
    assert torch.equal(O, Oa) and (buf[n:] == 255).all()
    flat, flat_n = O.reshape(-1, d), On.reshape(-1, d)
    assert torch.equal(flat[:-n_cut], flat_n[:-n_cut]) and not torch.equal(flat[-n_cut:], flat_n[-n_cut:])


@pytest.mark.parametrize("dtype,hq,hkv,nq,nk,d", [("bf16", 8, 2, 252, 1804, 128), ("bf16", 16, 4, 1008, 7455, 128),
                                                  ("bf16", 24, 8, 4032, 2100, 128), ("f32", 8, 2, 252, 1804, 128),
                                                  ("f32", 2, 1, 64, 336, 64)])
def test_frame_attn_takes_the_same_cut_in_the_workspace_it_asks_for(dtype, hq, hkv, nq, nk, d):
    Q, K, V = (dev(x, dtype) for x in _attn_case(dtype, hq, hkv, nq, nk, d, 23))
    n = pk.pc_frame_attn_workspace_bytes_for(pk.PC_BF16 if dtype == "bf16" else pk.PC_F32, hq, hkv, nq, nk, d)
    assert n > 0
    buf = torch.full((n + 4096,), 255, dtype=torch.uint8, device=DEV)
    ample = torch.empty(16 * hq * nq * (d * 4 + 8) + 512, dtype=torch.uint8, device=DEV)
    a, b, c = (pk.pc_frame_attn(Q, K, V, nk, d ** -0.5, ws=ws) for ws in (buf[:n], ample, None))
    assert torch.equal(a, b) and torch.equal(a, c) and (buf[n:] == 255).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nq,nk", [(1, 1), (64, 336), (70, 33), (130, 191)])
def test_frame_attn_f32_shapes(d, nq, nk):
    Q, K, V = _attn_case("f32", 4, 2, nq, nk, d, d + nq + nk)
    _attn_check("f32", Q, K, V, d ** -0.5)


# edges of the fp32 kernel's 16-row tiles, 32-key steps and key shares (17 rows x 5,000 keys: shares)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nq,nk", [(15, 31), (16, 32), (17, 33), (31, 255), (32, 256), (33, 257), (17, 5000), (301, 2501)])
def test_frame_attn_f32_tile_edges_and_key_shares(d, nq, nk):
    # 16 query rows per work-group, 32 in the last shape at D = 128; the first two shapes are one wave's step;
    # tiles of rows that span the three heads
    Q, K, V = _attn_case("f32", 3, 1, nq, nk, d, d + nq + nk)
    _attn_check("f32", Q, K, V, d ** -0.5)
    # without a workspace the keys are not cut: the same sums in another order
    a = pk.pc_frame_attn(dev(Q, None), dev(K, None), dev(V, None), nk, d ** -0.5)
    b = pk.pc_frame_attn(dev(Q, None), dev(K, None), dev(V, None), nk, d ** -0.5,
                         ws=torch.empty(16, dtype=torch.uint8, device=DEV))
    assert (a - b).abs().max().item() <= 2e-6   # two fp32 results of |O| < 4, each within a few 2^-24 |O| of exact


# at most one step of keys: one wave, written without a merge; row tiles that span heads, strided output
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,nq,nk", [(1, 1, 1, 1), (3, 1, 17, 3), (6, 2, 37, 17), (8, 2, 252, 31), (2, 1, 16, 32)])
def test_frame_attn_f32_few_keys(d, hq, hkv, nq, nk):
    Q, K, V = _attn_case("f32", hq, hkv, nq, nk, d, nq + nk)
    _attn_check("f32", Q, K, V, d ** -0.5)
    buf = torch.full((hq, nq + 3, d), 7.0, dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(dev(Q, None), dev(K, None), dev(V, None), nk, d ** -0.5, O=buf[:, :nq])
    assert np.abs(host(O) - orc.frame_attn(Q, K, V, d ** -0.5)[0]).max() <= 1e-5 and (buf[:, nq:] == 7).all()


@pytest.mark.parametrize("nq,nk", [(70, 900), (301, 2501)])
@pytest.mark.parametrize("step", [0.05, 0.6, 40.0])
def test_frame_attn_f32_reference_is_refreshed(nq, nk, step):
    # logits that climb along the key axis: the reference lags by up to 2^8 before the rows are rescaled
    Q, K, V = _attn_case("f32", 3, 1, nq, nk, 128, 9)
    Q[..., 0] = 8.0
    K *= 0.1
    K[..., 0] = step * (np.arange(nk) // 32) / (8.0 * 128 ** -0.5)
    lse = torch.empty((3, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(dev(Q, None), dev(K, None), dev(V, None), nk, 128 ** -0.5, lse=lse)
    rows = sorted({0, 15, 16, 31, 32, nq - 1} | set(range(0, nq, 37)))
    Ow, Lw = orc.frame_attn(Q[:, rows], K, V, 128 ** -0.5)
    # a logit L is an fp32 sum of products of magnitude L: its error is a few L 2^-24, and so is p's
    rel = 8 * max(1.0, np.abs(Lw).max()) * 2.0 ** -24
    assert np.abs(host(O)[:, rows] - Ow).max() <= 4 * rel + 1e-6
    assert np.abs(host(lse)[:, rows] - Lw).max() <= rel


def test_frame_attn_f32_takes_buffers_that_are_not_16_byte_aligned():
    Q, K, V = _attn_case("f32", 2, 1, 20, 70, 64, 12)
    def odd(x):
        t = torch.empty(x.size + 1, dtype=torch.float32, device=DEV)[1:].view(x.shape)
        return t.copy_(dev(x, None))
    O = pk.pc_frame_attn(odd(Q), odd(K), odd(V), 70, 0.125, O=odd(np.zeros_like(Q)))
    Ow, _ = orc.frame_attn(Q, K, V, 0.125)
    assert np.abs(host(O) - Ow).max() <= 1e-5


# A caller that masks keys through a coordinate of its own (the queries carry a constant there): their
# logits are -inf, the type's lowest value times a constant, or far below the rest.  Steps, waves, half
# tiles and key shares that hold nothing else, first and last ones among them: 32 rows per work-group
# in two and in ten shares (un-split: ATTN_32_ROWS_WHOLE), 256 un-split and in four shares of 1,920 keys; fp32 with 16
# and 32.
@pytest.mark.parametrize("value", [float("-inf"), "lowest", -3e5])
@pytest.mark.parametrize("masked", [slice(3, None, 5), slice(40, 300), slice(0, 140), slice(1900, 2040), slice(0, -3), slice(5, None)])
@pytest.mark.parametrize("dtype,d,fold,hq,hkv,nq,nk", [
    ("bf16", 128, False, 8, 2, 252, 1804), ("bf16", 128, True, 8, 2, 252, 1804), ("bf16", 128, False, 2, 1, 184, 5000),
    ("bf16", 128, False, 16, 4, 4032, 2048), ("bf16", 128, True, 16, 4, 4032, 2048),
    ("bf16", 128, False, 16, 4, 1008, 7455), ("bf16", 128, True, 16, 4, 1008, 7455),
    ("f32", 64, False, 2, 1, 64, 336), ("f32", 128, False, 2, 1, 33, 336), ("f32", 64, False, 2, 1, 20, 30), ("f32", 128, False, 8, 2, 252, 1804),
    ("f32", 64, False, 3, 1, 301, 2501)])
def test_masked_keys_weigh_nothing(dtype, d, fold, hq, hkv, nq, nk, masked, value):
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, V = (dev(x, dtype) for x in _attn_case(dtype, hq, hkv, nq, nk, d, nq + nk))
    Q[..., 0] = 4.0
    scale = d ** -0.5
    if fold:
        Q, scale = (Q.double() * q_fold(scale)).to(td), LN2
    keep = torch.ones(nk, dtype=torch.bool, device=DEV)
    keep[masked] = False
    keep[-1] |= not keep.any()      # a table shorter than the mask keeps its last key
    K[:, ~keep, 0] = torch.finfo(td).min if value == "lowest" else value
    rows = torch.arange(0, nq, max(1, nq // 40), device=DEV)
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(Q, K, V, nk, scale, lse=lse)
    Ow, Lw, mass = _masked_reference(Q, K, V, keep, scale, rows)
    err, lerr = (O[:, rows].double() - Ow).abs(), (lse[:, rows].double() - Lw).abs().max().item()
    # with three keys left |O| reaches 4, as in the tests of climbing logits above
    tol = (2 ** -5 if keep.sum() < 40 else 2e-2, 1e-3) if dtype == "bf16" else (1e-5, 1e-5)
    assert not O.isnan().any() and err.max().item() <= tol[0] and lerr <= tol[1], (err.max().item(), lerr)
    score = pk.pc_score(Q[:, rows].contiguous(), K, nk, scale).double()
    rel = max(2e-5, 6 * Lw.abs().max().item() * 1.4427 * 2.0 ** -23)      # as in the tests of pc_score
    assert (score[:, ~keep] == 0).all()
    assert ((score[:, keep] - mass).abs() <= 2e-7 + rel * mass).all()


def test_frame_attn_capacity_larger_than_rows():
    # K/V live in buffers with spare capacity (head stride > Nk*D), as a cache does
    Q, K, V = _attn_case("bf16", 4, 2, 100, 300, 128, 11)
    Kb = torch.zeros((2, 512, 128), dtype=torch.bfloat16, device=DEV)
    Vb = torch.full((2, 512, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    Kb[:, :300], Vb[:, :300] = dev(K, "bf16"), dev(V, "bf16")
    O = pk.pc_frame_attn(dev(Q, "bf16"), Kb, Vb, 300, 128 ** -0.5)
    Ow, _ = orc.frame_attn(Q, K, V, 128 ** -0.5)
    err = np.abs(host(O) - Ow)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3


# fp32: whatever lies in the spare rows behind the last key stays out of it, in a step's rows and in steps wholly
# behind the end: one and two waves' keys, rests of a step of every kind, waves that run out before the others (16
# and 32 rows per work-group), key shares
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,nq,nk", [(4, 2, 37, n) for n in (1, 3, 15, 17, 31, 33, 129, 255)] + [(2, 1, 64, 336), (8, 2, 252, 1804), (3, 1, 301, 2501)])
def test_frame_attn_f32_capacity_larger_than_rows(d, hq, hkv, nq, nk):
    Q, K, V = _attn_case("f32", hq, hkv, nq, nk, d, nk)
    buf = torch.full((2, hkv, nk + 300, d), float("nan"), dtype=torch.float32, device=DEV)
    buf[0, :, :nk], buf[1, :, :nk] = dev(K, None), dev(V, None)
    lse = torch.empty((hq, nq), dtype=torch.float32, device=DEV)
    O = pk.pc_frame_attn(dev(Q, None), buf[0], buf[1], nk, d ** -0.5, lse=lse)
    Ow, Lw = orc.frame_attn(Q, K, V, d ** -0.5)
    assert np.abs(host(O) - Ow).max() <= 1e-5 and np.abs(host(lse) - Lw).max() <= 1e-5


# ------------------------------------------------------------------------------- score
def _score_check(w, Qs, K, share=False, lse=None, fold=False):
    dt = w.dtype
    scale = w.scale
    if fold:
        Qs, scale = _fold(Qs, scale)
    got = host(pk.pc_score(dev(Qs, dt), dev(K, dt), K.shape[1], scale, lse=lse, share_heads=share)).astype(np.float64)
    want = orc.score(Qs, K, scale, share_heads=share)
    err = np.abs(got - want)
    # fp32 exponentials and sums of probabilities computed from exact bf16 products
    assert np.all(err <= 2e-7 + 2e-5 * want), (err.max(), (err / (want + 1e-30)).max())
    rep = w.Hq // w.Hkv
    np.testing.assert_allclose(got.sum(1), Qs.shape[1] * rep * (w.Hkv if share else 1), rtol=1e-5)
    return got, want


def test_score_f32_config1():
    w = synth.config1()
    _score_check(w, w.Q, w.K)


# edges of the fp32 passes' 16-row tiles and of the wave turns over keys (256 per turn)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_qs,nk", [(1, 1), (15, 17), (16, 16), (17, 31), (33, 257), (130, 515)])
def test_score_f32_tile_edges(d, n_qs, nk):
    Q, K, _ = _attn_case("f32", 6, 2, n_qs, nk, d, n_qs + nk)
    w = synth.config1()
    w.Hq, w.Hkv, w.D = 6, 2, d
    _score_check(w, Q, K)
    lse = torch.from_numpy(orc.frame_attn(Q, K, K, d ** -0.5)[1].astype(np.float32)).to(DEV)
    _score_check(w, Q, K, share=True, lse=lse)


# 1 to 18 units of 16 scoring rows per KV head: 1 to 7 waves and all eight; rows of several heads in one
# unit (n_qs below 16 and just above it); rows picked by index, the log-sum-exp a view with a larger stride
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rep,n_qs", [(1, 1), (3, 5), (1, 17), (4, 9), (2, 31), (3, 37), (8, 25), (4, 72)])
def test_score_f32_few_scoring_rows(d, rep, n_qs):
    hkv, nk, nq = 2, 333, 3 * n_qs
    Q, K, _ = _attn_case("f32", rep * hkv, hkv, nq, nk, d, rep + n_qs)
    picked = np.arange(n_qs)[::-1] * 3 + 1
    scale = d ** -0.5
    lse_all = orc.frame_attn(Q, K, K, scale)[1].astype(np.float32)
    lse = torch.zeros((rep * hkv, nq + 7), dtype=torch.float32, device=DEV)
    lse[:, :nq] = torch.from_numpy(lse_all).to(DEV)
    rows = torch.from_numpy(picked.astype(np.int32)).to(DEV)
    want = orc.score(np.ascontiguousarray(Q[:, picked]), K, scale)
    for given in (None, lse[:, :nq]):
        got = host(pk.pc_score(dev(Q, None), dev(K, None), nk, scale, lse=given, q_rows=rows)).astype(np.float64)
        assert np.all(np.abs(got - want) <= 2e-7 + 2e-5 * want)      # as in _score_check


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("share", [False, True])
def test_score_bf16_midsize(share, fold):
    w = synth.midsize()
    Qs = w.Q[:, w.score_rows]
    _score_check(w, Qs, w.K, share=share, fold=fold)


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("n_qs,nk", [(1, 1), (33, 255), (64, 256), (65, 257), (130, 1300)])
def test_score_bf16_ragged(n_qs, nk, fold):
    w = synth.midsize(n_past=1)
    rng = np.random.default_rng(n_qs + nk)
    Qs = synth.to_bf16(rng.standard_normal((4, n_qs, 128)).astype(np.float32))
    K = synth.to_bf16(rng.standard_normal((2, nk, 128)).astype(np.float32))
    w.Hq, w.Hkv = 4, 2
    _score_check(w, Qs, K, fold=fold)


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step", [0.05, 0.6, 40.0])
def test_score_bf16_row_reference_is_refreshed(step, fold):
    # the row pass sums exp2 against a standing reference and redoes a half tile only when a
    # partial sum runs away: logits drifting, climbing and jumping along the key axis
    rng = np.random.default_rng(4)
    hq, hkv, n_qs, nk, d = 4, 2, 90, 1100, 128
    w = synth.midsize()
    Qs = rng.standard_normal((hq, n_qs, d)).astype(np.float32)
    K = rng.standard_normal((hkv, nk, d)).astype(np.float32) * 0.1
    Qs[..., 0] = 8.0
    K[..., 0] = (step * (np.arange(nk) // 32) / (8.0 * d ** -0.5))[None, :]
    Qs, K = synth.to_bf16(Qs), synth.to_bf16(K)
    scale = d ** -0.5
    if fold:
        Qs, scale = _fold(Qs, scale)
    got = host(pk.pc_score(dev(Qs, "bf16"), dev(K, "bf16"), nk, scale)).astype(np.float64)
    want = orc.score(Qs, K, scale)
    # fp32 exponents: a logit of magnitude L carries an absolute rounding error of about
    # L * 2^-23 in base-2 units twice over (the product c*s and the subtraction of the LSE)
    rel = max(2e-5, 4 * step * (nk // 32) * 1.4427 * 2.0 ** -23)
    assert np.all(np.abs(got - want) <= 2e-7 + rel * want), (np.abs(got - want) / (want + 1e-30)).max()


SCORE_ACROSS_HEADS = [(3, 1, 31, 33), (6, 2, 43, 257), (2, 1, 33, 65), (8, 2, 252, 1804), (16, 2, 20, 30000),
                      (16, 8, 600, 6000), (6, 2, 1100, 12000), (4, 2, 2100, 65000)]
SCORE_512_FEW_KEYS = [(16, 4, 3990, nk) for nk in (1, 33, 64, 65, 129, 300)]
SCORE_512_FEW_ROWS = [(2, 1, n, 60000) for n in (1, 30, 50, 96, 130)]


# Scoring rows numbered through the heads of a group (n_qs is no multiple of a tile, or smaller than
# one), both forms of either pass: the first three shapes have 64 stationary rows per work-group in
# both; the next two have 512 in the column pass, which forms the normalisers of its rows itself or
# finds them formed; then 512 in both, the last with more rows than it prepares at a time.  step:
# logits climb along the key axis, as above.  The reference is the softmax in 64 bits, on the GPU.
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step", [0.0, 0.6, 40.0])
@pytest.mark.parametrize("hq,hkv,n_qs,nk", SCORE_ACROSS_HEADS)
def test_score_bf16_rows_across_heads(hq, hkv, n_qs, nk, step, fold):
    Q, K, _ = _attn_case("bf16", hq, hkv, n_qs, nk, 128, n_qs + nk)
    scale = 128 ** -0.5
    if step:
        step *= min(1.0, 125 / (nk // 32))      # as steep as on 4,000 keys at most
        Q[..., 0] = 8.0
        K *= 0.1
        K[..., 0] = step * (np.arange(nk) // 32) / (8.0 * scale)
        Q, K = synth.to_bf16(Q), synth.to_bf16(K)
    if fold:
        Q, scale = _fold(Q, scale)
    Qd, Kd = dev(Q, "bf16"), dev(K, "bf16")
    want = torch.zeros((hkv, nk), dtype=torch.float64, device=DEV)
    lse = torch.empty((hq, n_qs), dtype=torch.float64, device=DEV)
    for h in range(hq):
        s = (Qd[h].double() @ Kd[h * hkv // hq].double().t()) * scale
        lse[h] = torch.logsumexp(s, dim=1)
        want[h * hkv // hq] += torch.softmax(s, dim=1).sum(0)
    # exponents of up to |logit| log2(e) are formed in fp32, twice (the product, the normaliser), and a
    # caller's normaliser arrives rounded to fp32 besides
    rel = max(2e-5, 6 * lse.abs().max().item() * 1.4427 * 2.0 ** -23)
    for given in (None, lse.float()):
        got = pk.pc_score(Qd, Kd, nk, scale, lse=given).double()
        assert ((got - want).abs() <= 2e-7 + rel * want).all(), ((got - want).abs() / (want + 1e-30)).max().item()


# The 512-row passes at their shortest: row pass with one to three key tiles per share, column pass with one
# to five tiles of scoring rows, and a last block with a single key
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("step", [0.0, 0.6])
@pytest.mark.parametrize("hq,hkv,n_qs,nk", SCORE_512_FEW_KEYS + SCORE_512_FEW_ROWS)
def test_score_bf16_short_512_row_passes(hq, hkv, n_qs, nk, step, fold):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n_qs + nk)
    Q, K = (torch.randn((h, n, 128), generator=gen, device=DEV) for h, n in ((hq, n_qs), (hkv, nk)))
    scale = 128 ** -0.5
    if step:
        Q[..., 0] = 8.0
        K *= 0.1
        K[..., 0] = step * min(1.0, 125 / max(1, nk // 32)) * (torch.arange(nk, device=DEV) // 32) / (8.0 * scale)
    if fold:
        Q, scale = Q * q_fold(scale), LN2
    Q, K = Q.bfloat16(), K.bfloat16()
    rows = torch.arange(n_qs, device=DEV)
    _, lse, want = _masked_reference(Q, K, K, torch.ones(nk, dtype=torch.bool, device=DEV), scale, rows)
    rel = max(2e-5, 6 * lse.abs().max().item() * 1.4427 * 2.0 ** -23)     # as in the test above
    for given in (None, lse.float()):
        got = pk.pc_score(Q, K, nk, scale, lse=given).double()
        assert ((got - want).abs() <= 2e-7 + rel * want).all(), ((got - want).abs() / (want + 1e-30)).max().item()


# one score for all heads of a call whose query rows are cut: heads in one and in two rounds of eight, the
# parts' and the heads' sums in their order
@pytest.mark.parametrize("hq,hkv,n,nk,begin", [(16, 1, 512, 700, 0), (16, 4, 512, 4600, 3), (8, 8, 2100, 513, 0), (12, 12, 2100, 700, 65)])
def test_score_shared_heads_are_the_heads_added_in_order(hq, hkv, n, nk, begin):
    assert pk.pc_score_cut(hq, hkv, n, nk, LN2, True, nk - begin)[3] > 1
    rng = np.random.default_rng(hq * nk)
    q, k = (dev(synth.to_bf16(rng.standard_normal(s).astype(np.float32)), "bf16") for s in ((hq, n, 128), (hkv, nk, 128)))
    lse = torch.full((hq, n), 20.0, dtype=torch.float32, device=DEV)
    per_head = host(pk.pc_score(q, k, nk, LN2, lse=lse, key_range=(begin, nk)))[:, begin:]
    got = host(pk.pc_score(q, k, nk, LN2, lse=lse, share_heads=True, key_range=(begin, nk)))[0, begin:]
    want = np.zeros(nk - begin, np.float32)
    for h in range(hkv):
        want = want + per_head[h]
    assert np.isfinite(want).all() and (want > 0).all()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("fold", [False, True])
def test_score_with_supplied_lse_matches_internal_pass(fold):
    w = synth.midsize()
    Qs = w.Q[:, w.score_rows]
    Qo, scale = _fold(Qs, w.scale) if fold else (Qs, w.scale)
    _, L = orc.frame_attn(Qo, w.K, w.V, scale)
    got, _ = _score_check(w, Qs, w.K, lse=dev(L.astype(np.float32), None), fold=fold)
    assert got.shape == (w.Hkv, w.Nk)


def test_score_reuses_the_lse_of_an_attention_pass_through_the_row_index():
    # the LSE that pc_frame_attn emits for ALL query rows feeds pc_score for the sampled rows:
    # one QK^T pass instead of two.  A row's probabilities scale by exp(-d_lse), so the score
    # error is the attention kernel's LSE error (fp32 online softmax, ~1e-6) relative.
    for w in (synth.midsize(), synth.config1()):
        Q, K, V = dev(w.Q, w.dtype), dev(w.K, w.dtype), dev(w.V, w.dtype)
        lse = torch.empty((w.Hq, w.Nq), dtype=torch.float32, device=DEV)
        pk.pc_frame_attn(Q, K, V, w.Nk, w.scale, lse=lse)
        rows = w.score_rows.astype(np.int32)
        got = host(pk.pc_score(Q, K, w.Nk, w.scale, q_rows=dev(rows, None), lse=lse)).astype(np.float64)
        want = orc.score(w.Q[:, rows], w.K, w.scale)
        err = np.abs(got - want)
        print("lse reuse", w.name, err.max(), (err / (want + 1e-30)).max())
        assert np.all(err <= 2e-7 + 5e-5 * want), (err.max(), (err / (want + 1e-30)).max())


def test_score_row_index_equals_gathered_rows():
    # scoring rows picked through q_rows must give the same bits as scoring a gathered copy
    for w in (synth.midsize(), synth.config1()):
        rows = w.score_rows[::2].astype(np.int32)
        Q, K = dev(w.Q, w.dtype), dev(w.K, w.dtype)
        a = pk.pc_score(Q, K, w.Nk, w.scale, q_rows=dev(rows, None))
        b = pk.pc_score(dev(w.Q[:, rows], w.dtype), K, w.Nk, w.scale)
        assert torch.equal(a, b)
        want = orc.score(w.Q[:, rows], w.K, w.scale)
        assert np.all(np.abs(host(a) - want) <= 2e-7 + 2e-5 * want)


@pytest.mark.parametrize("share", [False, True])
@pytest.mark.parametrize("case", ["mid", "c1"])
def test_score_key_range_scores_only_the_range(case, share):
    # keys outside the range count in every normaliser but get no score: inside, the bits of the
    # full call; outside, whatever the buffer held
    w = synth.midsize() if case == "mid" else synth.config1()
    Q, K = dev(w.Q, w.dtype), dev(w.K, w.dtype)
    rows = dev(w.score_rows.astype(np.int32), None)
    full = pk.pc_score(Q, K, w.Nk, w.scale, q_rows=rows, share_heads=share)
    for a, b in ((0, w.Nk), (w.segments[1][0], w.Nk), (w.segments[2][0] + 3, w.Nk - 5), (17, 18)):
        part = torch.full_like(full, -7.0)
        pk.pc_score(Q, K, w.Nk, w.scale, q_rows=rows, share_heads=share, score=part, key_range=(a, b))
        assert torch.equal(part[:, a:b], full[:, a:b]), (a, b)
        assert torch.all(part[:, :a] == -7.0) and torch.all(part[:, b:] == -7.0)


def test_score_is_bit_reproducible():
    w = synth.midsize()
    Qs, K = dev(w.Q[:, w.score_rows], "bf16"), dev(w.K, "bf16")
    a = pk.pc_score(Qs, K, w.Nk, w.scale)
    b = pk.pc_score(Qs, K, w.Nk, w.scale)
    assert torch.equal(a, b)


# ------------------------------------------------------------------------------- select + compact
def _compact_run(w, sc, budgets, in_place, share=False, hsel=None):
    dt = w.dtype
    hsel = (1 if share else w.Hkv) if hsel is None else hsel
    K, V = dev(w.K, dt), dev(w.V, dt)
    pos = dev(np.broadcast_to(w.pos_k[None], (hsel, w.Nk, 3)).copy(), None)
    scd = dev(sc.astype(np.float32), None)
    plan, nk_out = pk.pc_compact_plan(w.segments, budgets)
    idx = torch.full((hsel, nk_out), -1, dtype=torch.int32, device=DEV)
    if in_place:
        segs, nk = pk.pc_compact(K, V, pos, scd, w.segments, budgets, share_heads=share, idx=idx)
        Ko, Vo, po = K[:, :nk], V[:, :nk], pos[:, :nk]
    else:
        Ko = torch.empty((w.Hkv, nk_out, w.D), dtype=K.dtype, device=DEV)
        Vo, po = torch.empty_like(Ko), torch.empty((hsel, nk_out, 3), dtype=torch.int32, device=DEV)
        segs, nk = pk.pc_compact(K, V, pos, scd, w.segments, budgets, share_heads=share, out=(Ko, Vo, po), idx=idx)
        assert torch.equal(K, dev(w.K, dt))           # out of place leaves the cache alone
    assert segs == plan and nk == nk_out
    # the two halves one by one, on a workspace that holds anything: the two-launch form, which small whole calls leave
    Kt, Vt, pt = (t.clone()[None] for t in (dev(w.K, dt), dev(w.V, dt), dev(np.broadcast_to(w.pos_k[None], (hsel, w.Nk, 3)).copy(), None)))
    out = None if in_place else tuple(torch.empty_like(t)[None] for t in (Ko, Vo, po))
    ws = torch.full((pk.pc_compact_workspace_bytes(w.Hkv, w.Nk, share),), 0xA5, dtype=torch.uint8, device=DEV)
    idx_t = torch.full_like(idx, -1)[None]
    for phase in (pk.PC_COMPACT_SELECT, pk.PC_COMPACT_GATHER):
        assert pk.pc_compact_batch(Kt, Vt, pt, scd[None], w.segments, budgets, share_heads=share, out=out, idx=idx_t,
                                   ws=ws, phases=phase) == (segs, nk)
    if in_place:
        pk.pc_compact_status(ws)
    for t, x in zip((Ko, Vo, po, idx), (*(out or (Kt, Vt, pt)), idx_t)):
        assert torch.equal(x[0, :, :nk], t)
    return host(Ko), host(Vo), host(po), host(idx), segs


@pytest.mark.parametrize("grid,launches", [((12, 21), 1), ((32, 33), 2)])
def test_compact_status_reports_the_abort_word(grid, launches):
    """pc_compact_status is PC_OK after an ordinary in-place call; the abort word (set here from the
    host, never by making a kernel wait in vain) turns into PC_ERR_ABORTED; the next call resets it."""
    w = synth.midsize(gh=grid[0], gw=grid[1])
    assert pk.pc_compact_cut(1, w.Hkv, pk.PC_BF16, w.D, w.segments, budgets_for(w), False, True)[0] == launches
    sc = dev(np.random.default_rng(5).random((w.Hkv, w.Nk)).astype(np.float32), None)
    budgets = budgets_for(w)
    ws = torch.empty(pk.pc_compact_workspace_bytes(w.Hkv, w.Nk), dtype=torch.uint8, device=DEV)

    def run():
        K, V = dev(w.K, w.dtype), dev(w.V, w.dtype)
        pos = dev(np.broadcast_to(w.pos_k[None], (w.Hkv, w.Nk, 3)).copy(), None)
        pk.pc_compact(K, V, pos, sc, w.segments, budgets, ws=ws)

    run()
    pk.pc_compact_status(ws)
    ws[:4].view(torch.int32).fill_(1)
    with pytest.raises(pk.PackCacheError) as e:
        pk.pc_compact_status(ws)
    assert e.value.status == -8
    run()
    pk.pc_compact_status(ws)


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("case", ["c1", "mid", "mid_f32"])
def test_compact_matches_oracle_on_given_scores(case, in_place):
    w = synth.config1() if case == "c1" else synth.midsize(dtype="f32" if case == "mid_f32" else "bf16")
    rng = np.random.default_rng(3)
    sc = rng.random((w.Hkv, w.Nk)).astype(np.float32)       # fp32 scores given: selection is exact
    budgets = budgets_for(w)
    Kw, Vw, pw, iw, sw = orc.compact(w.K, w.V, np.broadcast_to(w.pos_k[None], (w.Hkv, w.Nk, 3)),
                                     sc, w.segments, budgets)
    Kg, Vg, pg, ig, sg = _compact_run(w, sc, budgets, in_place)
    assert np.array_equal(ig, iw) and sg == sw
    assert np.array_equal(Kg, Kw.astype(np.float32)) and np.array_equal(Vg, Vw.astype(np.float32))
    assert np.array_equal(pg, pw)


@pytest.mark.parametrize("in_place", [False, True])
def test_compact_ties_zero_budgets_and_share_heads(in_place):
    w = synth.midsize(n_past=5)
    rng = np.random.default_rng(9)
    sc = (rng.integers(0, 4, (1, w.Nk)) / 4.0).astype(np.float32)   # heavy ties
    sc[0, w.segments[3][0]:w.segments[3][0] + w.segments[3][1]] = 0.25   # one frame all equal
    budgets = [s[1] for s in w.segments]
    budgets[2], budgets[3], budgets[4], budgets[5], budgets[6] = 0, 17, 1, w.n_frame - 1, 64
    Kw, Vw, pw, iw, sw = orc.compact(w.K, w.V, w.pos_k[None], sc, w.segments, budgets, share_heads=True)
    Kg, Vg, pg, ig, sg = _compact_run(w, sc, budgets, in_place, share=True)
    assert np.array_equal(ig, iw) and sg == sw
    assert np.array_equal(Kg, Kw.astype(np.float32)) and np.array_equal(Vg, Vw.astype(np.float32))
    assert np.array_equal(pg, pw)


def test_compact_long_segment_generic_select_and_negative_zero():
    # a frame longer than the register-resident limit takes the generic select path
    rng = np.random.default_rng(21)
    n = 5000
    segs = [(0, 8, pk.PC_SEG_TEXT, -1), (8, n, pk.PC_SEG_FRAME, 1), (8 + n, 40, pk.PC_SEG_SELF, 2)]
    nk = 8 + n + 40
    sc = rng.random((1, nk)).astype(np.float32)
    sc[0, 8:8 + 600] = 0.0
    sc[0, 8:8 + 600:2] = -0.0                                   # -0 ties with +0
    K = rng.standard_normal((1, nk, 64)).astype(np.float32)
    V = rng.standard_normal((1, nk, 64)).astype(np.float32)
    pos = rng.integers(0, 100, (1, nk, 3)).astype(np.int32)
    budgets = [8, n - 300, 40]
    Kw, Vw, pw, iw, sw = orc.compact(K, V, pos, sc, segs, budgets)
    Kd, Vd, pd = dev(K, "f32"), dev(V, "f32"), dev(pos, None)
    idx = torch.empty((1, sw[-1][0] + sw[-1][1]), dtype=torch.int32, device=DEV)
    sg, nko = pk.pc_compact(Kd, Vd, pd, dev(sc, None), segs, budgets, idx=idx)
    assert sg == sw and np.array_equal(host(idx), iw)
    assert np.array_equal(host(Kd[:, :nko]), Kw) and np.array_equal(host(pd[:, :nko]), pw)


# segment lengths (the first is an anchor), D, dtype, KV heads, share_heads, launches out of place and in place
COMPACT_SMALL = [
    ([5, 1, 2, 3], 128, "bf16", 1, False, (1, 1)),                       # frames shorter than a wave
    ([16, 64, 63, 64, 65, 64], 64, "f32", 2, False, (1, 1)),             # around one row of 64 keys
    ([0, 1023, 1024, 7], 128, "bf16", 2, True, (1, 1)),                  # the longest segments the one-launch form takes
    ([0, 1023, 1025, 7], 128, "bf16", 2, False, (2, 2)),                 # one key more: two launches
    ([3] + [70] * 23, 128, "f32", 1, False, (1, 1)),                     # 24 segments: the short table, two rounds of waves
    ([3] + [70] * 24, 128, "bf16", 24, False, (1, 1)),                   # 25: the long table; many heads, wide slices
    ([0] + [130] * 16 + [0, 200], 128, "bf16", 2, False, (2, 1)),        # empty segments between others
    ([0] + [60] * 15 + [0, 70], 128, "bf16", 2, False, (1, 1)),          # the same out of place
    ([3] + [16] * 26, 128, "bf16", 2, False, (2, 1)),                    # a second round of pruned segments
    ([7700] + [1024] * 31, 64, "f32", 1, False, (2, 1)),                 # 8,192 kept rows, sources above 32,767
    ([7701] + [1024] * 31, 64, "f32", 1, False, (2, 2)),                 # one kept row more
    ([7], 128, "bf16", 2, False, (1, 1)),                                # nothing pruned: in place nothing moves
    ([90, 300, 400], 128, "bf16", 8, False, (1, 1)),                     # 8 heads: 64-byte slices out of place only
    ([30, 60, 70], 128, "bf16", 56, False, (1, 1)),                      # whole rows: halves would be 280 work-groups
    ([10, 20, 20], 128, "bf16", 150, False, (2, 2)),                     # many heads, one chunk of the gather each
    ([10, 200, 200], 128, "bf16", 150, True, (2, 1)),                    # and several
]


def small_table(lens):
    """Segments and budgets of a table of COMPACT_SMALL: every kind of budget by turns, few rows of the 31 long ones."""
    segs, at = [], 0
    for i, n in enumerate(lens):
        segs.append((at, n, pk.PC_SEG_TEXT if i == 0 else pk.PC_SEG_FRAME, i))
        at += n
    if len(lens) == 32:
        return segs, at, [lens[0]] + [0] * 3 + [113] * 4 + [40] + [0] * 23
    return segs, at, [n if i == 0 else (0, n, n // 3, max(1, n - 1), 1)[(i + 2) % 5] for i, n in enumerate(lens)]


# In place, frames that are dropped whole are not what a one-launch compaction is bounded by: most of 42 segments and
# all but the newest of 60 keep nothing; with two dropped of 42 the call takes two launches.
@pytest.mark.parametrize("n_seg,dropped,launches", [(42, 32, 1), (60, 58, 1), (42, 2, 2)])
def test_compact_in_place_with_frames_dropped_whole(n_seg, dropped, launches):
    lens = [9] + [120] * (n_seg - 1)
    segs = [(sum(lens[:i]), n, pk.PC_SEG_TEXT if i == 0 else pk.PC_SEG_FRAME, i) for i, n in enumerate(lens)]
    budgets = [9] + [0] * dropped + [17 + i % 3 for i in range(n_seg - 1 - dropped)]
    assert pk.pc_compact_cut(1, 2, pk.PC_BF16, 128, segs, budgets, False, True)[0] == launches
    rng = np.random.default_rng(n_seg)
    at = sum(lens)
    sc = np.round(np.exp(rng.standard_normal((2, at))) * 64).astype(np.float32) / 64     # with ties
    K, V = (orc.round_to_bf16(rng.standard_normal((2, at, 128))).astype(np.float32) for _ in range(2))
    pos = rng.integers(0, 10000, (2, at, 3)).astype(np.int32)
    Kw, Vw, pw, _, sw = orc.compact(K, V, pos, sc, segs, budgets)
    Kd, Vd, pd = dev(K, "bf16"), dev(V, "bf16"), dev(pos, None)
    table, nk = pk.pc_compact(Kd, Vd, pd, dev(sc, None), segs, budgets)
    assert table == sw and nk == sw[-1][0] + sw[-1][1]
    for got, want in ((Kd, Kw), (Vd, Vw), (pd, pw)):
        assert np.array_equal(host(got)[:, :nk], want)


# Up to sixteen kept frames are one round of the one launch's waves wherever they stand among dropped ones: sixteen
# apart they take as long as side by side (in one wave's turn they took three times as long).
@pytest.mark.parametrize("front", [1, 40])
def test_compact_in_place_with_kept_frames_far_apart(front):
    n_seg, Hkv = 113, 2
    lens = [9] + [64] * (n_seg - 1)
    segs = [(sum(lens[:i]), n, pk.PC_SEG_TEXT if i == 0 else pk.PC_SEG_FRAME, i) for i, n in enumerate(lens)]
    at = sum(lens)
    rng = np.random.default_rng(front)
    sc = np.round(np.exp(rng.standard_normal((Hkv, at))) * 64).astype(np.float32) / 64     # with ties
    K, V = (orc.round_to_bf16(rng.standard_normal((Hkv, at, 128))).astype(np.float32) for _ in range(2))
    pos = rng.integers(0, 10000, (Hkv, at, 3)).astype(np.int32)

    def budgets(kept):   # `front` segments are kept whole, then those of `kept`
        return [n if i < front else 20 if i in kept else 0 for i, n in enumerate(lens)]
    apart, together = budgets(range(front, n_seg, 16)), budgets(range(front, front + len(range(front, n_seg, 16))))
    micros = []
    for b in (apart, together):
        assert pk.pc_compact_cut(1, Hkv, pk.PC_BF16, 128, segs, b, False, True)[0] == 1
        Kw, Vw, pw, iw, sw = orc.compact(K, V, pos, sc, segs, b)
        nk = sw[-1][0] + sw[-1][1]
        for idx in (None, torch.full((Hkv, nk), -1, dtype=torch.int32, device=DEV)):
            Kd, Vd, pd, sd = dev(K, "bf16"), dev(V, "bf16"), dev(pos, None), dev(sc, None)
            assert pk.pc_compact(Kd, Vd, pd, sd, segs, b, idx=idx) == (sw, nk)
            for got, want in ((Kd, Kw), (Vd, Vw), (pd, pw)):
                assert np.array_equal(host(got)[:, :nk], want)
            assert idx is None or np.array_equal(host(idx), iw)
        ws = torch.empty(pk.pc_compact_workspace_bytes(Hkv, at), dtype=torch.uint8, device=DEV)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                pk.pc_compact(Kd, Vd, pd, sd, segs, b, ws=ws)
        times = []
        for _ in range(10):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            graph.replay()
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end) * 50)
        micros.append(min(times))
    assert micros[0] <= 1.5 * micros[1], micros


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("lens,D,dtype,Hkv,share,launches", COMPACT_SMALL)
def test_compact_small_caches_select_and_move_in_one_launch(lens, D, dtype, Hkv, share, launches, in_place):
    rng = np.random.default_rng(sum(lens) + Hkv)
    segs, at, budgets = small_table(lens)
    code = pk.PC_BF16 if dtype == "bf16" else pk.PC_F32
    assert pk.pc_compact_cut(1, Hkv, code, D, segs, budgets, share, in_place)[0] == launches[in_place]
    hsel = 1 if share else Hkv
    sc = np.round(np.exp(rng.standard_normal((hsel, at))) * 64).astype(np.float32) / 64     # with ties
    K, V = (orc.round_to_bf16(rng.standard_normal((Hkv, at, D))).astype(np.float32) for _ in range(2))
    pos = rng.integers(0, 10000, (hsel, at, 3)).astype(np.int32)
    Kw, Vw, pw, iw, sw = orc.compact(K, V, pos, sc, segs, budgets, share_heads=share)
    Kd, Vd, pd = dev(K, dtype), dev(V, dtype), dev(pos, None)
    nk = sw[-1][0] + sw[-1][1]
    idx = torch.full((hsel, nk), -1, dtype=torch.int32, device=DEV)
    out = None if in_place else (torch.empty_like(Kd), torch.empty_like(Vd), torch.empty_like(pd))
    sg, nko = pk.pc_compact(Kd, Vd, pd, dev(sc, None), segs, budgets, share_heads=share, out=out, idx=idx)
    Ko, Vo, po = out or (Kd, Vd, pd)
    assert sg == sw and nko == nk and np.array_equal(host(idx), iw)
    assert np.array_equal(host(Ko[:, :nk]), Kw) and np.array_equal(host(Vo[:, :nk]), Vw)
    assert np.array_equal(host(po[:, :nk]), pw)


@pytest.mark.parametrize("Hkv,n,n_frames,dtype", [(1, 64, 4, "f32"), (2, 252, 6, "bf16"), (8, 120, 3, "bf16"), (4, 1100, 3, "bf16")])
def test_in_place_compaction_of_one_buffer_passed_as_keys_and_values(Hkv, n, n_frames, dtype):
    # small caches (which take one launch where K and V are two buffers) and a large one
    rng = np.random.default_rng(Hkv * n)
    segs = [(0, 16, pk.PC_SEG_TEXT, -1)] + [(16 + n * f, n, pk.PC_SEG_FRAME, f + 1) for f in range(n_frames)]
    nk, budgets = 16 + n * n_frames, [16] + [n * (f + 1) // (n_frames + 1) for f in range(n_frames)]
    K, sc = (rng.standard_normal(s).astype(np.float32) for s in ((Hkv, nk, 128), (Hkv, nk)))
    K = orc.round_to_bf16(K).astype(np.float32)
    pos = rng.integers(0, 10000, (Hkv, nk, 3)).astype(np.int32)
    Kw, _, pw, _, sw = orc.compact(K, K, pos, sc, segs, budgets)
    Kd, pd = dev(K, dtype), dev(pos, None)
    sg, nko = pk.pc_compact(Kd, Kd, pd, dev(sc, None), segs, budgets)
    assert sg == sw and np.array_equal(host(Kd[:, :nko]), Kw) and np.array_equal(host(pd[:, :nko]), pw)


def test_in_place_compaction_repeated_random_budgets():
    # the in-place ordering protocol against the out-of-place result, many budget patterns (_compact_run takes
    # the two launches of the protocol as well as the one of such a small cache)
    w = synth.midsize(n_past=9, gh=16, gw=21, n_text=24)
    rng = np.random.default_rng(100)
    for trial in range(12):
        sc = rng.random((w.Hkv, w.Nk)).astype(np.float32)
        budgets = [s[1] if s[2] != pk.PC_SEG_FRAME else int(rng.integers(0, s[1] + 1)) for s in w.segments]
        if trial == 0:
            budgets = [s[1] for s in w.segments]                       # nothing moves
        if trial == 1:
            budgets = [s[1] if s[2] != pk.PC_SEG_FRAME else 1 for s in w.segments]
        a = _compact_run(w, sc, budgets, in_place=False)
        b = _compact_run(w, sc, budgets, in_place=True)
        for x, y in zip(a[:4], b[:4]):
            assert np.array_equal(x, y), f"trial {trial}"


# ------------------------------------------------------------------------------- whole path
def _chain(w, rope):
    dt = w.dtype
    Q, K, V = dev(w.Q, dt), dev(w.K, dt), dev(w.V, dt)
    pos = dev(np.broadcast_to(w.pos_k[None], (w.Hkv, w.Nk, 3)).copy(), None)
    Qo, Ko = w.Q.astype(np.float64), w.K.astype(np.float64)
    newest = w.segments[-1]
    if rope:   # a1: rotate the new frame's queries and the newest cached frame's keys
        pk.pc_rope3d(Q, dev(w.pos_q, None), w.sections, w.base)
        kn = K[:, newest[0]:newest[0] + newest[1]]
        pk.pc_rope3d(kn, dev(w.pos_k[newest[0]:newest[0] + newest[1]], None), w.sections, w.base)
        rnd = orc.round_to_bf16 if dt == "bf16" else (lambda a: a.astype(np.float32).astype(np.float64))
        Qo = rnd(orc.rope3d(w.Q, w.pos_q, w.sections, w.base))
        Ko = Ko.copy()
        Ko[:, newest[0]:newest[0] + newest[1]] = rnd(orc.rope3d(
            w.K[:, newest[0]:newest[0] + newest[1]], w.pos_k[newest[0]:newest[0] + newest[1]], w.sections, w.base))
    # where the device rotation rounded differently from the oracle's, scores legitimately differ
    q_same = np.array_equal(host(Q).astype(np.float64), Qo)
    k_diff_rows = np.any(host(K).astype(np.float64) != Ko, axis=2)          # [Hkv][Nk]
    rows = dev(w.score_rows.astype(np.int32), None)
    sc = pk.pc_score(Q, K, w.Nk, w.scale, q_rows=rows)                       # a2
    budgets = budgets_for(w)                                                # a3
    idx = torch.empty((w.Hkv, pk.pc_compact_plan(w.segments, budgets)[1]), dtype=torch.int32, device=DEV)
    segs, nk = pk.pc_compact(K, V, pos, sc, w.segments, budgets, idx=idx)    # a4 + a5, in place
    O = pk.pc_frame_attn(Q, K, V, nk, w.scale)                               # a6
    # oracle, step by step
    sco = orc.score(Qo[:, w.score_rows], Ko, w.scale)
    Kp, Vp, pp, io, so = orc.compact(Ko, w.V, np.broadcast_to(w.pos_k[None], (w.Hkv, w.Nk, 3)), sco,
                                     w.segments, budgets)
    assert segs == so
    ig = host(idx)
    # identical inputs: the 1e-6 band.  Keys rotated to a different bf16 are exempt; if any
    # query element rounded differently every score moves a little and the band is 1e-5.
    n_ex = check_selection(ig, sco, w.segments, budgets, band=BAND if q_same else 1e-5,
                           other_input=k_diff_rows if rope else None)
    assert np.array_equal(host(pos[:, :nk]), np.stack([w.pos_k[ig[h]] for h in range(w.Hkv)]))
    # attention over the keys the device actually kept (identical to the oracle's set up to
    # the exempted ties), computed by the oracle in fp64
    Kk = np.stack([Ko[g][ig[g]] for g in range(w.Hkv)])
    Vk = np.stack([w.V[g][ig[g]].astype(np.float64) for g in range(w.Hkv)])
    Ow, _ = orc.frame_attn(Qo, Kk, Vk, w.scale)
    err = np.abs(host(O).astype(np.float64) - Ow)
    return err, n_ex, (ig == io).mean()


def test_whole_path_config1_fp32():
    err, n_ex, same = _chain(synth.config1(), rope=False)
    assert err.max() <= 1e-5
    assert n_ex == 0 and same == 1.0


def test_whole_path_midsize_bf16_with_rope():
    err, n_ex, same = _chain(synth.midsize(), rope=True)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
    assert same > 0.99


def test_full_budget_packed_equals_dense_on_device():
    w = synth.midsize()
    Q, K, V = dev(w.Q, "bf16"), dev(w.K, "bf16"), dev(w.V, "bf16")
    O_dense = pk.pc_frame_attn(Q, K, V, w.Nk, w.scale)
    pos = dev(w.pos_k[None].repeat(w.Hkv, 0), None)
    sc = pk.pc_score(Q[:, :64].contiguous(), K, w.Nk, w.scale)
    segs, nk = pk.pc_compact(K, V, pos, sc, w.segments, [s[1] for s in w.segments])
    assert nk == w.Nk and segs == w.segments
    assert torch.equal(pk.pc_frame_attn(Q, K, V, nk, w.scale), O_dense)


@pytest.mark.parametrize("in_place", [False, True])
def test_cache_mask_in_front_of_the_select(in_place):
    # masked tokens are never kept and are physically removed, also from frames within budget
    w = synth.midsize()
    rng = np.random.default_rng(8)
    valid = rng.random(w.Nk) < 0.4
    sco = orc.score(w.Q[:, w.score_rows], w.K, w.scale)
    budgets = budgets_for(w)
    want = orc.compact(w.K, w.V, np.broadcast_to(w.pos_k[None], (w.Hkv, w.Nk, 3)), sco, w.segments, budgets,
                       valid=valid)
    mb = pk.pc_masked_budgets(w.segments, budgets, valid.astype(np.uint8))
    assert mb == orc.masked_budgets(w.segments, budgets, valid)
    sc = dev(sco.astype(np.float32), None)
    pk.pc_mask_scores(sc, dev(valid.astype(np.uint8), None))
    assert np.array_equal(host(sc) == -1.0, np.broadcast_to(~valid[None], sco.shape))
    Kp, Vp, pp, idx, segs = _compact_run(w, host(sc), mb, in_place)
    assert segs == want[4] and Kp.shape[1] == want[0].shape[1]
    # selection on the fp32 image of the oracle's scores: exact up to fp32 ties
    sel_sc = np.where(valid[None], sco.astype(np.float32).astype(np.float64), -1.0)
    check_selection(idx, sel_sc, w.segments, mb)
    for h in range(w.Hkv):
        assert np.all(valid[idx[h]] | (idx[h] < w.segments[2][0]))
        assert np.array_equal(Kp[h], w.K[h][idx[h]]) and np.array_equal(Vp[h], w.V[h][idx[h]])
        assert np.array_equal(pp[h], w.pos_k[idx[h]])


@pytest.mark.parametrize("share", [False, True])
@pytest.mark.parametrize("in_place", [False, True])
def test_compact_batch_equals_layer_by_layer_and_the_oracle(in_place, share):
    # a stack of layers re-packed in one call: same rows, bit for bit, as one call per layer
    ws_ = [synth.midsize(seed=30 + l) for l in range(3)]
    w = ws_[0]
    hsel = 1 if share else w.Hkv
    cap = w.Nk + 17                                              # spare capacity: strides differ from sizes
    K = torch.zeros((3, w.Hkv, cap, w.D), dtype=torch.bfloat16, device=DEV)
    V = torch.zeros_like(K)
    pos = torch.zeros((3, hsel, cap, 3), dtype=torch.int32, device=DEV)
    sc = torch.zeros((3, hsel, cap), dtype=torch.float32, device=DEV)
    sco = []
    for l, wl in enumerate(ws_):
        K[l, :, :w.Nk] = dev(wl.K, "bf16")
        V[l, :, :w.Nk] = dev(wl.V, "bf16")
        pos[l, :, :w.Nk] = dev(np.broadcast_to(wl.pos_k[None], (hsel, w.Nk, 3)).copy(), None)
        sco.append(orc.score(wl.Q[:, wl.score_rows], wl.K, wl.scale, share_heads=share))
        sc[l, :, :w.Nk] = dev(sco[-1].astype(np.float32), None)
    budgets = budgets_for(w)
    plan, nk_out = pk.pc_compact_plan(w.segments, budgets)
    idx = torch.full((3, hsel, nk_out), -1, dtype=torch.int32, device=DEV)
    ref = []
    for l in range(3):                                           # one call per layer, out of place
        Ko = torch.empty((w.Hkv, nk_out, w.D), dtype=K.dtype, device=DEV)
        Vo, po = torch.empty_like(Ko), torch.empty((hsel, nk_out, 3), dtype=torch.int32, device=DEV)
        io = torch.empty((hsel, nk_out), dtype=torch.int32, device=DEV)
        pk.pc_compact(K[l], V[l], pos[l], sc[l], w.segments, budgets, share_heads=share, out=(Ko, Vo, po), idx=io)
        ref.append((Ko, Vo, po, io))
    if in_place:
        segs, nk = pk.pc_compact_batch(K, V, pos, sc, w.segments, budgets, share_heads=share, idx=idx)
        Kb, Vb, pb = K[:, :, :nk], V[:, :, :nk], pos[:, :, :nk]
    else:
        Kb = torch.empty((3, w.Hkv, nk_out, w.D), dtype=K.dtype, device=DEV)
        Vb, pb = torch.empty_like(Kb), torch.empty((3, hsel, nk_out, 3), dtype=torch.int32, device=DEV)
        segs, nk = pk.pc_compact_batch(K, V, pos, sc, w.segments, budgets, share_heads=share, out=(Kb, Vb, pb), idx=idx)
    assert segs == plan and nk == nk_out
    for l in range(3):
        Ko, Vo, po, io = ref[l]
        assert torch.equal(idx[l], io) and torch.equal(Kb[l], Ko) and torch.equal(Vb[l], Vo) and torch.equal(pb[l], po)
        check_selection(host(idx[l]), sco[l].astype(np.float32).astype(np.float64), w.segments, budgets)


@pytest.mark.parametrize("in_place", [False, True])
def test_compact_batch_with_many_long_segments_takes_the_wave_per_segment_select(in_place):
    # 4 layers x 4 heads x 101 segments = 1,616 selections in one call, the longest 4,096 rows:
    # the stack form of the select (one wave per segment).  Given fp32 scores, so the kept sets
    # are exact: ragged and 64-aligned lengths, heavy ties, an all-equal frame, -0 against +0,
    # negative and -inf scores, budgets 0, 1, len - 1 and len.
    rng = np.random.default_rng(77)
    L, Hkv, D = 4, 4, 128
    lens = [int(v) for v in rng.integers(1025, 2300, 100)]
    lens[0], lens[1], lens[2], lens[3], lens[4] = 4096, 4032, 1088, 1025, 2047
    segs, at = [(0, 24, pk.PC_SEG_TEXT, -1)], 24
    for f, n in enumerate(lens):
        segs.append((at, n, pk.PC_SEG_FRAME, f))
        at += n
    nk = at
    budgets = [24] + [int(rng.integers(1, n)) for n in lens]
    budgets[1], budgets[2], budgets[3], budgets[4], budgets[5] = 4095, 1, 0, 1024, 2047   # the last: nothing pruned
    budgets[6] = lens[5] + 7                                      # beyond the length: kept whole
    sc = rng.standard_normal((L, Hkv, nk)).astype(np.float32)
    sc[0] = np.exp(sc[0] * 1.5 - 6)                               # column-mass-like, one shared exponent range
    sc[1] = (rng.integers(0, 5, (Hkv, nk)) / 4.0).astype(np.float32)      # heavy ties
    s7 = segs[7]
    sc[2, :, s7[0]:s7[0] + s7[1]] = 0.125                         # one frame all equal
    s8 = segs[8]
    sc[2, :, s8[0]:s8[0] + 600] = 0.0
    sc[2, :, s8[0]:s8[0] + 600:2] = -0.0                          # -0 ties with +0
    s9 = segs[9]
    sc[3, :, s9[0]:s9[0] + s9[1]:3] = -np.inf                     # masked-style scores
    K = torch.randn((L, Hkv, nk, D), dtype=torch.bfloat16, device=DEV)
    V = torch.randn_like(K)
    pos = torch.randint(0, 1000, (L, Hkv, nk, 3), dtype=torch.int32, device=DEV)
    scd = dev(sc, None)
    plan, nk_out = pk.pc_compact_plan(segs, budgets)
    assert plan == orc.packed_segments(segs, budgets)
    idx = torch.full((L, Hkv, nk_out), -1, dtype=torch.int32, device=DEV)
    ref = []
    for l in range(L):                                            # one call per layer (the work-group form), out of place
        Ko = torch.empty((Hkv, nk_out, D), dtype=K.dtype, device=DEV)
        Vo, po = torch.empty_like(Ko), torch.empty((Hkv, nk_out, 3), dtype=torch.int32, device=DEV)
        io = torch.empty((Hkv, nk_out), dtype=torch.int32, device=DEV)
        pk.pc_compact(K[l], V[l], pos[l], scd[l], segs, budgets, out=(Ko, Vo, po), idx=io)
        ref.append((Ko, Vo, po, io))
    if in_place:
        segs_out, nko = pk.pc_compact_batch(K, V, pos, scd, segs, budgets, idx=idx)
        Kb, Vb, pb = K[:, :, :nko], V[:, :, :nko], pos[:, :, :nko]
    else:
        Kb = torch.empty((L, Hkv, nk_out, D), dtype=K.dtype, device=DEV)
        Vb, pb = torch.empty_like(Kb), torch.empty((L, Hkv, nk_out, 3), dtype=torch.int32, device=DEV)
        segs_out, nko = pk.pc_compact_batch(K, V, pos, scd, segs, budgets, out=(Kb, Vb, pb), idx=idx)
    assert segs_out == plan and nko == nk_out
    ig = host(idx)
    for l in range(L):
        for h in range(Hkv):
            want = np.concatenate([
                np.arange(s, s + n) if kind != pk.PC_SEG_FRAME else s + orc.select_topk(sc[l, h, s:s + n], min(n, b))
                for (s, n, kind, _), b in zip(segs, budgets)])
            assert np.array_equal(ig[l, h], want), (l, h)
        Ko, Vo, po, io = ref[l]
        assert torch.equal(idx[l], io) and torch.equal(Kb[l], Ko) and torch.equal(Vb[l], Vo) and torch.equal(pb[l], po)


@pytest.mark.parametrize("in_place", [False, True])
def test_select_and_gather_as_two_calls_on_two_streams(in_place):
    # the select half on a side stream, the gather half on the main stream behind an event:
    # same result, bit for bit, as the single call
    w = synth.midsize()
    sco = orc.score(w.Q[:, w.score_rows], w.K, w.scale)
    budgets = budgets_for(w)
    ref = _compact_run(w, sco, budgets, in_place)
    K, V = dev(w.K, "bf16"), dev(w.V, "bf16")
    pos = dev(np.broadcast_to(w.pos_k[None], (w.Hkv, w.Nk, 3)).copy(), None)
    sc = dev(sco.astype(np.float32), None)
    plan, nk = pk.pc_compact_plan(w.segments, budgets)
    idx = torch.full((w.Hkv, nk), -1, dtype=torch.int32, device=DEV)
    ws = torch.empty(pk.pc_compact_workspace_bytes(w.Hkv, w.Nk), dtype=torch.uint8, device=DEV)
    if in_place:
        out, (Ko, Vo, po) = None, (K, V, pos)
    else:
        Ko = torch.empty((w.Hkv, nk, w.D), dtype=K.dtype, device=DEV)
        Vo, po = torch.empty_like(Ko), torch.empty((w.Hkv, nk, 3), dtype=torch.int32, device=DEV)
        out = (Ko, Vo, po)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    select = pk.pc_compact_prepared(K, V, pos, sc, w.segments, budgets, ws, out=out, idx=idx,
                                    phases=pk.PC_COMPACT_SELECT, stream=side)
    gather = pk.pc_compact_prepared(K, V, pos, sc, w.segments, budgets, ws, out=out, idx=idx,
                                    phases=pk.PC_COMPACT_GATHER)
    select()
    done = torch.cuda.Event()
    done.record(side)
    torch.cuda.current_stream().wait_event(done)
    gather()
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ref[3])
    assert np.array_equal(host(Ko[:, :nk]), ref[0]) and np.array_equal(host(Vo[:, :nk]), ref[1])
    assert np.array_equal(host(po[:, :nk]), ref[2])


def test_batch_halves_on_two_streams_equal_the_single_batched_call():
    # a stack of three layers: select half on a side stream, gather half on the main stream
    w = synth.midsize()
    L = 3
    rng = np.random.default_rng(21)
    K = torch.stack([dev(synth.to_bf16(rng.standard_normal(w.K.shape).astype(np.float32)), "bf16") for _ in range(L)])
    V = torch.stack([dev(synth.to_bf16(rng.standard_normal(w.V.shape).astype(np.float32)), "bf16") for _ in range(L)])
    pos = dev(np.broadcast_to(w.pos_k[None, None], (L, w.Hkv, w.Nk, 3)).copy(), None)
    sc = torch.rand((L, w.Hkv, w.Nk), device=DEV)
    budgets = budgets_for(w)
    K1, V1, p1 = K.clone(), V.clone(), pos.clone()
    segs1, nk1 = pk.pc_compact_batch(K1, V1, p1, sc, w.segments, budgets)
    ws = torch.empty(pk.pc_compact_batch_workspace_bytes(L, w.Hkv, w.Nk), dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    pk.pc_compact_batch(K, V, pos, sc, w.segments, budgets, ws=ws, phases=pk.PC_COMPACT_SELECT, stream=side)
    done = torch.cuda.Event()
    done.record(side)
    torch.cuda.current_stream().wait_event(done)
    segs2, nk2 = pk.pc_compact_batch(K, V, pos, sc, w.segments, budgets, ws=ws, phases=pk.PC_COMPACT_GATHER)
    torch.cuda.synchronize()
    assert segs1 == segs2 and nk1 == nk2
    assert torch.equal(K[:, :, :nk1], K1[:, :, :nk1]) and torch.equal(V[:, :, :nk1], V1[:, :, :nk1])
    assert torch.equal(pos[:, :, :nk1], p1[:, :, :nk1])


def test_random_shapes_attention_score_compaction():
    # a seeded walk over ragged shapes and head groupings: every call against the oracle
    rng = np.random.default_rng(2024)
    for it in range(24):
        hkv = int(rng.choice([1, 2, 3]))
        hq = hkv * int(rng.choice([1, 2, 4]))
        nq, nk = int(rng.integers(1, 400)), int(rng.integers(1, 1500))
        Q = synth.to_bf16(rng.standard_normal((hq, nq, 128)).astype(np.float32))
        K = synth.to_bf16(rng.standard_normal((hkv, nk, 128)).astype(np.float32))
        V = synth.to_bf16(rng.standard_normal((hkv, nk, 128)).astype(np.float32))
        scale = 128 ** -0.5
        _attn_check("bf16", Q, K, V, scale)
        n_qs = int(rng.integers(1, min(nq, 200) + 1))
        rows = np.sort(rng.choice(nq, size=n_qs, replace=False)).astype(np.int32)
        sc = pk.pc_score(dev(Q, "bf16"), dev(K, "bf16"), nk, scale, q_rows=dev(rows, None))
        want = orc.score(Q[:, rows], K, scale)
        assert np.all(np.abs(host(sc) - want) <= 2e-7 + 2e-5 * want), (it, hq, hkv, nq, nk)
        # a random segment table over the keys: [text | frames...], random budgets
        n_text = int(rng.integers(0, min(nk, 40) + 1))
        n_cuts = min(int(rng.integers(0, 6)), nk - n_text)
        cuts = np.sort(rng.choice(np.arange(n_text, nk + 1), size=n_cuts, replace=False))
        bounds = [n_text] + [int(c) for c in cuts] + [nk]
        segs = [(0, n_text, pk.PC_SEG_TEXT, -1)] + [(a, b - a, pk.PC_SEG_FRAME, f + 1)
                                                    for f, (a, b) in enumerate(zip(bounds[:-1], bounds[1:]))]
        budgets = [n_text] + [int(rng.integers(0, s[1] + 2)) for s in segs[1:]]
        pos = np.broadcast_to(np.arange(nk, dtype=np.int32)[None, :, None], (hkv, nk, 3)).copy()
        Kd, Vd, pd = dev(K, "bf16"), dev(V, "bf16"), dev(pos, None)
        plan, nk_out = pk.pc_compact_plan(segs, budgets)
        idx = torch.full((hkv, max(nk_out, 1)), -1, dtype=torch.int32, device=DEV)
        segs_out, nk2 = pk.pc_compact(Kd, Vd, pd, sc, segs, budgets, idx=idx)
        assert segs_out == plan == orc.packed_segments(segs, budgets) and nk2 == nk_out
        if nk_out:
            ig = host(idx)[:, :nk_out]
            check_selection(ig, host(sc).astype(np.float64), segs, budgets, band=0.0)   # exact on the device's own scores
            for h in range(hkv):
                assert np.array_equal(host(Kd[h, :nk_out]), K[h][ig[h]]) and np.array_equal(host(Vd[h, :nk_out]), V[h][ig[h]])
                assert np.array_equal(host(pd[h, :nk_out]), pos[h][ig[h]])


def test_random_segment_tables_batched_in_and_out_of_place():
    # random cache sizes (up to 40k rows), segment tables (also segments longer than the
    # register-resident select handles), budgets, layer counts, tie-heavy scores, both selection
    # granularities: kept sets against a full sort, moved rows bit for bit, in place == out of place
    for it in range(12):
        rng = np.random.default_rng(7000 + it)
        hkv, L = int(rng.choice([1, 2, 4])), int(rng.choice([1, 2, 3]))
        nk = int(rng.integers(1, 40000))
        n_text = int(rng.integers(0, min(nk, 300) + 1))
        n_cuts = min(int(rng.integers(0, 40)), nk - n_text)
        cuts = np.sort(rng.choice(np.arange(n_text, nk + 1), size=n_cuts, replace=False))
        bounds = [n_text] + [int(c) for c in cuts] + [nk]
        segs = [(0, n_text, pk.PC_SEG_TEXT, -1)] + [(a, b - a, pk.PC_SEG_FRAME, f + 1)
                                                    for f, (a, b) in enumerate(zip(bounds[:-1], bounds[1:]))]
        frac = float(rng.choice([0.05, 0.3, 0.7, 0.95, 1.0]))
        budgets = [n_text] + [int(min(s[1], max(0, round(s[1] * frac) + int(rng.integers(-2, 3))))) for s in segs[1:]]
        share = bool(rng.integers(0, 2))
        hsel = 1 if share else hkv
        g = torch.Generator(device=DEV)
        g.manual_seed(7000 + it)
        K = torch.randn((L, hkv, nk, 128), device=DEV, generator=g).to(torch.bfloat16)
        V = torch.randn((L, hkv, nk, 128), device=DEV, generator=g).to(torch.bfloat16)
        pos = torch.randint(0, 1000, (L, hsel, nk, 3), device=DEV, generator=g, dtype=torch.int32)
        sc = torch.rand((L, hsel, nk), device=DEV, generator=g)
        if it % 2:
            sc = (sc * 8).floor() / 8                             # many equal scores
        plan, nko = pk.pc_compact_plan(segs, budgets)
        if nko == 0:
            continue
        Ko = torch.empty((L, hkv, nko, 128), dtype=K.dtype, device=DEV)
        Vo = torch.empty_like(Ko)
        po = torch.empty((L, hsel, nko, 3), dtype=torch.int32, device=DEV)
        io = torch.empty((L, hsel, nko), dtype=torch.int32, device=DEV)
        pk.pc_compact_batch(K, V, pos, sc, segs, budgets, share_heads=share, out=(Ko, Vo, po), idx=io)
        sch, ioh = host(sc).astype(np.float64), host(io)
        for l in range(L):
            check_selection(ioh[l], sch[l], segs, budgets, band=0.0)
            for h in range(hkv):
                sel = io[l, 0 if share else h].long()
                assert torch.equal(Ko[l, h], K[l, h].index_select(0, sel)), (it, l, h)
                assert torch.equal(Vo[l, h], V[l, h].index_select(0, sel)), (it, l, h)
            for h in range(hsel):
                assert torch.equal(po[l, h], pos[l, h].index_select(0, io[l, h].long()))
        i2 = torch.empty_like(io)
        pk.pc_compact_batch(K, V, pos, sc, segs, budgets, share_heads=share, idx=i2)
        assert torch.equal(i2, io) and torch.equal(K[:, :, :nko], Ko) and torch.equal(V[:, :, :nko], Vo)
        assert torch.equal(pos[:, :, :nko], po), it


def test_step_captured_in_a_hip_graph_replays_to_the_eager_result():
    """The whole step (restore, a1..a6, compaction in place, key shares in the attention) recorded
    into a HIP graph on a side stream and replayed several times, with eager work and
    synchronisations in between: every replay must give the eager run's bits (the kernels are
    deterministic, nothing in the calls allocates or synchronises when workspaces are passed, and
    the in-place bookkeeping is cleared by a kernel, not by a memset node)."""
    w = synth.midsize(n_past=14, gamma=0.95)     # 2,740 keys stay: the attention cuts them into two shares
    dt = w.dtype
    Q0, K0, V0 = dev(w.Q, dt), dev(w.K, dt), dev(w.V, dt)
    pos0 = dev(np.broadcast_to(w.pos_k[None], (w.Hkv, w.Nk, 3)).copy(), None)
    Q, K, V, pos = Q0.clone(), K0.clone(), V0.clone(), pos0.clone()
    pos_q, newest = dev(w.pos_q, None), w.segments[-1]
    pos_new = dev(w.pos_k[newest[0]:newest[0] + newest[1]], None)
    rows = dev(w.score_rows.astype(np.int32), None)
    budgets = budgets_for(w)
    nk_out = pk.pc_compact_plan(w.segments, budgets)[1]
    assert pk.pc_compact_cut(1, w.Hkv, pk.PC_BF16, w.D, w.segments, budgets, False, True)[0] == 2   # the bookkeeping's form
    sc = torch.empty((w.Hkv, w.Nk), dtype=torch.float32, device=DEV)
    O, lse = torch.empty_like(Q), torch.empty((w.Hq, w.Nq), dtype=torch.float32, device=DEV)
    ws_s = torch.empty(pk.pc_score_workspace_bytes(w.Hq, w.Hkv, rows.numel(), w.Nk), dtype=torch.uint8, device=DEV)
    ws_c = torch.empty(pk.pc_compact_workspace_bytes(w.Hkv, w.Nk), dtype=torch.uint8, device=DEV)
    n_ws_a = pk.pc_frame_attn_workspace_bytes(w.Hq, w.Nq, nk_out, w.D)
    assert n_ws_a > 0, "this shape is meant to take the key-share path"
    ws_a = torch.empty(n_ws_a, dtype=torch.uint8, device=DEV)

    def step():
        Q.copy_(Q0), K.copy_(K0), V.copy_(V0), pos.copy_(pos0)
        pk.pc_rope3d(Q, pos_q, w.sections, w.base)
        pk.pc_rope3d(K[:, newest[0]:newest[0] + newest[1]], pos_new, w.sections, w.base)
        pk.pc_score(Q, K, w.Nk, w.scale, score=sc, ws=ws_s, q_rows=rows)
        segs, nk = pk.pc_compact(K, V, pos, sc, w.segments, budgets, ws=ws_c)
        assert nk == nk_out
        pk.pc_frame_attn(Q, K, V, nk, w.scale, O=O, lse=lse, ws=ws_a)

    step()                                   # eager; also the first-use set-up of every kernel
    torch.cuda.synchronize()
    want = [t.clone() for t in (O, lse, K[:, :nk_out], V[:, :nk_out], pos[:, :nk_out], sc)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for replay in range(4):
        for t in (O, lse, sc):               # eager work between the replays: scribble on the outputs
            t.fill_(float(replay + 7))
        K.zero_(), pos.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = (O, lse, K[:, :nk_out], V[:, :nk_out], pos[:, :nk_out], sc)
        for i, (g, x) in enumerate(zip(got, want)):
            assert torch.equal(g, x), f"replay {replay}: output {i} differs from the eager run"
    pk.pc_compact_status(ws_c)


def _marshalled_calls():
    """Every call that the compiled half of the binding takes, as (name, call); a call makes its own outputs."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(4)
    rand = lambda *shape: torch.randn(shape, device=DEV, generator=gen).to(torch.bfloat16)
    Q, K, V = rand(4, 40, 128), rand(2, 90, 128), rand(2, 90, 128)
    pos_q = torch.randint(0, 500, (40, 3), dtype=torch.int32, device=DEV, generator=gen)
    pos = torch.randint(0, 500, (2, 90, 3), dtype=torch.int32, device=DEV, generator=gen)
    sc = torch.rand((2, 90), device=DEV, generator=gen)
    rows = torch.arange(0, 40, 3, dtype=torch.int32, device=DEV)
    segs, budgets = [(0, 10, pk.PC_SEG_TEXT, -1), (10, 50, pk.PC_SEG_FRAME, 1), (60, 25, pk.PC_SEG_FRAME, 2)], [10, 20, 25]
    empty = lambda n: torch.empty(n, dtype=torch.uint8, device=DEV)

    def rope(x=None, sections=(32, 48, 48)):
        x = Q.clone() if x is None else x
        return pk.pc_rope3d(x, pos_q, sections, 1e4, out_scale=2), x

    def score(K=K, **kw):
        out = torch.zeros((2, 90), device=DEV)
        r = pk.pc_score(Q, K, 90, 0.1, score=out, ws=empty(pk.pc_score_workspace_bytes(4, 2, 14, 90)), q_rows=rows,
                        key_range=(10, 85), **kw)
        return r is out, out

    def compact(K=K, budgets=budgets, **kw):
        k, v, p = K.clone(), V.clone(), pos.clone()
        r = pk.pc_compact(k, v, p, sc, segs, budgets, ws=empty(pk.pc_compact_workspace_bytes(2, 85)), **kw)
        return r, k[:, :r[1]], v[:, :r[1]], p[:, :r[1]]

    def batch(idx=True, **kw):
        k, v, p, s = (torch.stack([t, t.flip(0)]) for t in (K, V, pos, sc))
        i = torch.zeros((2, 2, 55), dtype=torch.int32, device=DEV)
        r = pk.pc_compact_batch(k, v, p, s, segs, budgets, idx=i, ws=empty(pk.pc_compact_batch_workspace_bytes(2, 2, 85)), **kw)
        return r, k[:, :, :r[1]], v[:, :, :r[1]], p[:, :, :r[1]], i

    def attn(Q=Q, V=V, **kw):
        O, lse = torch.zeros_like(Q), torch.zeros(Q.shape[:2], device=DEV)
        r = pk.pc_frame_attn(Q, K, V, 85, 0.1, O=O, lse=lse, **kw)
        return r is O, O, lse

    # out of place: a destination of another capacity, and (batch) one whose layers lie apart and heads close together
    def compact_out(K=K, room=60):
        out = tuple(torch.full((2, room, n), 7, dtype=t.dtype, device=DEV) for t, n in ((K, 128), (V, 128), (pos, 3)))
        i = torch.zeros((2, 64), dtype=torch.int32, device=DEV)[:, :60]
        r = pk.pc_compact(K, V, pos, sc, segs, budgets, out=out, idx=i, ws=empty(pk.pc_compact_workspace_bytes(2, 85)))
        return r, *out, i

    def batch_out(share=False, long=1):
        Kb, Vb, pb, sb = (torch.cat([torch.stack([t, t.flip(0)])] * long, dim=2) for t in (K, V, pos, sc))
        sel = 1 if share else 2
        pb, sb = pb[:, :sel], sb[:, :sel]
        out = tuple(torch.full((2, 3, 70 * long, n), 7, dtype=t.dtype, device=DEV)[:, :h] for t, n, h in ((K, 128, 2), (V, 128, 2), (pos, 3, sel)))
        table = [(85 * j + a, n, kind, f) for j in range(long) for a, n, kind, f in segs]
        assert pk.pc_compact_cut(2, 2, pk.PC_BF16, 128, table, budgets * long, share)[0] == (1 if long == 1 else 2)
        r = pk.pc_compact_batch(Kb, Vb, pb, sb, table, budgets * long, share_heads=share, out=out,
                                ws=empty(pk.pc_compact_batch_workspace_bytes(2, 2, 85 * long, share)))
        return r, *out

    def batch_short(lead):
        Kb, Vb, pb, sb = (torch.stack([t, t.flip(0)]) for t in (K, V, pos, sc))
        Ko, Vo, po = Kb.clone(), Vb.clone(), pb.clone()
        return pk.pc_compact_batch(Kb, Vb, pb, sb, segs, budgets, out=lead(Ko, Vo, po),
                                   ws=empty(pk.pc_compact_batch_workspace_bytes(2, 2, 85)))

    calls = {"rope3d": rope, "score": score, "compact": compact, "compact_batch": batch, "frame_attn": attn,
             "compact out": compact_out, "compact_batch out": batch_out, "compact_batch out, one selection": lambda: batch_out(share=True),
             "compact_batch out, two launches": lambda: batch_out(long=30)}
    refused = [lambda: rope(sections=(32, 48, 40)), lambda: rope(x=Q.transpose(0, 1)), lambda: score(K=K[..., :64]),
               lambda: compact(K=K.to(torch.float16)), lambda: compact(budgets=[10, -1, 25]),
               lambda: compact(out=(K.clone(), V.clone()[:, :80], pos.clone())), lambda: batch(share_heads=True),
               lambda: attn(V=torch.cat([V, V], dim=1)), lambda: compact_out(room=30),
               lambda: batch_short(lambda a, b, c: (a, b[:, :, :80], c)), lambda: batch_short(lambda a, b, c: (a, b.transpose(0, 1), c)),
               lambda: batch_short(lambda a, b, c: (a, b, c[:, :1])), lambda: batch_short(lambda a, b, c: (a[..., :64], b[..., :64], c))]
    return calls, refused


def test_plain_calls_are_marshalled_alike_by_both_halves_of_the_binding(monkeypatch):
    from paper_2601_04359_amd import binding
    calls, refused = _marshalled_calls()
    pk.pc_budget(pk.PC_BUDGET_POW, 10, 1, 0.5, 0)
    native, seen = binding._NATIVE, []
    assert native

    class Spy:
        def __getattr__(self, name):
            f = getattr(native, name)
            return lambda *a: seen.append((name, f(*a))) or seen[-1][1]

    def outcome(call):
        try:
            return call()
        except pk.PackCacheError as e:
            return e.status, str(e)

    same = lambda a, b: torch.equal(a, b) if torch.is_tensor(a) else a == b
    assert len(calls) == 9
    for name, call in [*calls.items(), *((None, r) for r in refused)]:
        seen.clear()
        monkeypatch.setattr(binding, "_NATIVE", Spy())
        got = outcome(call)
        assert name is None or any(n == name.split()[0] and r is not None for n, r in seen)   # no fallback for a plain call
        monkeypatch.setattr(binding, "_NATIVE", False)
        want = outcome(call)
        assert len(got) == len(want) and all(same(a, b) for a, b in zip(got, want)), (name, got, want)
        assert name is not None or isinstance(want[0], int)


def test_an_exception_inside_the_library_comes_back_as_a_python_error(monkeypatch):
    """No entry point of the library throws; a C++ function that does stands in for one (host code: nothing is
    launched).  The interpreter's lock is back when the error is made, in every call that gives it up."""
    import ctypes
    from paper_2601_04359_amd import binding
    calls, _ = _marshalled_calls()
    L = pk.lib()
    throws = ctypes.cast(ctypes.CDLL("libstdc++.so.6")._ZSt17__throw_bad_allocv, ctypes.c_void_p).value
    size = ctypes.cast(L.pc_frame_attn_workspace_bytes_for, ctypes.c_void_p).value
    try:
        binding._NATIVE.bind(*[throws] * 5, size, throws, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
        for name, call in calls.items():
            with pytest.raises(RuntimeError, match="bad_alloc"):
                call()
    finally:
        binding._bind_native(L)
    for call in calls.values():
        call()


def test_cache_views_are_the_same_from_both_halves_of_the_binding(monkeypatch):
    from paper_2601_04359_amd import binding
    pk.pc_budget(pk.PC_BUDGET_POW, 10, 1, 0.5, 0)
    native = binding._NATIVE
    layer = tuple(torch.zeros((2, 50, n), dtype=t, device=DEV) for n, t in ((128, torch.bfloat16), (128, torch.bfloat16), (3, torch.int32)))
    stack = tuple(torch.zeros((3, 2, 50, n), device=DEV) for n in (128, 128, 3))
    shape = lambda views: [(v.data_ptr(), tuple(v.shape), v.stride()) for v in views]
    for caches, dim in ((layer, 1), (stack, 2)):
        for start, n in ((0, 50), (0, 1), (17, 9), (49, 1), (17, 33), (50, 0), (3, 0), (17, 34), (50, 4), (60, 2)):   # to the end and past it
            monkeypatch.setattr(binding, "_NATIVE", native)
            views = binding._rows(*caches, dim, start, n)
            assert (native.rows(*caches, dim, start, n) is None) == (start + n > 50)
            monkeypatch.setattr(binding, "_NATIVE", False)
            assert shape(views) == shape(binding._rows(*caches, dim, start, n)), (dim, start, n)
