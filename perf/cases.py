"""Timed cases of the PackCache hot path, as a program that uses this package calls it.

What such a program does with the package falls into six kinds of work, and a case is one of them:

  roll     one frame step of one layer through rollout.RollingLayer: the newest frame is written
           into the cache and rotated, the step's queries are rotated, the cache is scored and
           re-packed in place, the queries attend over it (with `window`: the sliding window moves
           on and the retained rows are rebased first)
  oneshot  the same calls made one by one over a FULL cache, packed out of place (the sweep over
           frame indices, and the default step of bench.py)
  stack    one frame step of several layers through rollout.RollingStack: attention first, its
           log-sum-exp feeds the scores, one batched re-pack at the end
  attn     pc_frame_attn alone (iterative decoding: many passes per frame over one cache)
  score    pc_score alone, with or without the log-sum-exp of an attention pass
  compact  pc_compact / pc_compact_batch alone on given scores, in place or out of place

Sizes are those of the repository's configurations, tests and bench.py (tiny fp32 case, the
252-token "midsize" frames, 48 x 84-token frames with 16/4 and 24/8 heads, frames 24 and 48, 28
layers), and a half-resolution frame of 24 x 42 tokens between them.

    python -c "import perf.cases as c; print(*c.listed(), sep='\\n')"
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2601_04359_amd as pk
from paper_2601_04359_amd import synth
from paper_2601_04359_amd.rollout import RollingLayer, RollingStack

DEV = "cuda:0"
SECTIONS = {64: (16, 24, 24), 128: (32, 48, 48)}
BASE = 10000.0


# ------------------------------------------------------------------------------ the cases
def listed() -> list[dict]:
    return [
        # the smallest layer in use (fp32, 64-token frames): launches and host time are all there is
        dict(name="tiny_roll_f32", kind="roll", dtype="f32", Hq=2, Hkv=1, D=64, n=64, n_text=16, n_past=4,
             mode="pow", gamma=0.7, b_min=8, n_score=64, fold=False, share=False, window=0),
        # a small bf16 layer with ragged sizes (252-token frames, 40 text tokens)
        dict(name="midsize_roll", kind="roll", dtype="bf16", Hq=8, Hkv=2, D=128, n=252, n_text=40, n_past=6,
             mode="pow", gamma=0.85, b_min=32, n_score=100, fold=False, share=False, window=0),
        # the same layer in the fp32 tier, the full cache attended over
        dict(name="midsize_attn_f32", kind="attn", dtype="f32", Hq=8, Hkv=2, D=128, n=252, Nk=1804, fold=False,
             lse=True),
        # the paper's fixed-budget rule with a sliding window of 12 frames: the window moves on every step
        dict(name="window_roll_24h", kind="roll", dtype="bf16", Hq=24, Hkv=8, D=128, n=4032, n_text=256, n_past=13,
             mode="half", gamma=1.0, b_min=336, n_score=512, fold=True, share=False, window=12),
        # half-resolution frames: attention over a packed cache of frame 24, plain softmax scale
        dict(name="halfgrid_attn", kind="attn", dtype="bf16", Hq=16, Hkv=4, D=128, n=1008, Nk=7455, fold=False,
             lse=False),
        # bench.py's default step: the whole path at frame 24
        dict(name="frame24_oneshot", kind="oneshot", dtype="bf16", Hq=16, Hkv=4, D=128, n=4032, n_text=256,
             n_past=23, mode="pow", gamma=0.85, b_min=512, n_score=512, fold=True, share=False),
        # the late rollout: layers of the 24/8-head stack at frame 48, re-packed together
        dict(name="frame48_stack_24h", kind="stack", dtype="bf16", Hq=24, Hkv=8, D=128, n=4032, n_text=256,
             n_past=47, mode="pow", gamma=0.85, b_min=512, n_score=512, fold=True, share=False, layers=3),
        # the full-cache baseline at frame 48, the largest attention
        dict(name="frame48_attn_dense", kind="attn", dtype="bf16", Hq=16, Hkv=4, D=128, n=4032, Nk=193792,
             fold=False, lse=True),
        # scoring the full cache of frame 48, both passes
        dict(name="frame48_score", kind="score", dtype="bf16", Hq=16, Hkv=4, D=128, n=4032, n_score=512, Nk=193792,
             key0=0, fold=False, lse=False, share=False),
        # scoring fed by attention's log-sum-exp, one selection for all heads, prunable keys only
        dict(name="halfgrid_score_lse", kind="score", dtype="bf16", Hq=16, Hkv=4, D=128, n=1008, n_score=512,
             Nk=8463, key0=1264, fold=True, lse=True, share=True),
        # one layer's cache re-packed in place at frame 48 with the steepest decay
        dict(name="frame48_compact_layer", kind="compact", dtype="bf16", Hkv=4, D=128, n=4032, n_text=256, n_past=47,
             mode="pow", gamma=0.7, b_min=512, layers=1, in_place=True, share=False),
        # the 28-layer stack re-packed in one call
        dict(name="frame48_compact_stack", kind="compact", dtype="bf16", Hkv=4, D=128, n=4032, n_text=256, n_past=47,
             mode="pow", gamma=0.85, b_min=512, layers=28, in_place=True, share=False),
    ]


def _between(rng, lo, hi) -> int:
    """A whole number of [lo, hi], even over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng) -> dict:
    kind = rng.choice(["roll", "roll", "roll", "oneshot", "stack", "attn", "attn", "score", "score", "compact",
                       "compact"])
    f32 = kind != "stack" and rng.random() < 0.15
    if f32:   # the correctness tier runs at small sizes only
        Hq, Hkv = rng.choice([(2, 1), (3, 1), (8, 2)])
        D, n, n_past = rng.choice([64, 128]), _between(rng, 33, 300), _between(rng, 1, 8)
    else:
        Hq, Hkv = rng.choice([(2, 1), (6, 2), (8, 2), (16, 4), (16, 4), (24, 8)])
        D, n, n_past = 128, _between(rng, 64, 4032), _between(rng, 1, 47)
    n_text = _between(rng, 16, 256)
    mode = rng.choice(["pow", "pow", "pow", "norm", "half", "slide"])
    c = dict(kind=kind, dtype="f32" if f32 else "bf16", Hq=Hq, Hkv=Hkv, D=D, n=n, n_text=n_text, n_past=n_past,
             mode=mode, gamma=rng.choice([0.7, 0.85, 0.95]), b_min=max(1, n // 8) if mode == "pow" else 0,
             n_score=min(n, rng.choice([100, 512])), fold=rng.random() < 0.5, share=rng.random() < 0.2)
    if kind == "roll":
        c["window"] = 0
        if mode in ("norm", "half") and rng.random() < 0.5:
            c["window"] = rng.randint(2, 12)
            c["b_min"], c["n_past"] = n // c["window"], c["window"] + 1
    elif kind == "stack":
        c["layers"] = 1 if Hq * n > 65000 else 2 if Hq * n > 40000 else rng.randint(2, 6)
    elif kind in ("attn", "score"):
        full = n_text + n * (1 + n_past)
        c["Nk"] = min(_between(rng, n_text + n, full), 100000 if Hq > 16 else 193792)
        c["lse"] = rng.random() < 0.5
        if kind == "score":
            c["key0"] = rng.choice([0, n_text + n - 1])
        for k in ("n_text", "n_past", "mode", "gamma", "b_min") + (("n_score", "share") if kind == "attn" else ()):
            del c[k]
    elif kind == "compact":
        c["layers"] = rng.choice([1, 1, _between(rng, 2, 28)])
        while c["layers"] * Hkv * n * n_past > 28 * 4 * 4032 * 47:
            c["layers"] -= 1
        c["in_place"] = rng.random() < 0.6
        for k in ("Hq", "n_score", "fold"):
            del c[k]
    return c


# ------------------------------------------------------------------------------ inputs
def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _directions(seed, hkv, d):
    """One unit vector per KV group on the slowest rotary pairs: the mean direction of its queries."""
    lf = synth.low_frequency_dims(SECTIONS[d])
    u = np.zeros((hkv, d), np.float32)
    u[:, lf] = np.random.default_rng(seed).standard_normal((hkv, lf.size)).astype(np.float32)
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    return torch.from_numpy(u).to(DEV)


def _keys(out, u, bias, gen):
    """N(0,1) plus bias[row] along the group's direction; out [..][Hkv][rows][D]."""
    out.normal_(generator=gen)
    if bias is not None:
        out.add_((bias[:, None] * u[:, None, :]).to(out.dtype))


def _queries(out, u, gen, mul=1.0):
    rep = out.shape[-3] // u.shape[0]
    out.normal_(generator=gen)
    out.add_((math.sqrt(out.shape[-1]) * u.repeat_interleave(rep, dim=0))[:, None, :].to(out.dtype))
    if mul != 1.0:
        out.mul_(mul)


def _row_bias(segments):
    """0.5 for the anchors, 0.3 * 0.9^dist for a past frame at distance dist."""
    frames = [i for i, s in enumerate(segments) if s[2] == pk.PC_SEG_FRAME]
    bias = np.zeros(segments[-1][0] + segments[-1][1], np.float32)
    for i, (a, ln, kind, _) in enumerate(segments):
        bias[a:a + ln] = 0.5 if kind != pk.PC_SEG_FRAME else 0.3 * 0.9 ** (len(frames) - frames.index(i))
    return torch.from_numpy(bias).to(DEV)


def _positions(segments, n, n_text):
    """(t, h, w) of every row of the table: text token i at (i, i, i), a frame's rows on its grid."""
    gw = max(1, int(round(math.sqrt(n * 84 / 48))))
    rows = []
    for a, ln, kind, f in segments:
        i = np.arange(ln)
        if kind == pk.PC_SEG_TEXT:
            rows.append(np.stack([i, i, i], axis=1))
        else:
            i = i * n // max(ln, 1)     # a packed frame's rows are spread over its grid
            rows.append(np.stack([np.full(ln, n_text + 4 * f), 8 * (i // gw), 8 * (i % gw)], axis=1))
    return torch.from_numpy(np.concatenate(rows).astype(np.int32)).to(DEV)


def _by_distance(case, n_past):
    modes = {"pow": pk.PC_BUDGET_POW, "norm": pk.PC_BUDGET_NORM, "half": pk.PC_BUDGET_HALF, "slide": pk.PC_BUDGET_SLIDE}
    return pk.pc_budget(modes[case["mode"]], case["n"], n_past, case["gamma"], case["b_min"])


def _full_table(case):
    n, n_text = case["n"], case["n_text"]
    segs = [(0, n_text, pk.PC_SEG_TEXT, -1), (n_text, n, pk.PC_SEG_COND, 0)]
    for f in range(1, case["n_past"] + 1):
        segs.append((n_text + n * f, n, pk.PC_SEG_FRAME, f))
    return segs


def _rolling_table(case):
    """The table a rolling cache holds when the step with n_past past frames begins, before its
    newest frame is appended: what the step before left."""
    full = _full_table(case)[:-1]
    n_past = case["n_past"] - 1
    return pk.pc_compact_plan(full, pk.segment_budgets(full, _by_distance(case, n_past)))[0]


def _step_inputs(case, seed, layers, cache, table):
    """Cache rows, the frame to append and the step's queries of a stack of rolling layers."""
    n, n_text, dt = case["n"], case["n_text"], _dtype(case)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    K, V, pos = cache
    nk = table[-1][0] + table[-1][1]
    new = [(0, n, pk.PC_SEG_FRAME, case["n_past"])]
    st = {"k_new": torch.empty((layers, case["Hkv"], n, case["D"]), dtype=dt, device=DEV),
          "pos_new": _positions(new, n, n_text),
          "pos_q": _positions([(0, n, pk.PC_SEG_FRAME, case["n_past"] + 1)], n, n_text),
          "Q0": torch.empty((layers, case["Hq"], n, case["D"]), dtype=dt, device=DEV)}
    st["v_new"] = torch.empty_like(st["k_new"])
    st["v_new"].normal_(generator=gen)
    V.normal_(generator=gen)
    K.normal_(generator=gen)
    bias, bias_new = _row_bias(table), torch.full((n,), 0.3 * 0.9, device=DEV)
    for l in range(layers):
        u = _directions(seed * 64 + l, case["Hkv"], case["D"])
        K[l, :, :nk].add_((bias[:, None] * u[:, None, :]).to(dt))
        _keys(st["k_new"][l], u, bias_new, gen)
        _queries(st["Q0"][l], u, gen)
    pos.zero_()
    pos[..., :nk, :] = _positions(table, n, n_text)
    st["pos_new_rows"] = st["pos_new"].expand(pos.shape[:-2] + (n, 3)).contiguous()
    st["table"] = table
    return st


def prepare(case: dict, seed: int):
    kind, dt = case["kind"], _dtype(case)
    D, n, scale = case["D"], case["n"], case["D"] ** -0.5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    fold = case.get("fold", False)
    call_scale = pk.PC_SCALE_FOLDED if fold else scale
    q_scale = pk.folded_q_scale(scale) if fold else 1.0

    if kind in ("roll", "stack"):
        table = _rolling_table(case)
        nk = table[-1][0] + table[-1][1]
        args = dict(capacity=nk + n, n_frame=n, scale=scale, mode=case["mode"], gamma=case["gamma"],
                    b_min=case["b_min"], n_score=case["n_score"], sections=SECTIONS[D], base=BASE, dtype=dt,
                    device=DEV, share_heads=case["share"], fold_scale=fold)
        if kind == "roll":
            if case["window"]:
                args["slide_t_scale"] = 4
            layer = RollingLayer(case["Hq"], case["Hkv"], D, **args)
            st = _step_inputs(case, seed, 1, (layer.K[None], layer.V[None], layer.pos[None]), table)
            st.update(layer=layer, Q=torch.empty_like(st["Q0"][0]), O=torch.empty_like(st["Q0"][0]))
        else:
            stack = RollingStack(case["layers"], case["Hq"], case["Hkv"], D, **args)
            st = _step_inputs(case, seed, case["layers"], (stack.K, stack.V, stack.pos), table)
            st.update(stack=stack, Q=torch.empty_like(st["Q0"][0]), O=torch.empty_like(st["Q0"]),
                      lse=torch.empty(st["Q0"].shape[:3], dtype=torch.float32, device=DEV))
        st.update(case=case, nk=nk)
        return st

    if kind == "oneshot":
        full = _full_table(case)
        nk = full[-1][0] + full[-1][1]
        hsel = 1 if case["share"] else case["Hkv"]
        K = torch.empty((case["Hkv"], nk, D), dtype=dt, device=DEV)
        V = torch.empty_like(K)
        pos = torch.empty((hsel, nk, 3), dtype=torch.int32, device=DEV)
        st = _step_inputs(case, seed, 1, (K[None], V[None], pos[None]), full)
        _, nk_out = pk.pc_compact_plan(full, pk.segment_budgets(full, _by_distance(case, case["n_past"])))
        rows = torch.from_numpy(synth.strided_rows(n, case["n_score"]).astype(np.int32)).to(DEV)
        st.update(case=case, nk=nk, K=K, V=V, pos=pos, rows=rows, call_scale=call_scale, q_scale=q_scale,
                  Q=torch.empty_like(st["Q0"][0]), O=torch.empty_like(st["Q0"][0]),
                  score=torch.empty((hsel, nk), dtype=torch.float32, device=DEV),
                  out=(torch.empty((case["Hkv"], nk_out, D), dtype=dt, device=DEV),
                       torch.empty((case["Hkv"], nk_out, D), dtype=dt, device=DEV),
                       torch.empty((hsel, nk_out, 3), dtype=torch.int32, device=DEV)),
                  ws_s=torch.empty(max(16, pk.pc_score_workspace_bytes(case["Hq"], case["Hkv"], rows.numel(), nk,
                                                                       case["share"])),
                                   dtype=torch.uint8, device=DEV),
                  ws_c=torch.empty(max(16, pk.pc_compact_workspace_bytes(case["Hkv"], nk, case["share"])),
                                   dtype=torch.uint8, device=DEV))
        return st

    if kind in ("attn", "score"):
        nk = case["Nk"]
        u = _directions(seed, case["Hkv"], D)
        K = torch.empty((case["Hkv"], nk, D), dtype=dt, device=DEV)
        Q = torch.empty((case["Hq"], n, D), dtype=dt, device=DEV)
        age = torch.arange(nk, device=DEV).flip(0) // n + 1
        bias = torch.where(torch.arange(nk, device=DEV) < n, 0.5, 0.3 * 0.9 ** age.float())
        _keys(K, u, bias, gen)
        _queries(Q, u, gen, q_scale)
        st = dict(case=case, K=K, Q=Q, call_scale=call_scale)
        if kind == "attn":
            st.update(V=torch.empty_like(K).normal_(generator=gen), O=torch.empty_like(Q),
                      lse=torch.empty((case["Hq"], n), dtype=torch.float32, device=DEV) if case["lse"] else None)
            return st
        rows = torch.from_numpy(synth.strided_rows(n, case["n_score"]).astype(np.int32)).to(DEV)
        hsel = 1 if case["share"] else case["Hkv"]
        st.update(rows=rows, score=torch.zeros((hsel, nk), dtype=torch.float32, device=DEV), lse=None,
                  ws=torch.empty(max(16, pk.pc_score_workspace_bytes(case["Hq"], case["Hkv"], rows.numel(), nk,
                                                                     case["share"])),
                                 dtype=torch.uint8, device=DEV))
        if case["lse"]:   # as the attention pass over the same cache gives it
            lse = torch.empty((case["Hq"], n), dtype=torch.float32, device=DEV)
            pk.pc_frame_attn(Q, K, K, nk, call_scale, lse=lse)
            st["lse"] = lse
        return st

    # compact: caches and the importances of a scoring call (log-normal over the keys of a frame)
    full = _full_table(case)
    nk = full[-1][0] + full[-1][1]
    layers, hsel = case["layers"], 1 if case["share"] else case["Hkv"]
    lead = (layers,) if layers > 1 else ()
    K = torch.empty(lead + (case["Hkv"], nk, D), dtype=dt, device=DEV).normal_(generator=gen)
    V = torch.empty_like(K).normal_(generator=gen)
    pos = torch.empty(lead + (hsel, nk, 3), dtype=torch.int32, device=DEV)
    pos[:] = _positions(full, n, case["n_text"])
    score = torch.empty(lead + (hsel, nk), dtype=torch.float32, device=DEV).normal_(generator=gen)
    score.add_(_row_bias(full)).exp_().mul_(1.0 / nk)
    out = None
    if not case["in_place"]:
        _, nk_out = pk.pc_compact_plan(full, pk.segment_budgets(full, _by_distance(case, case["n_past"])))
        out = (torch.empty(lead + (case["Hkv"], nk_out, D), dtype=dt, device=DEV),
               torch.empty(lead + (case["Hkv"], nk_out, D), dtype=dt, device=DEV),
               torch.empty(lead + (hsel, nk_out, 3), dtype=torch.int32, device=DEV))
    nbytes = (pk.pc_compact_batch_workspace_bytes(layers, case["Hkv"], nk, case["share"]) if layers > 1 else
              pk.pc_compact_workspace_bytes(case["Hkv"], nk, case["share"]))
    return dict(case=case, table=full, K=K, V=V, pos=pos, score=score, out=out,
                ws=torch.empty(nbytes, dtype=torch.uint8, device=DEV))


# ------------------------------------------------------------------------------ one pass
def run(st):
    return _RUN[st["case"]["kind"]](st)


def _run_roll(st):
    case, layer = st["case"], st["layer"]
    n, frame = case["n"], case["n_past"]
    layer.segments, layer.nk, layer.shift = list(st["table"]), st["nk"], 0     # the step begins
    layer.advance_window()
    k, v, p = layer.reserve(n)
    k.copy_(st["k_new"][0])              # the model's projections write the newest frame's rows ...
    v.copy_(st["v_new"][0])
    p.copy_(st["pos_new_rows"][0])
    layer.commit(n, pk.PC_SEG_FRAME, frame, rotate_with=st["pos_new"])
    st["Q"].copy_(st["Q0"][0])           # ... and the step's queries, un-rotated
    layer.step(st["Q"], O=st["O"], q_pos=st["pos_q"])
    return {"O": st["O"], "Q": st["Q"], "nk": layer.nk}


def _run_oneshot(st):
    case = st["case"]
    a, n = st["nk"] - case["n"], case["n"]
    k_new = st["K"][:, a:a + n]
    st["Q"].copy_(st["Q0"][0])           # the step's queries and the newest frame's keys arrive un-rotated
    k_new.copy_(st["k_new"][0])
    pk.pc_rope3d(st["Q"], st["pos_q"], SECTIONS[case["D"]], BASE, out_scale=st["q_scale"])
    pk.pc_rope3d(k_new, st["pos_new"], SECTIONS[case["D"]], BASE)
    pk.pc_score(st["Q"], st["K"], st["nk"], st["call_scale"], score=st["score"], share_heads=case["share"],
                ws=st["ws_s"], q_rows=st["rows"])
    budgets = pk.segment_budgets(st["table"], _by_distance(case, case["n_past"]))
    _, nk = pk.pc_compact(st["K"], st["V"], st["pos"], st["score"], st["table"], budgets, share_heads=case["share"],
                          out=st["out"], ws=st["ws_c"])
    pk.pc_frame_attn(st["Q"], st["out"][0], st["out"][1], nk, st["call_scale"], O=st["O"])
    return {"O": st["O"], "score": st["score"], "Q": st["Q"], "nk": nk}


def _run_stack(st):
    case, stack = st["case"], st["stack"]
    n = case["n"]
    stack.segments, stack.nk = list(st["table"]), st["nk"]
    k, v, p = stack.reserve(n)
    k.copy_(st["k_new"])
    v.copy_(st["v_new"])
    p.copy_(st["pos_new_rows"])
    stack.commit(n, pk.PC_SEG_FRAME, case["n_past"], rotate_with=st["pos_new"])
    for l in range(case["layers"]):
        st["Q"].copy_(st["Q0"][l])
        pk.pc_rope3d(st["Q"], st["pos_q"], SECTIONS[case["D"]], BASE, out_scale=stack.q_out_scale)
        stack.attend(l, st["Q"], O=st["O"][l], lse=st["lse"][l])
        stack.score_layer(l, st["Q"], lse=st["lse"][l])
    stack.repack()
    return {"O": st["O"], "lse": st["lse"], "nk": stack.nk}


def _run_attn(st):
    pk.pc_frame_attn(st["Q"], st["K"], st["V"], st["case"]["Nk"], st["call_scale"], O=st["O"], lse=st["lse"])
    return {"O": st["O"], "lse": st["lse"]}


def _run_score(st):
    case = st["case"]
    return pk.pc_score(st["Q"], st["K"], case["Nk"], st["call_scale"], lse=st["lse"], score=st["score"],
                       share_heads=case["share"], ws=st["ws"], q_rows=st["rows"],
                       key_range=(case["key0"], case["Nk"]) if case["key0"] else None)


def _run_compact(st):
    case = st["case"]
    budgets = pk.segment_budgets(st["table"], _by_distance(case, case["n_past"]))
    call = pk.pc_compact_batch if case["layers"] > 1 else pk.pc_compact
    _, nk = call(st["K"], st["V"], st["pos"], st["score"], st["table"], budgets, share_heads=case["share"],
                 out=st["out"], ws=st["ws"])
    K, V, pos = st["out"] or (st["K"], st["V"], st["pos"])
    return {"K": K, "V": V, "pos": pos, "nk": nk}


_RUN = {"roll": _run_roll, "oneshot": _run_oneshot, "stack": _run_stack, "attn": _run_attn, "score": _run_score,
        "compact": _run_compact}


# ------------------------------------------------------------------------------ what a pass needs
def _plan(case, table):
    """(packed rows, rows that move, rows of the segments that lose any) for `table` in place."""
    n_past = sum(1 for s in table if s[2] == pk.PC_SEG_FRAME)
    after, nk = pk.pc_compact_plan(table, pk.segment_budgets(table, _by_distance(case, n_past)))
    first = next((i for i, (a, b) in enumerate(zip(table, after)) if a[1] != b[1]), len(table))
    moved = sum(s[1] for s in after[first:])
    pruned = sum(a[1] for a, b in zip(table, after) if a[1] != b[1])
    return nk, moved, pruned


def _attn_work(Hq, Hkv, n, nk, D, elt):
    return 2 * D * elt * (Hq * n + Hkv * nk), 4.0 * Hq * n * nk * D


def _score_work(Hq, Hkv, rows, nk, scored, D, elt, lse, hsel):
    return (D * elt * (Hq * rows + Hkv * nk) + 4 * hsel * scored,
            2.0 * D * Hq * rows * (scored + (0 if lse else nk)))


def _compact_work(case, moved, pruned, hsel):
    elt = 4 if case["dtype"] == "f32" else 2
    return moved * (case["Hkv"] * 4 * case["D"] * elt + hsel * 24) + 4 * hsel * pruned


def work(case: dict) -> dict:
    kind, n, D = case["kind"], case["n"], case["D"]
    elt = 4 if case["dtype"] == "f32" else 2
    Hq, Hkv = case.get("Hq"), case["Hkv"]
    hsel = 1 if case.get("share") else Hkv
    if kind == "attn":
        b, f = _attn_work(Hq, Hkv, n, case["Nk"], D, elt)
    elif kind == "score":
        b, f = _score_work(Hq, Hkv, case["n_score"], case["Nk"], case["Nk"] - case["key0"], D, elt, case["lse"], hsel)
    elif kind == "compact":
        table = _full_table(case)
        nk, moved, pruned = _plan(case, table)
        if not case["in_place"]:
            moved = nk                       # out of place every kept row is copied
        b, f = case["layers"] * _compact_work(case, moved, pruned, hsel), 0.0
    else:
        layers = case.get("layers", 1)
        if kind == "oneshot":
            table = _full_table(case)
        else:
            table = [s for s in _rolling_table(case) if s[1] > 0 or not case.get("window")]
            table = table + [(table[-1][0] + table[-1][1], n, pk.PC_SEG_FRAME, case["n_past"])]
        dense = table[-1][0] + table[-1][1]
        nk, moved, pruned = _plan(case, table)
        if kind == "oneshot":
            moved = nk
        first = next((s[0] for s in table if s[2] == pk.PC_SEG_FRAME), 0)
        b1, f1 = _attn_work(Hq, Hkv, n, dense if kind == "stack" else nk, D, elt)
        b2, f2 = _score_work(Hq, Hkv, case["n_score"], dense,
                             dense if kind == "oneshot" else pruned, D, elt, kind == "stack", hsel)
        # the newest frame's K, V and the queries: written by the producer, rotated (K and Q) in place
        b3 = n * D * elt * (Hkv * 2 * 2 + Hkv * 2 + Hq * 2 * 2)
        if case.get("window"):
            b3 += 2 * Hkv * elt * SECTIONS[D][0] * max(0, dense - n - first)
        b, f = layers * (b1 + b2 + b3 + _compact_work(case, moved, pruned, hsel)), layers * (f1 + f2)
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case: dict):
    """About four times what the path differs by from the same computation in 64 bits."""
    kind = case["kind"]
    if kind == "compact":
        return "exact"                       # rows are moved bit for bit, the choice is exact on given scores
    if kind == "score":
        return {"rel": 2e-6, "max": 1e-5}    # measured 4.7e-7 and 1.9e-6
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5}    # measured 1.2e-6 and 9.0e-6
    return {"rel": 1e-2, "max": 6.5e-2}      # measured 2.4e-3 and 1.6e-2 (the output's own rounding: 1.7e-3, 3.9e-3)
