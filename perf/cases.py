"""The calls whose speed is tracked: what a serving program has this library do, through its
public entry points (``mcd.Head``, ``mcd_head_step``, ``mcd_next_input``, ``mcd_deinterleave``,
``mcd_interleave``), over the range it meets.

``listed()`` gives the named cases, ``draw(rng)`` one more of the same ranges, ``prepare`` what a
program holds before the call, ``run`` one pass, ``work`` the bytes and operations a pass cannot do
without, ``tolerance`` how far another correct implementation may be, ``exact`` the outputs in 64
bits from plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_02119_amd import mcd

TEXT_VOCAB = 151936          # text head of the repository's mixed workload


def _step(name, H, K, V, pairs=0, solo=0, text=0, V_text=0, T_text=0, dtype="bf16", w=3.0, T=1.0,
          top_k=0, top_p=1.0, frames=505, first=0, bias=False, shuffle=False):
    """A decode step of the head; `first`: ids of the first stream where it differs from V."""
    return dict(name=name, kind="step", H=H, K=K, V=V, first=first, pairs=pairs, solo=solo,
                text=text, V_text=V_text, T_text=T_text, dtype=dtype, w=w, T=T, top_k=top_k,
                top_p=top_p, frames=frames, bias=bias, shuffle=shuffle)


def listed():
    return [
        # the smallest head of the workload table, fp32: a call is all launches and latency
        _step("tiny_fp32", 256, 4, 1024, pairs=2, dtype="fp32", top_k=50, frames=29),
        # one guided request alone on the GPU: an interactive user
        _step("one_pair", 4096, 8, 4096, pairs=1, w=2.0, top_p=0.95),
        # the workload table's small decode batch
        _step("memory_bound_decode", 2048, 8, 2048, pairs=16, T=0.9, top_k=50, frames=249),
        # the headline batch: the whole head is read for 128 rows, nucleus sampling
        _step("weight_streaming", 4096, 8, 4096, pairs=64, w=2.0, top_p=0.95),
        # nine streams of unequal size (one SSL stream, eight codec streams)
        _step("opuslm_9_streams", 4096, 9, 1024, pairs=64, w=2.0, top_p=0.95, first=4096,
              frames=504),
        # the CFG ablation's two sides: 512 rows guided in pairs, 512 rows on their own
        _step("cfg_on", 4096, 16, 1024, pairs=256, T=0.8, top_k=20, frames=241),
        _step("cfg_off", 4096, 16, 1024, solo=512, T=0.8, top_k=20, frames=241),
        # the largest: a full continuous batch of guided, plain and text rows, shuffled
        _step("mfma_mixed", 4096, 8, 4096, pairs=256, solo=256, text=128, V_text=TEXT_VOCAB,
              top_k=50, frames=121, shuffle=True),
        # requests all in their text phase: the text head alone, with the phase mask
        _step("text_phase", 4096, 8, 4096, text=24, V_text=TEXT_VOCAB, T_text=TEXT_VOCAB - 4096),
        # odd sizes throughout, all row kinds, a stream-embedding bias, top-k and top-p together
        _step("ragged_batch", 1600, 7, 1003, pairs=37, solo=21, text=9, V_text=32003, w=1.7,
              T=0.85, top_k=30, top_p=0.9, frames=311, bias=True, shuffle=True),
        # the backbone's next input of the largest batch
        dict(name="next_input", kind="next_input", H=4096, K=8, V=4096, pairs=256, solo=256,
             text=128, V_text=TEXT_VOCAB, dtype="bf16"),
        # requests that have finished: their token streams to frame grids and back
        dict(name="delay_pattern", kind="delay", n_req=64, steps=1500, K=8),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["fp32", "text", "next_input", "delay"])
    if kind == "delay":
        return dict(kind="delay", n_req=_spread(rng, 1, 256), steps=_spread(rng, 64, 1500),
                    K=rng.randint(2, 16))
    if kind == "next_input":
        return dict(kind="next_input", H=64 * _spread(rng, 16, 64), K=rng.randint(2, 12),
                    V=_spread(rng, 256, 4096), pairs=_spread(rng, 1, 256),
                    solo=rng.randint(0, 128), text=rng.randint(0, 64),
                    V_text=_spread(rng, 4000, TEXT_VOCAB), dtype=rng.choice(["bf16", "bf16", "fp32"]))
    if kind == "text":
        V_text = _spread(rng, 8000, TEXT_VOCAB)
        case = _step("", 64 * _spread(rng, 16, 64), 8, 1024, text=_spread(rng, 1, 128),
                     V_text=V_text, T_text=rng.choice([0, V_text // 64 * 32]))
    elif kind == "fp32":
        case = _step("", 4 * _spread(rng, 16, 128), rng.randint(2, 8), _spread(rng, 64, 1024),
                     pairs=rng.randint(1, 4), solo=rng.randint(0, 3), dtype="fp32",
                     top_k=rng.choice([0, 1, 50]), frames=rng.randint(20, 200))
    else:
        top_k, top_p = rng.choice([(0, 0.95), (0, 1.0), (20, 1.0), (50, 1.0), (50, 0.9)])
        text = rng.choice([0, 0, rng.randint(1, 128)])
        case = _step("", 64 * _spread(rng, 16, 64), rng.randint(2, 8), _spread(rng, 512, 4096),
                     pairs=_spread(rng, 1, 256), solo=rng.choice([0, _spread(rng, 1, 256)]),
                     text=text, V_text=_spread(rng, 8000, TEXT_VOCAB) if text else 0,
                     w=rng.choice([1.5, 2.0, 3.0]), T=rng.choice([0.0, 0.8, 0.9, 1.0, 1.0]),
                     top_k=top_k, top_p=top_p, frames=rng.randint(60, 600),
                     bias=rng.random() < 0.25, shuffle=rng.random() < 0.5)
    del case["name"]
    return case


# ---- inputs ----------------------------------------------------------------

def _dtype(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


def _sizes(case):
    """Ids of every stream."""
    return [case.get("first") or case["V"]] + [case["V"]] * (case["K"] - 1)


def _normal(gen, shape, dtype, scale=1.0):
    """N(0, scale^2) in blocks, so that no large fp32 copy is held."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    rows = max(1, (1 << 26) // max(1, out[0].numel()))
    for i in range(0, shape[0], rows):
        block = torch.randn((min(rows, shape[0] - i),) + tuple(shape[1:]), generator=gen,
                            device="cuda")
        out[i:i + rows] = block.mul_(scale)
    return out


def _layout(case, rng):
    """pair_map, row_kind and request number of every row: guided pairs (Main, Companion), plain
    rows, text rows; shuffled as a scheduler leaves them where the case says so."""
    P, S, X = case["pairs"], case["solo"], case["text"]
    kind = np.array([mcd.MCD_ROW_COND, mcd.MCD_ROW_UNCOND] * P + [mcd.MCD_ROW_SOLO] * S
                    + [mcd.MCD_ROW_TEXT] * X, np.uint8)
    pair = np.full(len(kind), -1, np.int32)
    pair[:2 * P] = np.arange(2 * P) ^ 1
    request = np.concatenate([np.repeat(np.arange(P), 2), P + np.arange(S + X)])
    if case.get("shuffle"):
        perm = rng.permutation(len(kind))
        inverse = np.argsort(perm)
        moved = pair[perm]
        pair = np.where(moved >= 0, inverse[moved], -1).astype(np.int32)
        kind, request = kind[perm], request[perm]
    return kind, pair, request


def _cuda(a, dtype=None):
    return torch.from_numpy(np.ascontiguousarray(a, dtype)).to("cuda")


def _weights(case, gen):
    """Hidden states, head weights, bias and text-head weights."""
    H, K = case["H"], case["K"]
    sizes, dtype, scale = _sizes(case), _dtype(case), 1.0 / math.sqrt(case["H"])
    R = 2 * case["pairs"] + case["solo"] + case["text"]
    hidden = _normal(gen, (R, H), dtype)
    shape = (K, case["V"], H) if len(set(sizes)) == 1 else (sum(sizes), H)
    W = _normal(gen, shape, dtype, scale)
    bias = torch.randn(sum(sizes), generator=gen, device="cuda") if case["bias"] else None
    W_text = _normal(gen, (case["V_text"], H), dtype, scale) if case["V_text"] else None
    return hidden, W, bias, W_text


def _prepare_step(case, seed):
    gen, rng = torch.Generator("cuda").manual_seed(seed), np.random.default_rng(seed)
    K, sizes, frames = case["K"], _sizes(case), case["frames"]
    hidden, W, bias, W_text = _weights(case, gen)
    head = mcd.Head(W, list(range(K)), max(sizes), bias, W_text,
                    sizes if len(set(sizes)) > 1 else None, case["T_text"])
    kind, pair, request = _layout(case, rng)
    plan = head.plan(pair, kind)
    R, n_req = len(kind), plan.Rs + plan.n_text
    # each request is at a step of its own, the last K - 1 of them in its drain
    step = rng.integers(0, frames + K - 1, n_req)[request]
    key = rng.integers(0, 2 ** 62, n_req)[request]
    main = (kind == mcd.MCD_ROW_COND) | (kind == mcd.MCD_ROW_SOLO)
    full = lambda v, dt: torch.full((R,), v, dtype=dt, device="cuda")  # noqa: E731
    tokens = torch.full((R, K), -1, dtype=torch.int32, device="cuda")
    grid = torch.full((max(n_req, 1), K, frames), -1, dtype=torch.int32, device="cuda")
    modality = torch.zeros(R, dtype=torch.uint8, device="cuda")
    scores = torch.zeros((max(plan.Rs, 1), sum(sizes)), dtype=torch.float32, device="cuda")
    args = dict(R=R, counts=plan.counts, plan=plan.dev, hidden=hidden,
                cfg_w=full(case["w"], torch.float32), temperature=full(case["T"], torch.float32),
                top_k=full(case["top_k"], torch.int32), top_p=full(case["top_p"], torch.float32),
                rng_key=_cuda(key, np.int64), step=_cuda(step, np.int32),
                n_frames=full(frames, torch.int32),
                grid_slot=_cuda(np.where(main, request, -1), np.int32), seed=seed,
                tokens_out=tokens, frame_grid=grid, n_slots=n_req, F_max=frames, scores=scores,
                workspace=head.workspace(R), modality_out=modality)
    return dict(kind="step", head=head, plan=plan, args=args,
                out=dict(tokens=tokens, grid=grid, modality=modality,
                         scores=scores[:plan.Rs]) if plan.Rs else
                dict(tokens=tokens, modality=modality))


def _prepare_next_input(case, seed):
    gen, rng = torch.Generator("cuda").manual_seed(seed), np.random.default_rng(seed)
    H, K, V = case["H"], case["K"], case["V"]
    E = _normal(gen, (K * (V + 1), H), _dtype(case)).view(K, V + 1, H)
    E_text = _normal(gen, (case["V_text"], H), _dtype(case))
    kind, _, request = _layout(dict(case, shuffle=True), rng)
    R, n = len(kind), int(request.max()) + 1
    tok = rng.integers(0, V, (n, K))
    tok[rng.random((n, K)) < 0.02] = V            # pads: a stream not yet, or no longer, running
    tok = tok[request]
    is_text = kind == mcd.MCD_ROW_TEXT
    tok[is_text, :] = V
    tok[is_text, 0] = rng.integers(0, case["V_text"], int(is_text.sum()))
    out = torch.zeros((R, H), dtype=_dtype(case), device="cuda")
    return dict(kind="next_input", E=E, E_text=E_text, tokens=_cuda(tok, np.int32),
                row_kind=_cuda(kind), pad=V, out=out,
                workspace=torch.zeros(256, dtype=torch.uint8, device="cuda"))


def _prepare_delay(case, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    n, T, K = case["n_req"], case["steps"], case["K"]
    streams = torch.randint(0, 4096, (n, T, K), generator=gen, device="cuda", dtype=torch.int32)
    grid = torch.zeros((n, K, T - (K - 1)), dtype=torch.int32, device="cuda")
    return dict(kind="delay", streams=streams, grid=grid, delays=np.arange(K, dtype=np.int32),
                back=torch.zeros_like(streams))


def prepare(case, seed):
    if case["kind"] == "step":
        return _prepare_step(case, seed)
    if case["kind"] == "next_input":
        return _prepare_next_input(case, seed)
    return _prepare_delay(case, seed)


# ---- one pass --------------------------------------------------------------

def run(s):
    if s["kind"] == "step":
        mcd.mcd_head_step(s["head"].handle, **s["args"])
        return s["out"]
    if s["kind"] == "next_input":
        mcd.mcd_next_input(s["E"], s["tokens"], s["row_kind"], s["pad"], s["out"],
                           E_text=s["E_text"], workspace=s["workspace"])
        return s["out"]
    mcd.mcd_deinterleave(s["streams"], s["delays"], s["grid"])
    mcd.mcd_interleave(s["grid"], s["delays"], 4096, s["back"])
    return s["grid"], s["back"]


def work(case):
    if case["kind"] == "delay":
        n, T, K = case["n_req"], case["steps"], case["K"]
        return {"bytes": 4 * n * K * 2 * (T + T - (K - 1)), "flops": 0}
    eb = 4 if case["dtype"] == "fp32" else 2
    H, K = case["H"], case["K"]
    audio, text = 2 * case["pairs"] + case["solo"], case["text"]
    if case["kind"] == "next_input":
        return {"bytes": (audio * (K + 1) + 2 * text) * H * eb + 4 * (audio + text) * K,
                "flops": audio * K * H}
    # weights of the heads that have rows, hidden states, scores written, tokens written
    N = sum(_sizes(case)) if audio else 0
    N_text = case["V_text"] if text else 0
    sampled = case["pairs"] + case["solo"]
    return {"bytes": ((N + N_text) * H + (audio + text) * H) * eb + 4 * sampled * N
            + 4 * (audio + text + sampled) * K,
            "flops": 2 * H * (audio * N + text * N_text)}


def tolerance(case):
    """Scores are fp32 sums of exact products over H: sums in another order differ by a few 1e-7
    of the scores' size.  A token moves only where two perturbed scores are that close."""
    if case["kind"] == "step":
        return {"rel": 2.5e-6, "max": 4e-5, "differ": 0.005}
    return "exact"     # whole numbers, or sums exact in fp64 and rounded once


# ---- the same in 64 bits ---------------------------------------------------

def exact(case, seed):
    if case["kind"] == "delay":
        return None    # whole numbers
    if case["kind"] == "next_input":
        s = _prepare_next_input(case, seed)
        rows = s["tokens"].long()
        out = torch.zeros(s["out"].shape, dtype=torch.float64, device="cuda")
        for k in range(case["K"]):
            out += s["E"][k][rows[:, k].clamp(max=case["V"])].double()
        text = s["row_kind"] == mcd.MCD_ROW_TEXT
        out[text] = s["E_text"][rows[text, 0]].double()
        return out
    if case["pairs"] + case["solo"] == 0:
        return None    # text rows give tokens only
    gen, rng = torch.Generator("cuda").manual_seed(seed), np.random.default_rng(seed)
    hidden, W, bias, _ = _weights(case, gen)
    kind, pair, _ = _layout(case, rng)
    main = np.flatnonzero(kind == mcd.MCD_ROW_COND)
    solo = np.flatnonzero(kind == mcd.MCD_ROW_SOLO)
    rows = lambda i: hidden[torch.from_numpy(i).long().to("cuda")].double()  # noqa: E731
    W = W.reshape(-1, case["H"])
    w, parts = float(np.float32(case["w"])), []
    inv = 1.0 / float(np.float32(case["T"])) if case["T"] > 0 else 1.0
    for n in range(0, W.shape[0], 8192):
        Wn = W[n:n + 8192].double().t().contiguous()
        b = 0.0 if bias is None else bias[n:n + 8192].double()
        guided = w * (rows(main) @ Wn + b) + (1 - w) * (rows(pair[main]) @ Wn + b)
        parts.append(torch.cat([guided, rows(solo) @ Wn + b]) * inv)
    return dict(tokens=None, grid=None, modality=None, scores=torch.cat(parts, 1))
