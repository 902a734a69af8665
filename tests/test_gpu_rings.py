"""Every streaming tile with more 64-k slices than its rings hold: each stage is filled again while
the tile computes, and the waits of the steady state and of the end run.  Scores and text partials
against float64 on the GPU."""
import numpy as np
import pytest

from tests._compare import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_02119_amd import mcd  # noqa: E402
from tests._route import route  # noqa: E402
from tests._tiles import (  # noqa: E402
    ALONE, MIXED, TWO, WIDE, alone_sizes, mixed_sizes, wide_sizes, wrapping_slices)

# bf16 products are exact in fp32.  A fp32 sum of n of them, of variance 1 / n each, has rounding
# errors of standard deviation about sqrt(n) 2^-24 / 2 in any order: 1e-6 at n = 1216, and the
# largest of 10^7 sums is six times that.  A stale or early slice moves a sum by about 0.1.
TOL = 2e-5


def check(Mg, N, text, V_text):
    r = route(Mg, N, text, V_text)
    H = 64 * wrapping_slices(max(r.audio.stages, r.text.stages))
    say(f"case M={Mg} N={N} text={text} V_text={V_text} H={H} {r}")
    gen = torch.Generator("cuda").manual_seed(Mg + N + text + V_text)

    def normal(rows, scale):
        return (torch.randn(rows, H, generator=gen, device="cuda") * scale).bfloat16()
    # streams of at most 4096 ids, N in all
    sizes = [4096] * (N // 4096) + ([N % 4096] if N % 4096 else []) if Mg else [1]
    W, Wt = normal(sum(sizes), H ** -0.5), normal(V_text, H ** -0.5) if text else None
    head = mcd.Head(W, list(range(len(sizes))), max(sizes), None, Wt, sizes)
    pairs = Mg // 4
    solo = Mg - 2 * pairs
    kind = np.array([0, 1] * pairs + [2] * solo + [3] * text, np.uint8)
    pair = np.full(len(kind), -1, np.int32)
    pair[:2 * pairs] = np.arange(2 * pairs) ^ 1
    perm = np.random.default_rng(Mg).permutation(len(kind))
    inv = np.argsort(perm)
    moved = pair[perm]
    kind, pair = kind[perm], np.where(moved >= 0, inv[moved], -1).astype(np.int32)
    plan = head.plan(pair, kind)
    R, Rs = len(kind), pairs + solo
    hidden = normal(R, 1.0)
    full = lambda v, dt: torch.full((R,), v, dtype=dt, device="cuda")  # noqa: E731
    scores = torch.full((max(Rs, 1), sum(sizes)), float("nan"), device="cuda")
    ws = head.workspace(R)
    mcd.mcd_head_logits(
        head.handle, R=R, counts=plan.counts, plan=plan.dev, hidden=hidden,
        cfg_w=full(2.0, torch.float32), temperature=full(0.5, torch.float32),
        top_k=full(0, torch.int32), top_p=full(1.0, torch.float32), rng_key=None,
        step=full(0, torch.int32), n_frames=full(1, torch.int32), grid_slot=full(-1, torch.int32),
        seed=0, tokens_out=torch.zeros(R, len(sizes), dtype=torch.int32, device="cuda"),
        frame_grid=None, n_slots=0, F_max=0, scores=scores, workspace=ws)
    torch.cuda.synchronize()
    assert mcd.mcd_read_device_status(ws) == 0
    rows = plan.host[8:]
    if Mg:
        order = torch.from_numpy(rows[:Mg].astype(np.int64)).cuda()
        logits = hidden[order].double() @ W.double().t().contiguous()
        want = torch.cat([2.0 * logits[0:2 * pairs:2] - logits[1:2 * pairs:2],
                          logits[2 * pairs:]]) / 0.5
        err = float((scores.double() - want).abs().max())
        say(f"  score error {err:.2e}")
        assert err <= 6 * TOL          # w = 2, 1 - w = -1, 1 / T = 2
    if text:
        order = torch.from_numpy(rows[Mg:Mg + text].astype(np.int64)).cuda()
        logits = hidden[order].double() @ Wt.double().t().contiguous()
        parts = (V_text + 31) // 32
        pad = torch.full((text, parts * 32), float("-inf"), dtype=torch.float64, device="cuda")
        pad[:, :V_text] = logits
        top, at = pad.view(text, parts, 32).topk(2, dim=2)
        # partials in the workspace: a float per row and part, then (256-byte aligned for R rows)
        # its id
        ids_at = 256 + (R * parts * 4 + 255) // 256 * 256
        val = ws[256:256 + text * parts * 4].view(torch.float32).view(text, parts)
        ids = ws[ids_at:ids_at + text * parts * 4].view(torch.int32).view(text, parts)
        err = float((val.double() - top[:, :, 0]).abs().max())
        say(f"  text partial error {err:.2e}")
        assert err <= TOL
        first = torch.arange(parts, device="cuda") * 32
        wrong = (ids.long() != at[:, :, 0] + first) & (top[:, :, 0] - top[:, :, 1] > 2 * TOL)
        assert not bool(wrong.any())


@pytest.mark.parametrize("tile", ALONE)
def test_audio_alone(tile):
    check(*alone_sizes(tile, False), 0, 0)


@pytest.mark.parametrize("tile", ALONE)
def test_text_alone(tile):
    check(0, 0, *alone_sizes(tile, True))


@pytest.mark.parametrize("audio,text", MIXED)
def test_mixed_launch(audio, text):
    check(*mixed_sizes(audio, text))


@pytest.mark.parametrize("text", WIDE)
def test_beside_wide_audio(text):
    check(*wide_sizes(text))


@pytest.mark.parametrize("sizes,audio,text", TWO)
def test_two_launches(sizes, audio, text):
    check(*sizes)
