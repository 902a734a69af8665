"""GPU parity at the edges of the kernels' tiles and of their dispatch: shapes just below, at and
just above a tile's rows, columns and k groups, each checked against the CPU oracle (scores within
the bound of the data type, tokens bit for bit except where the oracle flags a near tie)."""
import numpy as np
import pytest

import oracle
from paper_2607_02119_amd import inputs
from tests._compare import TokenCheck, say, score_rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_02119_amd import harness, mcd  # noqa: E402
from tests.test_gpu_graph import (  # noqa: E402
    test_step_replayed_from_a_graph_equals_eager as replay)

from tests._route import route, shape  # noqa: E402

GAP_TOL, TOPK_TOL, TOPP_TOL = 1e-3, 1e-4, 1e-5


def check_one_step(wl, t, score_tol):
    dw = harness.DeviceWorkload(wl)
    dw.load_hidden([t])
    dw.tokens.fill_(-1)
    dw.run_step(t, hidden_index=0)
    torch.cuda.synchronize()
    o = oracle.head_step(dw.host_head, inputs.make_batch(wl, t, dw.layout), seed=dw.seed,
                         gap_tol=GAP_TOL, topk_tol=TOPK_TOL, topp_tol=TOPP_TOL)
    tc = TokenCheck()
    tc.add(dw.tokens.cpu().numpy(), o["tokens"], o["flags"], where=f"t={t}")
    tc.assert_ok(wl.name)
    if wl.Rs:
        rows = [r for r, _ in dw.plan.sampled_rows()]
        err = score_rel_err(dw.scores.cpu().numpy(), rows, o["scores"],
                            oracle.stream_sizes(dw.host_head))
        say(f"  score rel err {err:.3e}")
        assert err <= score_tol
    assert dw.status() == 0


# fp32 head: row blocks of 16, 32 and 64 rows and row tiles beyond, 16-column
# (text: 32-column) workgroups, k16 groups dealt to four waves; H below one
# group, not a multiple of 16, and not a multiple of 4
F32 = [
    # H, V, pairs, solo, text, V_text
    (4, 1, 0, 1, 0, 0),
    (3, 5, 1, 0, 1, 1),
    (16, 16, 8, 0, 1, 32),
    (17, 17, 8, 1, 2, 33),
    (64, 31, 16, 0, 16, 64),
    (272, 40, 16, 1, 17, 31),
    (255, 33, 30, 4, 33, 65),
    (1028, 20, 32, 1, 65, 97),
]


@pytest.mark.parametrize("H,V,pairs,solo,text,V_text", F32)
def test_fp32_head_tiles(H, V, pairs, solo, text, V_text):
    wl = inputs.Workload(f"f32_{H}_{V}", H=H, K=2, V=V, n_pairs=pairs, n_solo=solo, n_text=text,
                         V_text=V_text, dtype="f32", top_k=3, steps=4, shuffle=True,
                         bias=H % 2 == 0)
    say(f"case {wl.name} R={wl.R}")
    check_one_step(wl, 2, 1e-5)


# top-k through the short list: one group of ids per lane and two, the list's
# capacity (128 groups) reached and passed, k above the parts that have a
# score, masked ids, ties at the bound, with and without a nucleus; one
# workgroup per vector and (from 1024 vectors of at most 1024 ids) one wave
TOPK = [
    # V, K, Rs, sigma, quantum, top_k, top_p, masked share, mask value
    (2, 2, 3, 1.0, 0.0, 1, 1.0, 0.0, 0.0),
    (5, 4, 256, 1.0, 0.0, 4, 0.9, 0.0, 0.0),
    (255, 2, 5, 2.0, 0.0, 254, 0.95, 0.0, 0.0),
    (513, 2, 5, 2.0, 0.0, 1, 0.5, 0.0, 0.0),
    (4096, 2, 6, 3.6, 0.0, 64, 1.0, 0.0, 0.0),
    (4096, 2, 6, 3.6, 0.0, 64, 0.9, 0.0, 0.0),
    (4095, 2, 6, 3.6, 0.0, 110, 0.9, 0.0, 0.0),
    (4096, 2, 6, 3.6, 0.0, 128, 1.0, 0.0, 0.0),
    (4096, 2, 6, 3.6, 0.0, 256, 0.8, 0.0, 0.0),
    (2048, 2, 6, 3.6, 0.125, 50, 1.0, 0.0, 0.0),
    (2048, 2, 6, 3.6, 0.125, 50, 0.9, 0.0, 0.0),
    (2048, 2, 6, 1.0, 1.0, 20, 0.9, 0.0, 0.0),
    (4096, 2, 6, 2.0, 0.0, 50, 0.9, 0.99, -1e30),
    (4096, 2, 6, 2.0, 0.0, 50, 1.0, 0.5, -3.0e38),
    (1024, 4, 256, 3.6, 0.0, 64, 0.9, 0.0, 0.0),
    (1024, 4, 256, 3.6, 0.0, 100, 1.0, 0.0, 0.0),
    (1024, 4, 256, 3.6, 0.125, 40, 0.9, 0.0, 0.0),
    (1003, 4, 256, 3.6, 0.0, 30, 0.9, 0.9, -1e30),
    (130, 8, 128, 2.0, 0.0, 129, 0.99, 0.0, 0.0),
    # the largest cut of the list and the first of the bins, for each form
    (4096, 2, 6, 3.6, 0.0, 96, 0.9, 0.0, 0.0),
    (4096, 2, 6, 3.6, 0.0, 97, 0.9, 0.0, 0.0),
    (2048, 2, 6, 3.6, 0.0, 96, 1.0, 0.0, 0.0),
    (2048, 2, 6, 3.6, 0.0, 97, 1.0, 0.0, 0.0),
    (1024, 2, 6, 3.6, 0.0, 60, 0.9, 0.0, 0.0),
    (1024, 2, 6, 3.6, 0.0, 61, 0.9, 0.0, 0.0),
    (1024, 2, 6, 3.6, 0.0, 120, 1.0, 0.0, 0.0),
    (1024, 2, 6, 3.6, 0.0, 121, 1.0, 0.0, 0.0),
    (1024, 4, 256, 3.6, 0.0, 120, 0.9, 0.0, 0.0),
    (1024, 4, 256, 3.6, 0.0, 121, 0.9, 0.0, 0.0),
    (512, 4, 256, 3.6, 0.0, 511, 0.9, 0.0, 0.0),
    (256, 4, 256, 3.6, 0.0, 255, 1.0, 0.0, 0.0),
    # masked to the lowest fp32 value, to -1e30 and to -inf; unmasked scores
    # below the first cut of the bound's search (32 under the maximum)
    (4096, 2, 6, 2.0, 0.0, 50, 0.9, 0.995, -3.4028234663852886e38),
    (1024, 4, 256, 2.0, 0.0, 20, 1.0, 0.95, -3.4028234663852886e38),
    (2048, 2, 6, 2.0, 0.0, 50, 1.0, 0.99, -1e30),
    (4096, 2, 6, 2.0, 0.0, 50, 0.9, 0.995, -np.inf),
    (4096, 2, 6, 40.0, 0.0, 64, 1.0, 0.0, 0.0),
    (1024, 4, 256, 40.0, 0.0, 50, 0.9, 0.9, -1e30),
]


def sampler_only(V, K, Rs, top_k, top_p):
    wl = inputs.Workload("sampler", H=64, K=K, V=V, n_pairs=0, n_solo=Rs, top_k=top_k,
                         top_p=top_p, steps=3 * K)
    return wl, harness.DeviceWorkload(wl, weights=dict(
        H=64, K=K, V=V, pad_id=V, delays=np.arange(K, dtype=np.int32),
        W=np.zeros((K, V, 64), np.uint16), bias=None, W_text=None))


@pytest.mark.parametrize("V,K,Rs,sigma,quantum,top_k,top_p,share,value", TOPK)
def test_topk_list_edges(V, K, Rs, sigma, quantum, top_k, top_p, share, value):
    """The sampler alone on the same scores as the oracle; the exemptions are its own rounding:
    top-2 gaps below 1e-4, nucleus cuts within 1e-6 of p; top-k cuts are exact."""
    say(f"case V={V} K={K} Rs={Rs} top_k={top_k} top_p={top_p} q={quantum} masked={share}")
    wl, dw = sampler_only(V, K, Rs, top_k, top_p)
    tc = TokenCheck()
    srow = [r for r, _ in dw.plan.sampled_rows()]
    for t in (K - 1, K):
        sc = inputs.make_scores(Rs, wl.N, t, sigma=sigma, quantum=quantum)
        sc[np.random.default_rng(t).random(sc.shape) < share] = value
        dw.tokens.fill_(-1)
        dw.sample_only(t, harness.to_device(sc))
        torch.cuda.synchronize()
        o = oracle.sample_rows(dw.host_head, inputs.make_batch(wl, t, dw.layout), srow,
                               [-1] * Rs, sc.astype(np.float64), gap_tol=1e-4, topk_tol=0.0,
                               topp_tol=1e-6)
        tc.add(dw.tokens.cpu().numpy(), o["tokens"], o["flags"], where=f"t={t}")
    tc.assert_ok(f"V={V} k={top_k}")


@pytest.mark.parametrize("V,K,Rs,top_p", [(4096, 4, 4, 1.0), (512, 8, 128, 0.9)])
def test_topk_infinite_scores_give_valid_ids(V, K, Rs, top_p):
    """Infinite scores with a top-k cut: a valid id, and a finite score's id wherever only some
    scores are minus infinity."""
    say(f"case infinite V={V} K={K} Rs={Rs}")
    wl, dw = sampler_only(V, K, Rs, 20, top_p)
    sc = inputs.make_scores(Rs, wl.N, 1, sigma=2.0)
    sc[2, :V] = -np.inf
    sc[3, :V:5] = np.inf
    sc[0, V:2 * V] = -np.inf
    sc[0, V + 11] = 1.0
    sc[1, V:2 * V:2] = -np.inf
    dw.tokens.fill_(-1)
    dw.sample_only(K - 1, harness.to_device(sc))
    torch.cuda.synchronize()
    rows = [r for r, _ in dw.plan.sampled_rows()]
    g = dw.tokens.cpu().numpy()[rows]
    assert np.all((g >= 0) & (g < V))
    assert g[0, 1] == 11 and g[1, 1] % 2 == 1


# streaming tiles (copying and computing waves apart) at the edges of their
# rows and columns, audio and text; fewer slices of 64 k than ring stages, an
# odd number of slices, and slice counts around the hidden rows' register
# buffers (test_gpu_rings.py: more slices than ring stages, for every tile)
STREAM = [
    # H, V, K, pairs, solo, text, V_text      audio tile, text tile
    (64, 33, 1, 16, 0, 1, 65, "32x64", "32x64"),
    (64, 4096, 8, 16, 1, 0, 0, "64x128", None),
    (192, 4096, 8, 32, 0, 0, 0, "64x128", None),
    (448, 4096, 8, 64, 0, 0, 0, "128x128", None),
    (576, 61, 3, 32, 1, 33, 129, "128x64", "64x64"),
    (832, 64, 2, 63, 2, 64, 63, "128x64", "64x64"),
    (128, 4096, 9, 15, 1, 32, 33001, "32x128", "32x128"),
    (960, 4096, 9, 1, 0, 0, 0, "32x128", None),
    (320, 4093, 9, 20, 24, 65, 32801, "64x256", "128x256"),
    (64, 300, 2, 64, 1, 128, 257, "128x256", "128x64"),
    (704, 1027, 3, 70, 13, 0, 0, "32x64", None),
]


def check_tiles(wl, audio, text):
    """The batch takes the tiles it stands for."""
    r = route(2 * wl.n_pairs + wl.n_solo, wl.N, wl.n_text, wl.V_text, wl.H)
    assert (audio is None or shape(r.audio) == audio) and (text is None or shape(r.text) == text), r


@pytest.mark.parametrize("H,V,K,pairs,solo,text,V_text,audio_tile,text_tile", STREAM)
def test_streaming_tile_edges(H, V, K, pairs, solo, text, V_text, audio_tile, text_tile):
    wl = inputs.Workload(f"stream_{H}_{V}", H=H, K=K, V=V, n_pairs=pairs, n_solo=solo, n_text=text,
                         V_text=V_text, dtype="bf16", top_k=5, steps=2 * K, shuffle=True,
                         bias=V % 2 == 1)
    say(f"case {wl.name} R={wl.R} N={wl.N}")
    check_tiles(wl, audio_tile, text_tile)
    check_one_step(wl, K, 1e-5)


# audio rows beyond 128: whole rounds of 256 x 256 tiles against 128 x 256 ones
# (the last round of the former full, half full and empty)
ROWS = [
    # V, K, pairs, solo, tile
    (4096, 8, 128, 0, "128x256"),
    (4096, 8, 256, 0, "256x256"),
    (4096, 8, 256, 1, "128x256"),
    (4096, 6, 256, 256, "128x256"),
    (3000, 5, 65, 30, "128x128"),
]


@pytest.mark.parametrize("V,K,pairs,solo,tile", ROWS)
def test_row_tile_choice(V, K, pairs, solo, tile):
    wl = inputs.Workload(f"rows_{V}_{K}_{pairs}", H=128, K=K, V=V, n_pairs=pairs, n_solo=solo,
                         dtype="bf16", top_k=5, steps=2 * K, shuffle=True)
    say(f"case {wl.name} R={wl.R} N={wl.N}")
    check_tiles(wl, tile, None)
    check_one_step(wl, K, 1e-5)


# audio and text rows in one launch of streaming tiles: every pair of row
# heights (audio rows beyond 128 too), narrow and wide columns on either side
MIXED = [
    # V, K, pairs, solo, text, V_text
    (50, 2, 1, 0, 1, 33),
    (60, 3, 16, 0, 33, 200),
    (61, 3, 15, 1, 65, 32801),
    (70, 3, 16, 1, 32, 32801),
    (300, 2, 32, 0, 64, 100),
    (4096, 9, 20, 2, 128, 70),
    (33, 2, 32, 1, 20, 150),
    (4093, 9, 64, 0, 40, 32900),
    (90, 4, 60, 8, 100, 64),
    (100, 3, 64, 1, 9, 32801),
    (1000, 4, 80, 9, 60, 90),
    (700, 3, 130, 0, 128, 300),
]


@pytest.mark.parametrize("V,K,pairs,solo,text,V_text", MIXED)
def test_mixed_streaming_launch(V, K, pairs, solo, text, V_text):
    wl = inputs.Workload(f"mixed_{V}_{text}", H=192, K=K, V=V, n_pairs=pairs, n_solo=solo,
                         n_text=text, V_text=V_text, dtype="bf16", top_k=5, steps=2 * K,
                         shuffle=True, bias=V % 2 == 1)
    say(f"case {wl.name} R={wl.R} N={wl.N}")
    check_one_step(wl, K, 1e-5)


def test_two_stream_step_replayed_from_a_graph():
    """More than 128 text rows: audio and text rows on two streams, fork and join in the graph."""
    replay("two_streams", dict(H=128, K=3, V=37, n_pairs=10, n_solo=5, n_text=150, V_text=300,
                               dtype="bf16", top_k=7, steps=6, shuffle=True))


# delay pattern: one thread per token or one per frame (step), by codebooks, frames
# per request (64) and frames in all (32768, 65536 and 2^20); codebook counts
# around the eight in flight and the 16-byte store; request lengths around whole
# waves and blocks; large and equal delays, F = 0
DELAY = [
    # n_req, K, F, delays
    (3, 8, 64, range(8)),
    (2, 8, 63, range(8)),
    (5, 7, 200, (0, 3, 3, 1, 0, 9, 2)),
    (2, 9, 65, range(9)),
    (1, 32, 130, range(31, -1, -1)),
    (4, 12, 257, [100] * 12),
    (600, 4, 300, (0, 1, 2, 3)),
    (3, 1, 64, (5,)),
    (2, 4, 0, (0, 1, 2, 70)),
    (512, 8, 64, range(8)),
    (512, 3, 64, (0, 1, 0)),
    (520, 8, 63, range(8)),
    (511, 4, 64, (2, 0, 1, 0)),
    (170, 7, 200, (0, 3, 3, 1, 0, 9, 2)),
    (512, 9, 65, range(9)),
    (256, 32, 130, range(31, -1, -1)),
    (128, 12, 257, [100] * 12),
    (110, 5, 301, (4, 0, 0, 1, 30)),
    (64, 16, 513, range(16)),
    (520, 1, 64, (5,)),
    (1024, 1, 64, (5,)),
    (1023, 2, 64, (1, 0)),
    (1024, 2, 64, (1, 0)),
    (300, 6, 700, range(6)),
    (2100, 2, 500, (0, 5)),
    (33000, 4, 64, (0, 1, 2, 3)),
]


@pytest.mark.parametrize("n_req,K,F,delays", DELAY)
@pytest.mark.parametrize("shift", [0, 1])
def test_delay_pattern_rows(n_req, K, F, delays, shift):
    """`shift`: the stream buffer starts that many tokens past a 16-byte boundary."""
    delays = np.array(list(delays), np.int32)
    say(f"case delay n_req={n_req} K={K} F={F} shift={shift}")
    T = F + int(delays.max())
    G = np.random.default_rng(K).integers(0, 4096, (n_req, K, F)).astype(np.int32)
    buf = torch.full((n_req * T * K + shift,), -7, dtype=torch.int32, device="cuda")
    streams = buf[shift:].view(n_req, T, K)
    grid = torch.from_numpy(G).cuda()
    mcd.mcd_interleave(grid, delays, 4096, streams)
    back = torch.full_like(grid, -7)
    mcd.mcd_deinterleave(streams, delays, back)
    torch.cuda.synchronize()
    want = np.full((n_req, T, K), 4096, np.int32)
    for k, dk in enumerate(delays):
        want[:, dk:dk + F, k] = G[:, k]
    assert np.array_equal(streams.cpu().numpy(), want)
    assert np.array_equal(back.cpu().numpy(), G)
    assert (buf[:shift] == -7).all()


# the tile shape chosen by rounds x (rows + columns), each shape with ragged
# rows and columns and with several row tiles (runs per XCD of unequal length)
SHAPES = [
    # V, K, pairs, solo, text, V_text         audio tile, text tile
    (1003, 7, 37, 21, 0, 0, "64x64", None),        # two row tiles
    (4095, 3, 64, 0, 0, 0, "64x96", None),         # two row tiles
    (4001, 6, 20, 0, 0, 0, "64x96", None),
    (4096, 2, 100, 0, 0, 0, "128x64", None),       # two row tiles
    (4093, 2, 140, 20, 0, 0, "128x128", None),     # three row tiles
    (4003, 5, 40, 20, 0, 0, "128x128", None),
    (2001, 1, 65, 0, 0, 0, "32x64", None),         # five row tiles
    (257, 1, 250, 3, 0, 0, "32x64", None),         # sixteen row tiles
    (10, 1, 0, 0, 95, 7021, None, "64x64"),
    (10, 1, 0, 0, 120, 12290, None, "128x64"),     # past one round of 64 x 96
    (10, 1, 0, 0, 120, 12280, None, "64x96"),      # two row tiles, the last 8 columns short
    (10, 1, 0, 0, 40, 2000, None, "32x64"),        # two row tiles
]


@pytest.mark.parametrize("V,K,pairs,solo,text,V_text,audio_tile,text_tile", SHAPES)
def test_tile_shapes(V, K, pairs, solo, text, V_text, audio_tile, text_tile):
    wl = inputs.Workload(f"shape_{V}_{K}_{pairs}_{text}", H=128, K=K, V=V, n_pairs=pairs,
                         n_solo=solo, n_text=text, V_text=V_text, dtype="bf16", top_k=5,
                         steps=2 * K + 1, shuffle=True)
    say(f"case {wl.name} R={wl.R} N={wl.N}")
    check_tiles(wl, audio_tile, text_tile)
    check_one_step(wl, K, 1e-5)
