"""The choice of tiles for a bf16 step, on the host: every streaming tile that is built is reached
by some batch, alone and beside the other part, and batches go to the route that is meant."""
import pytest

pytest.importorskip("paper_2607_02119_amd.mcd", reason="libmcd.so not built")

from tests._route import route, shape  # noqa: E402
from tests._tiles import ALONE, MIXED, TWO, WIDE, alone_sizes, mixed_sizes, wide_sizes  # noqa: E402


@pytest.mark.parametrize("text", [False, True])
@pytest.mark.parametrize("tile", ALONE)
def test_tile_alone_is_reached(tile, text):
    M, N = alone_sizes(tile, text)
    r = route(0, 0, M, N) if text else route(M, N)
    assert r.launches == 1 and shape(r.text if text else r.audio) == tile
    assert (r.text if text else r.audio).stages >= 3


@pytest.mark.parametrize("audio,text", MIXED)
def test_mixed_tiles_are_reached(audio, text):
    r = route(*mixed_sizes(audio, text))
    assert (r.launches, shape(r.audio), shape(r.text)) == (1, audio, text)


@pytest.mark.parametrize("text", WIDE)
def test_text_tiles_beside_wide_audio_are_reached(text):
    r = route(*wide_sizes(text))
    assert (r.launches, shape(r.audio), shape(r.text)) == (1, "256x256", text)


@pytest.mark.parametrize("sizes,audio,text", TWO)
def test_two_launches_are_reached(sizes, audio, text):
    r = route(*sizes, H=832)
    assert (r.launches, shape(r.audio), shape(r.text)) == (2, audio, text)


# audio rows (of 32768 columns), text rows, text columns, H: launches.  Measured as one launch of
# streaming tiles and as two, us: see the numbers.
FORMS = [
    (512, 24, 151936, 4096, 1),      # 321 / 344
    (512, 64, 151936, 4096, 1),      # 352 / 358
    (600, 64, 151936, 4096, 1),      # 361 / 400; 256 x 256 tiles are one fifth padding
    (768, 64, 151936, 4096, 2),      # 419 / 413
    (768, 64, 151936, 2560, 1),      # 297 / 299
    (768, 24, 151936, 4096, 1),      # 389 / 409
    (896, 64, 151936, 4096, 1),      # 429 / 450; one eighth padding
    (1024, 24, 151936, 4096, 2),     # 455 / 448
    (1024, 64, 151936, 4096, 2),     # 484 / 466
    (1024, 64, 151936, 2048, 1),     # 267 / 273
    (1024, 64, 151936, 1600, 1),     # 224 / 234
    (1280, 24, 151936, 4096, 2),     # 527 / 516
    (1536, 64, 151936, 4096, 2),     # 622 / 581
    (1536, 64, 151936, 1600, 2),     # 287 / 279
    (2048, 24, 151936, 4096, 2),     # 734 / 699
    (1024, 8, 8000, 4096, 1),        # 275 / 308
    (1800, 24, 151936, 4096, 2),     # 692 / 639
    (1664, 24, 151936, 2560, 2),     # 450 / 429
    (1664, 24, 151936, 1600, 1),     # 293 / 298
    (1800, 24, 151936, 2048, 2),     # 385 / 366
    (1800, 24, 151936, 1600, 2),     # 326 / 311
    (1800, 8, 8000, 4096, 2),        # 524 / 495
    (1800, 8, 8000, 2560, 2),        # 388 / 357
    (1800, 8, 8000, 2048, 1),        # 295 / 300
    (2432, 8, 8000, 1600, 2),        # 323 / 318
    (2432, 8, 8000, 1024, 1),        # 222 / 233
    (2304, 8, 8000, 4096, 1),        # the text tiles fill the last round of 256 x 256 tiles only
    (2048, 8, 8000, 4096, 2),        # 562 / 549
    (2048, 8, 8000, 1024, 2),        # 211 / 188
    (2048, 64, 32003, 1024, 1),      # 211 / 220
]


@pytest.mark.parametrize("rows,text,V_text,H,launches", FORMS)
def test_few_text_rows_beside_many_audio_rows(rows, text, V_text, H, launches):
    r = route(rows, 32768, text, V_text, H)
    assert r.launches == launches
    assert shape(r.audio) == ("256x256" if launches == 2 else "128x256")


def test_parts_alone_and_many_text_rows():
    assert route(0, 0).launches == 0
    assert shape(route(512, 32768).audio) == "256x256"
    r = route(25, 111, 150, 300)          # more than 128 text rows: two launches
    assert r.launches == 2 and shape(r.text) == "256x128"


@pytest.mark.parametrize("tile,most", [("32x64", 6), ("64x64", 6), ("64x96", 6), ("128x64", 8)])
def test_weight_rings_of_small_tiles_stay_short(tile, most):
    """A longer ring holds back the first hidden rows: 64 rows of 16384 columns at H 1024 took
    11.5 us with all the stages that fit and 10.3 with six (10.3 in the four-wave tile before)."""
    assert route(*alone_sizes(tile, False)).audio.stages <= most
