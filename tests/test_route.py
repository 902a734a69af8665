"""The choice of tiles for a bf16 step, on the host: every streaming tile that is built is reached
by some batch, alone and beside the other part, and batches go to the route that is meant."""
import pytest

pytest.importorskip("paper_2607_02119_amd.mcd", reason="libmcd.so not built")

from tests._route import route, shape  # noqa: E402
from tests._tiles import ALONE, MIXED, WIDE, alone_sizes, mixed_sizes, wide_sizes  # noqa: E402


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
