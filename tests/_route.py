"""The library's own choice of tiles for a bf16 step (test code)."""
from __future__ import annotations

import collections
import ctypes

from paper_2607_02119_amd import mcd

Tile = collections.namedtuple("Tile", "rows cols stages")
Route = collections.namedtuple("Route", "launches audio text")

_route = ctypes.CDLL(mcd._LIB_PATH).mcd_projection_route
_route.restype = None
_route.argtypes = [ctypes.c_int32] * 5 + [ctypes.POINTER(ctypes.c_int32)]


def route(Mg, N, n_text=0, V_text=0, H=4096):
    """launches, and the tile (rows, columns, 64-k slices of the weight ring) of the audio and of
    the text part; zeros for a part that is not there, no stages outside the streaming tiles."""
    out = (ctypes.c_int32 * 7)()
    _route(Mg, N, n_text, V_text, H, out)
    return Route(out[0], Tile(*out[1:4]), Tile(*out[4:7]))


def shape(tile):
    return f"{tile.rows}x{tile.cols}"
