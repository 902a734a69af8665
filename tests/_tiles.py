"""Small batches that reach each tile of the bf16 projections (test code)."""
from __future__ import annotations

from tests._route import route, shape

# rows and columns with a ragged last tile, in ascending order of the work
ROWS = (31, 61, 95, 127, 189, 250, 381, 509)
COLS = (61, 1003, 2001, 4001, 5003, 8003, 10001, 12283, 16381, 20001, 24571, 28001, 32765, 40957,
        49001, 65501)
ALONE = ("32x64", "32x128", "64x64", "64x96", "64x128", "64x256", "128x64", "128x128", "128x256")
MIXED = [(f"{ra}x{ca}", f"{rt}x{ct}")
         for ra, wa in ((32, 128), (64, 256), (128, 256)) for ca in (64, wa)
         for rt, wt in ((32, 128), (64, 256), (128, 256)) for ct in (64, wt)]
WIDE = ("128x64", "128x128", "128x256")   # text tiles beside 256 x 256 audio tiles


def alone_sizes(tile, text):
    """Rows and columns of the smallest listed batch of one part that takes `tile`."""
    sizes = sorted(((M, N) for M in ROWS for N in COLS if M <= 128 or not text),
                   key=lambda s: s[0] * s[1])
    for M, N in sizes:
        r = route(0, 0, M, N) if text else route(M, N)
        if shape(r.text if text else r.audio) == tile:
            return M, N
    raise AssertionError(f"no batch takes {tile}")


def mixed_sizes(audio, text):
    """Audio rows and columns, text rows and columns of a batch that takes both tiles in one
    launch."""
    def part(tile):
        rows, cols = map(int, tile.split("x"))
        return {32: 31, 64: 61, 128: 127}[rows], 1003 if cols == 64 else 32765
    return (*part(audio), *part(text))


def wide_sizes(text):
    return 189, 65501, 95, {"128x64": 2001, "128x128": 32765, "128x256": 40957}[text]


# audio rows and columns, text rows and columns of batches that run as two launches, and their
# tiles: 256 x 256 audio tiles in at least three rounds beside a text part of a round or more, and
# in four beside a smaller one
TWO = [((765, 65501, 31, 65501), "256x256", "32x256"),
       ((765, 65501, 61, 65501), "256x256", "64x256"),
       ((1021, 65501, 31, 2001), "256x256", "32x256")]


def wrapping_slices(stages):
    """A number of 64-k slices that takes a weight ring of `stages` round, and the hidden rows'
    ring and registers (at most 2 + 8 slices) too, ending in the middle of each."""
    n = max(stages, 11) + 2
    while n % 2 == 0 or n % 3 == 0 or (stages and n % stages == 0):
        n += 1
    return n
