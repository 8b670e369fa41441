"""Float64 configuration ids are what tuning files hold: the id a file names keeps its tile shape, or, where
that kernel is gone, runs on one whose tiles are smaller by a quarter of the area at most (256 x 32, made
for outputs of few columns: on tiles of the same 32 columns)."""

import re

from paper_2201_01257_amd import _lib

# tile shapes of the ids when tuning files were first written
TILES = [(64, 64), (128, 64), (64, 128), (128, 128), (32, 64), (128, 80), (80, 128), (64, 80), (32, 256), (256, 32),
         (128, 128), (128, 80), (64, 80), (64, 64), (128, 128)]


def test_ids_keep_their_tiles():
    lib = _lib.load()
    for i, (m, n) in enumerate(TILES):
        name = lib.tamm_config_name(0, i).decode()
        got = tuple(int(x) for x in re.match(r"f64_m(\d+)n(\d+)k", name).groups())
        if (m, n) == (256, 32):
            assert got[1] == 32, (i, name)
        else:
            assert got[0] * got[1] * 4 >= m * n * 3 and got[0] * got[1] <= m * n, (i, name)
    assert lib.tamm_config_name(0, len(TILES)).decode() == ""  # no more than these
