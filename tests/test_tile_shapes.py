"""CPU: how tensors are dealt out to the workgroups of the tiled quantizers (csrc/tile_shapes.hpp, compiled for the
host)."""
import pytest

from . import _host_model as hm


# (fp32, BF16): the fastest of three where both sides of a line were timed, see tile_shapes.hpp
@pytest.mark.parametrize("rows,cols,fp32,bf16", [
    (16, 16, 4, 4), (512, 512, 4, 4), (2048, 2048, 4, 4), (736, 5360, 4, 4),       # up to 1024 units of 4 tile rows
    (4240, 1024, 8, 8), (4096, 2048, 8, 8), (1024, 8192, 8, 8),                    # up to 1024 units of 8
    (3536, 2496, 16, 16), (2320, 4000, 16, 16), (3072, 3072, 16, 16), (5216, 2384, 8, 16),
    (8192, 2048, 8, 16), (7168, 2048, 8, 16), (4096, 4096, 8, 16),                 # up to 1024 units of 16
    (4096, 4112, 8, 8), (5120, 4096, 8, 8), (4096, 5632, 8, 8),                    # a second turn for the rest of them
    (4096, 6144, 16, 16), (5120, 5120, 16, 16), (8192, 4096, 16, 16), (8192, 8192, 16, 16), (16384, 8192, 16, 16)])
def test_height_of_units(rows, cols, fp32, bf16):
    assert (hm.tile_unit_rows(rows, cols, True), hm.tile_unit_rows(rows, cols, False)) == (fp32, bf16)


def test_height_of_units_follows_the_compute_units():
    """Half the chip is full of half as much."""
    for rows, cols in ((2048, 1024), (2048, 2048), (4096, 1024), (1152, 4096), (4096, 2064), (8192, 8192)):
        for xf32 in (False, True):
            assert hm.tile_unit_rows(rows, cols, xf32, 128) == hm.tile_unit_rows(2 * rows, cols, xf32, 256), (rows, cols)
