"""CPU: how tensors are dealt out to the workgroups of the tiled quantizers (csrc/tile_shapes.hpp, compiled for the
host)."""
import random

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


def _map(rows, cols):
    """tile_map() as its comment has it: die S % 8 takes super-tile S, counted in rows of super-tiles."""
    nt_r, nt_c = -(-rows // 64), -(-cols // 128)
    best, best_most = None, None
    for wide, high in ((8, 16), (8, 8), (4, 8), (4, 4), (2, 4), (2, 2), (1, 2), (1, 1)):
        sx, sy = min(nt_c, wide), min(nt_r, high)
        across = -(-nt_c // sx)
        supers = across * -(-nt_r // sy)
        if (wide, high) == (8, 16) and supers > 64:
            return sx, sy
        tiles = [0] * 8
        for S in range(supers):
            tiles[S % 8] += min(nt_c - S % across * sx, sx) * min(nt_r - S // across * sy, sy)
        if best is None or max(tiles) < best_most:
            best, best_most = (sx, sy), max(tiles)
        if max(tiles) <= 32 or max(tiles) * 32 <= nt_r * nt_c * 5:
            break
    return best


def _sizes():
    rng = random.Random(46)
    yield from ((1, 8), (64, 128), (65, 129), (16, 1 << 20), (1 << 20, 8), (736, 1024), (1008, 4096), (5248, 6192), (8192, 8192), (8640, 560), (6496, 528),
                (1 << 31, 512), (512, 1 << 31))
    for _ in range(3000):
        yield int(2 ** rng.uniform(0, 15)), int(2 ** rng.uniform(3, 15)) // 8 * 8


def test_map_of_tiles():
    for rows, cols in _sizes():
        sx, sy, _ = hm.tile_map(rows, cols)
        assert (sx, sy) == _map(rows, cols), (rows, cols)


def test_every_tile_has_one_workgroup():
    """The kernel's way from a workgroup to its tile, over the whole launch."""
    for rows, cols in _sizes():
        nt_r, nt_c = -(-rows // 64), -(-cols // 128)
        if nt_r * nt_c > 2000:
            continue
        sx, sy, grid = hm.tile_map(rows, cols)
        nsx = -(-nt_c // sx)
        seen = set()
        for block in range(grid):
            slot, xcd = divmod(block, 8)
            round_, within = divmod(slot, sx * sy)
            S = round_ * 8 + xcd
            r, c = S // nsx * sy + within // sx, S % nsx * sx + within % sx
            if r < nt_r and c < nt_c:
                assert (r, c) not in seen, (rows, cols, block)
                seen.add((r, c))
        assert len(seen) == nt_r * nt_c, (rows, cols)


@pytest.mark.parametrize("rows,cols", [(8640, 560), (8752, 592), (6496, 528), (10608, 3184), (736, 1024), (1344, 2208)])
def test_every_die_has_its_share(rows, cols):
    """8640 x 560: super-tiles of 4 x 4 in rows of two, one of them a single tile wide, all on every other die."""
    nt_r, nt_c = -(-rows // 64), -(-cols // 128)
    sx, sy, _ = hm.tile_map(rows, cols)
    across = -(-nt_c // sx)
    tiles = [0] * 8
    for r in range(nt_r):
        for c in range(nt_c):
            tiles[(r // sy * across + c // sx) % 8] += 1
    assert max(tiles) <= max(32, nt_r * nt_c * 5 / 32), (sx, sy, tiles)
