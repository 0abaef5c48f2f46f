"""CPU: which kernel a matrix product takes (csrc/gemm_shapes.hpp, compiled for the host)."""
import random

import pytest

from . import _host_model as hm

# (rows of A, rows of B, contraction length) -> kernel
EXPECTED = {
    # a wide weight and few rows: the tiles are many, but most of their rows do not exist
    (33, 28672, 8192): "tile64", (64, 28672, 8192): "tile64", (64, 28672, 4096): "tile64",
    (48, 32768, 8192): "tile64", (64, 57344, 8192): "tile64", (48, 128256, 4096): "tile64",
    (64, 151936, 3584): "tile64", (65, 28672, 8192): "tile128", (96, 128256, 4096): "tile128",
    (128, 28672, 8192): "tile128", (128, 57344, 8192): "tile128", (128, 128256, 4096): "tile128",
    (192, 28672, 8192): "tile64", (196, 29536, 4096): "tile256x128", (199, 14464, 14336): "tile128",
    (256, 28672, 8192): "tile256x128",
    # ... and with K not a multiple of 256
    (1, 28672, 8256): "tile32", (16, 28672, 8256): "tile32", (32, 201088, 2880): "tile32",
    (48, 28672, 8256): "tile64", (128, 28672, 8256): "tile128", (256, 28672, 8256): "tile256x128",
    # the same with A and B exchanged
    (28672, 64, 4128): "tile64", (201088, 31, 2880): "tile64x32",
    # few rows
    (1, 8192, 8192): "skinny", (16, 8192, 8192): "skinny", (32, 28672, 8192): "skinny",
    (33, 8192, 8192): "skinny", (64, 8192, 8192): "skinny", (64, 4096, 4096): "tile32",
    (16, 8192, 2880): "tile32", (128, 4096, 4096): "tile64x32", (128, 8192, 8192): "tile64long",
    (200, 4096, 4096): "tile64",
    # ... along a long K
    (33, 4096, 28672): "skinny", (48, 2048, 53248): "skinny", (64, 4096, 28672): "tile32",
    (33, 4096, 8192): "tile32", (33, 4096, 4128): "tile32", (33, 1024, 16384): "tile32",
    (65, 5120, 28672): "tile32", (96, 5120, 8192): "tile32", (65, 4096, 53248): "tile32",
    (256, 2048, 28672): "tile32", (384, 1024, 53248): "tile32", (65, 5120, 11008): "tile32",
    (256, 2048, 11008): "tile64x32", (65, 5120, 8160): "tile64", (65, 8192, 28672): "tile64long",
    (128, 8192, 28672): "tile64long", (256, 4096, 28672): "tile64long", (512, 2048, 53248): "tile64long",
    (128, 8192, 2880): "tile64", (192, 8192, 8192): "tile64",
    # large and middling products
    (8192, 8192, 8192): "dma", (2816, 4096, 4096): "dma", (192, 128256, 4096): "dma",
    (512, 28672, 8192): "dma", (4352, 4096, 2048): "tile64", (2048, 4096, 4096): "tile256x128",
    (8192, 8192, 8160): "tile256x128", (1000, 4096, 4096): "tile128", (2880, 1440, 1056): "tile64",
    (1340, 4464, 5504): "tile256x128", (431, 7440, 2048): "tile128", (5834, 1600, 1024): "tile64",
    (1, 1, 1 << 25): "staged",
}


@pytest.mark.parametrize("size", EXPECTED, ids=lambda s: "x".join(map(str, s)))
def test_expected_kernel(size):
    assert hm.choose_gemm(*size) == EXPECTED[size]


def test_large_tiles_are_mostly_filled():
    """No drawn product gets large tiles that hold more than 1 / 0.62 of what tiles of 64 x 64 do."""
    rng = random.Random(4648)
    for _ in range(20000):
        M, N = (int(2 ** rng.uniform(0, 18)) for _ in range(2))
        K = int(2 ** rng.uniform(0, 10)) * rng.choice((32, 128, 256))
        kernel = hm.choose_gemm(M, N, K)
        if kernel in ("dma", "tile128", "tile256x128"):
            bm, bn = (256, 256) if kernel == "dma" else hm.tile_shape(kernel)[:2]
            assert (-(-M // 64) * 64) * (-(-N // 64) * 64) > 0.61 * (-(-M // bm) * bm) * (-(-N // bn) * bn), (
                M, N, K, kernel)


def test_no_launch_is_too_large():
    """A launch holds fewer than 2^32 lanes; every size that 256 x 256 tiles of 256 lanes could cover
    within that is covered, by any kernel."""
    sizes = [(1, 1 << 31, 32), ((1 << 31), 1, 32), (1, 3 * 10 ** 8, 32), (1, (1 << 30) + 32, 256),
             (32, 1 << 30, 128), (3 * 10 ** 8, 17, 96), (200, 1 << 31, 160)]
    rng = random.Random(4649)
    while len(sizes) < 20000:
        M, N = (int(2 ** rng.uniform(0, 31)) for _ in range(2))
        K = 32 * int(2 ** rng.uniform(0, 20))
        if -(-M // 256) * -(-N // 256) * 256 < 1 << 32:
            sizes.append((M, N, K))
    for M, N, K in sizes:
        kernel = hm.choose_gemm(M, N, K)
        assert hm.gemm_lanes(kernel, M, N) < 1 << 32, (M, N, K, kernel)
        assert kernel != "dma" or (K % 128 == 0 and K <= 1 << 24), (M, N, K)
