"""CPU: which kernel a matrix product takes (csrc/gemm_shapes.hpp, compiled for the host)."""
import random

import pytest

from . import _host_model as hm

# (rows of A, rows of B, contraction length) -> kernel
EXPECTED = {
    # a wide weight and few rows: the tiles are many, but most of their rows do not exist
    (33, 28672, 8192): "tile64", (64, 28672, 8192): "tile64", (64, 28672, 4096): "tile64",
    (48, 32768, 8192): "tile64", (64, 57344, 8192): "tile64", (48, 128256, 4096): "tile64",
    (64, 151936, 3584): "tile64", (65, 28672, 8192): "dma128", (96, 128256, 4096): "tile128",
    (128, 28672, 8192): "dma128", (128, 57344, 8192): "tile128", (128, 128256, 4096): "tile128",
    (192, 28672, 8192): "dma256x128", (196, 29536, 4096): "dma256x128", (199, 14464, 14336): "dma128",
    (256, 28672, 8192): "dma256x128",
    # ... and with K not a multiple of 256
    (1, 28672, 8256): "tile32", (16, 28672, 8256): "tile32", (32, 201088, 2880): "tile32",
    (48, 28672, 8256): "tile64", (128, 28672, 8256): "dma128", (256, 28672, 8256): "dma256x128",
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
    (512, 28672, 8192): "dma", (4352, 4096, 2048): "tile64", (2048, 4096, 4096): "dma256x128",
    (8192, 8192, 8160): "dma", (1000, 4096, 4096): "dma128", (2880, 1440, 1056): "tile64",
    (1340, 4464, 5504): "dma256x128", (431, 7440, 2048): "dma128", (5834, 1600, 1024): "tile64",
    (6000, 8000, 96): "dma", (2816, 4096, 4064): "dma", (6144, 6400, 1056): "dma", (3072, 3072, 992): "tile64",
    (4096, 4608, 3040): "dma256x128", (6798, 880, 4160): "dma256x128", (1000, 4096, 992): "tile128",
    (3000, 3000, 1024): "tile64", (1000, 5232, 32): "dma256x128", (2048, 4096, 256): "dma256x128",
    # ... several turns of 256 x 128 tiles, filled to 66 %, 70 %, 74 %
    (8324, 1925, 256): "tile64", (6496, 2681, 2688): "tile64", (8328, 2176, 256): "dma256x128",
    (1344, 13184, 1824): "tile256x128",
    # lines of C that do not begin at multiples of 16 bytes: in BF16 and fp32 ...
    (2048, 4095, 32): "tile256x128", (2048, 4095, 992): "tile256x128", (2048, 4095, 1024): "dma256x128",
    (5727, 954, 256): "tile64", (4055, 738, 1536): "tile64", (4055, 738, 2048): "dma128", (2816, 4095, 128): "dma",
    # beyond 32-bit lane offsets
    (1, 1, 1 << 25): "staged", (1, 1, (1 << 24) + 32): "staged", (4096, 8192, (1 << 24) + 32): "staged",
}
# ... and in BF16 only
EXPECTED_BF16_F32 = {
    (2048, 4092, 256): ("tile256x128", "dma256x128"), (1000, 4092, 1056): ("tile128", "dma128"),
    (2816, 4092, 256): ("dma", "dma"),
}


@pytest.mark.parametrize("size", EXPECTED, ids=lambda s: "x".join(map(str, s)))
def test_expected_kernel(size):
    assert (hm.choose_gemm(*size), hm.choose_gemm(*size, f32=True)) == (EXPECTED[size],) * 2


@pytest.mark.parametrize("size", EXPECTED_BF16_F32, ids=lambda s: "x".join(map(str, s)))
def test_expected_kernel_by_type(size):
    assert (hm.choose_gemm(*size), hm.choose_gemm(*size, f32=True)) == EXPECTED_BF16_F32[size]


LARGE = {"dma": (256, 256), "dma256x128": (256, 128), "dma128": (128, 128), "tile256x128": (256, 128),
         "tile128": (128, 128)}


def test_large_tiles_are_mostly_filled():
    """No drawn product gets large tiles that hold more than 1 / 0.62 of what tiles of 64 x 64 do, or that are so few
    that most of the chip is idle."""
    rng = random.Random(4648)
    seen = dict.fromkeys(LARGE, 0)
    for _ in range(40000):
        M, N = (int(2 ** rng.uniform(0, 18)) for _ in range(2))
        K = int(2 ** rng.uniform(0, 10)) * rng.choice((32, 128, 256))
        kernel = hm.choose_gemm(M, N, K, rng.random() < 0.5)
        if kernel in LARGE:
            bm, bn = LARGE[kernel]
            tm, tn = -(-M // bm), -(-N // bn)
            assert (-(-M // 64) * 64) * (-(-N // 64) * 64) > 0.61 * tm * bm * tn * bn, (M, N, K, kernel)
            assert tm * tn >= 0.62 * 256 and M > 64 and N > 64 and K <= 1 << 24, (M, N, K, kernel)
            seen[kernel] += 1
    assert min(seen.values()) > 10, seen


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
    seen = set()
    for M, N, K in sizes:
        for f32 in (False, True):
            kernel = hm.choose_gemm(M, N, K, f32)
            assert hm.gemm_lanes(kernel, M, N) < 1 << 32, (M, N, K, kernel)
            assert kernel != "dma" or K <= 1 << 24, (M, N, K)
            # (what the sizes alone would choose and a launch does not hold)
            if kernel in ("dma", "staged") and (-(-M // 64) * 64) * (-(-N // 64) * 64) <= 0.61 * (
                    -(-M // 256) * -(-N // 256) * 65536):
                seen.add(kernel)
    assert seen == {"dma", "staged"}
