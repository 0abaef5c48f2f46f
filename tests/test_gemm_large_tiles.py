"""Products in the large tiles (256 x 256, 256 x 128 and 128 x 128): which take them (CPU), and their results (GPU)."""
import random

import numpy as np
import pytest
import torch

from . import _host_model as hm

TILES = {"dma": (256, 256), "dma256x128": (256, 128), "dma128": (128, 128)}


@pytest.mark.parametrize("size,kernel", [
    ((8192, 8192, 8160), "dma"), ((6000, 8000, 96), "dma"), ((2816, 4096, 4064), "dma"),
    ((6144, 6400, 1056), "dma"), ((3072, 3072, 992), "tile64"), ((4096, 4608, 3040), "dma256x128"),
    ((2048, 4096, 4096), "dma256x128"), ((192, 28672, 8192), "dma256x128"), ((6798, 880, 4160), "dma256x128"),
    ((1000, 4096, 4096), "dma128"), ((128, 28672, 8192), "dma128"), ((1000, 4096, 992), "tile128"),
    ((64, 28672, 8192), "tile64"), ((28672, 64, 4128), "tile64"), ((3000, 3000, 1024), "tile64"),
    ((2880, 1440, 1056), "tile64"), ((1, 1, (1 << 24) + 32), "staged"), ((16, 8192, 2880), "tile32"),
    ((8192, 8192, 8192), "dma"), ((4096, 8192, (1 << 24) + 32), "staged")])
def test_kernel_of_a_product(size, kernel):
    assert hm.gemm_kernel(*size) == kernel


def test_products_leave_the_choice_only_for_filled_tiles():
    rng = random.Random(4660)
    for _ in range(20000):
        M, N = (int(2 ** rng.uniform(0, 18)) for _ in range(2))
        K = 32 * int(2 ** rng.uniform(0, 20))
        kernel, chosen = hm.gemm_kernel(M, N, K), hm.choose_gemm(M, N, K)
        if kernel != chosen:
            assert kernel in TILES and K <= 1 << 24 and M > 64 and N > 64, (M, N, K, kernel)
            bm, bn = TILES[kernel]
            tm, tn = -(-M // bm), -(-N // bn)
            assert tm * tn >= 0.62 * 256 and M * N > 0.3 * tm * tn * bm * bn, (M, N, K, kernel)
            assert hm.gemm_lanes(kernel, M, N) < 1 << 32, (M, N, K, kernel)
        else:
            assert hm.gemm_lanes(kernel, M, N) < 1 << 32 or hm.gemm_lanes("dma", M, N) >= 1 << 32, (M, N, K)


# 256 x 256: one unit of 32 steps; one chunk less a unit, two and three units; a chunk and one, two, three units; the
# ring of four stages just filled, and gone round; rows and columns past the edges, an odd N
SIZES = [(3300, 3400, 32, ""), (3312, 3401, 64, "a"), (3300, 3399, 96, ""), (3300, 3408, 160, "b"),
         (3312, 3408, 192, "ab"), (3329, 3400, 224, ""), (3300, 3331, 480, ""), (3301, 3400, 544, ""),
         (3300, 3411, 704, ""), (3300, 3400, 1184, "")]
SIZES = [("dma", *size) for size in SIZES] + [
    # whole chunks: one; the ring just filled, and gone round
    ("dma", 3300, 3401, 128, ""), ("dma", 3312, 3407, 512, "a"), ("dma", 3329, 3331, 768, ""),
    # 256 x 128 (five stages of 128): a unit, a chunk, a chunk and a unit, ...; N odd, and one column past a tile
    ("dma256x128", 1000, 5232, 32, ""), ("dma256x128", 992, 5231, 128, "a"), ("dma256x128", 1024, 5249, 160, ""),
    ("dma256x128", 961, 5248, 512, "b"), ("dma256x128", 1000, 5227, 544, ""), ("dma256x128", 1000, 5232, 640, ""),
    ("dma256x128", 1001, 5230, 672, ""), ("dma256x128", 1000, 5236, 896, ""), ("dma256x128", 1008, 5232, 1184, "ab"),
    ("dma256x128", 130, 32768, 128, ""),
    # ... and every remainder of N by the 8 (BF16) or 4 (fp32) columns that a lane stores
    ("dma256x128", 1000, 5226, 64, ""), ("dma256x128", 992, 5229, 96, ""), ("dma256x128", 1000, 5240, 96, ""),
    # 128 x 128 (four stages of 256, each wave a quarter of them)
    ("dma128", 1000, 3000, 1024, ""), ("dma128", 1024, 3071, 1056, ""), ("dma128", 897, 3072, 1120, ""),
    ("dma128", 992, 2945, 1152, "a"), ("dma128", 1001, 3056, 1248, "b"), ("dma128", 1000, 3001, 1280, ""),
    ("dma128", 193, 14000, 1536, ""), ("dma128", 127, 28611, 1312, "")]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,M,N,K,tiled", SIZES)
def test_products_in_large_tiles_are_exact(kernel, M, N, K, tiled):
    """Codes on the grid, scales 0.5 .. 4: every product is a multiple of 1/8 and their magnitudes add up to less
    than 2^21, so every partial sum is exact in fp32 whatever the order."""
    from paper_2512_02010_amd import binding as B
    assert hm.gemm_kernel(M, N, K) == kernel
    print(f"gemm {kernel} case M={M} N={N} K={K} tiled={tiled!r}", flush=True)
    rng = np.random.default_rng(M * 7919 + N * 31 + K)
    grid = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])

    def operand(rows, tiles, scale_bytes, values):
        codes = rng.integers(0, 256, (rows, K // 2), dtype=np.uint8)
        pick = rng.integers(0, 3, (rows // 16 if tiles else rows, K // 16))
        s = np.repeat(np.array(values)[pick], 16, axis=1)
        v = np.stack((grid[codes & 15], grid[codes >> 4]), axis=-1).reshape(rows, K)
        v = v * (np.repeat(s, 16, axis=0) if tiles else s)
        return torch.from_numpy(codes).cuda(), torch.from_numpy(np.array(scale_bytes, np.uint8)[pick]).cuda(), v

    ca, sa, va = operand(M, "a" in tiled, (0x30, 0x38, 0x40), (0.5, 1.0, 2.0))
    cb, sb, vb = operand(N, "b" in tiled, (0x38, 0x40, 0x48), (1.0, 2.0, 4.0))
    want = va @ vb.T
    assert (np.abs(va) @ np.abs(vb).T).max() < 2.0 ** 21
    one = torch.ones(1, dtype=torch.float32, device="cuda")
    flags = (B.GEMM_A_TILE_SCALES if "a" in tiled else 0) | (B.GEMM_B_TILE_SCALES if "b" in tiled else 0)
    got = B.nvfp4_46_gemm(ca, sa, one, cb, sb, one, out_dtype=B.OUT_F32, flags=flags)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), want)
    got16 = B.nvfp4_46_gemm(ca, sa, one, cb, sb, one, out_dtype=B.OUT_BF16, flags=flags)
    assert torch.equal(got16.cpu(), torch.from_numpy(want.astype(np.float32)).to(torch.bfloat16))
