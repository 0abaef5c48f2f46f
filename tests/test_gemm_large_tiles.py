"""GPU: products in the large tiles of k_gemm_dma (256 x 256, 256 x 128 and 128 x 128)."""
import numpy as np
import pytest
import torch

from . import _host_model as hm

# 256 x 256: one unit of 32 steps; one chunk less a unit, two and three units; a chunk and one, two, three units; the
# ring of four stages just filled, and gone round; rows and columns past the edges, an odd N
SIZES = [(3300, 3400, 32, ""), (3312, 3401, 64, "a"), (3300, 3399, 96, ""), (3300, 3408, 160, "b"),
         (3312, 3408, 192, "ab"), (3329, 3400, 224, ""), (3300, 3331, 480, ""), (3301, 3400, 544, ""),
         (3300, 3411, 704, ""), (3300, 3400, 1184, "")]
SIZES = [("dma", *size) for size in SIZES] + [
    # whole chunks: one; the ring just filled, and gone round
    ("dma", 3300, 3401, 128, ""), ("dma", 3312, 3407, 512, "a"), ("dma", 3329, 3331, 768, ""),
    # 256 x 128 (five stages of 128): a unit, a chunk, a chunk and a unit, ...
    ("dma256x128", 1000, 5232, 32, ""), ("dma256x128", 992, 5232, 128, "a"), ("dma256x128", 1024, 5256, 160, ""),
    ("dma256x128", 961, 5248, 512, "b"), ("dma256x128", 1000, 5224, 544, ""), ("dma256x128", 1000, 5232, 640, ""),
    ("dma256x128", 1001, 5240, 672, ""), ("dma256x128", 1000, 5232, 896, ""), ("dma256x128", 1008, 5232, 1184, "ab"),
    ("dma256x128", 130, 32768, 128, ""),
    # ... N odd, one column past a tile, and with every remainder by the 8 (BF16) or 4 (fp32) columns that a lane stores
    ("dma256x128", 992, 5231, 1024, "a"), ("dma256x128", 1024, 5249, 1056, ""), ("dma256x128", 1000, 5227, 1152, ""),
    ("dma256x128", 1001, 5230, 1184, ""), ("dma256x128", 1000, 5236, 1024, ""), ("dma256x128", 1000, 5226, 1088, ""),
    ("dma256x128", 992, 5229, 1280, "a"),
    # 128 x 128 (four stages of 256, each wave a quarter of them)
    ("dma128", 1000, 3000, 1024, ""), ("dma128", 1024, 3064, 1056, ""), ("dma128", 897, 3072, 1120, ""),
    ("dma128", 992, 2952, 1152, "a"), ("dma128", 1001, 3056, 1248, "b"), ("dma128", 1000, 3008, 1280, ""),
    ("dma128", 193, 14000, 1536, ""), ("dma128", 127, 28608, 1312, ""),
    ("dma128", 1024, 3071, 2080, ""), ("dma128", 992, 2945, 2048, "a"), ("dma128", 1000, 3001, 2304, ""),
    ("dma128", 127, 28611, 2144, ""), ("dma128", 1000, 3002, 2272, "")]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,M,N,K,tiled", SIZES)
def test_products_in_large_tiles_are_exact(kernel, M, N, K, tiled):
    """Codes on the grid, scales 0.5 .. 4: every product is a multiple of 1/8 and their magnitudes add up to less
    than 2^21, so every partial sum is exact in fp32 whatever the order."""
    from paper_2512_02010_amd import binding as B
    assert (hm.choose_gemm(M, N, K), hm.choose_gemm(M, N, K, f32=True)) == (kernel, kernel)
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
