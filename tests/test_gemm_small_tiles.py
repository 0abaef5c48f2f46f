"""GPU: products in the tiles of k_gemm_tile: every length of the last chunk (the copies of the tile that have a piece of
it multiply, the others do not), tiles whole and cut by an edge of C, more workgroups than compute units."""
import numpy as np
import pytest
import torch

from . import _host_model as hm

# K = whole chunks, and chunks and 1, 2, 3, ... units of 32 steps, up to one short of a chunk
SIZES = [("tile32", 40, 520, 32), ("tile32", 33, 500, 512), ("tile32", 64, 1024, 1056), ("tile32", 90, 2010, 736),
         ("tile32", 128, 2000, 992), ("tile32", 64, 1023, 1024),
         ("tile64x32", 100, 3000, 256), ("tile64x32", 97, 3001, 288), ("tile64x32", 128, 3008, 576),
         ("tile64x32", 100, 3000, 608), ("tile64x32", 101, 2999, 480),
         ("tile64", 200, 4096, 512), ("tile64", 2880, 1440, 32), ("tile64", 2881, 1441, 320), ("tile64", 1501, 1433, 352),
         ("tile64", 1500, 1440, 160), ("tile64", 300, 2000, 480), ("tile64", 1472, 1408, 768), ("tile64", 2880, 1440, 1056),
         # ... scales before the first chunk (K from 1024 to 2016, no whole chunks): the last 16 bytes of a tile's whole and cut
         ("tile64", 575, 2049, 1056), ("tile64", 513, 2001, 1120), ("tile64", 901, 1601, 2016), ("tile64", 1001, 1000, 1312),
         ("tile64", 592, 2064, 1056, "a"), ("tile64", 575, 2064, 1184, "b"), ("tile64", 912, 1616, 2016, "ab"),
         ("tile64", 901, 1601, 2080),
         ("tile64long", 141, 4652, 8256), ("tile64long", 128, 4700, 8672), ("tile64long", 192, 4096, 8704),
         ("tile64long", 191, 4097, 8320),
         ("tile128", 1000, 4096, 800), ("tile128", 1000, 3900, 640), ("tile128", 990, 3999, 736),
         ("tile128", 1024, 4096, 768), ("tile128", 1000, 3901, 928),
         ("tile256x128", 2048, 4095, 640), ("tile256x128", 2000, 4094, 352), ("tile256x128", 1999, 4093, 96)]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,M,N,K,tiled", [(*size, "")[:5] for size in SIZES])
def test_products_in_small_tiles_are_exact(kernel, M, N, K, tiled):
    """Codes on the grid, scales 0.5 .. 2: every product is a multiple of 1/16 and their magnitudes add up to less
    than 2^20, so every partial sum is exact in fp32 whatever the order."""
    from paper_2512_02010_amd import binding as B
    assert (hm.choose_gemm(M, N, K), hm.choose_gemm(M, N, K, f32=True)) == (kernel, kernel)
    print(f"gemm {kernel} case M={M} N={N} K={K} tiled={tiled!r}", flush=True)
    rng = np.random.default_rng(M * 7919 + N * 31 + K)
    grid = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])

    def operand(rows, tiles):
        codes = rng.integers(0, 256, (rows, K // 2), dtype=np.uint8)
        pick = rng.integers(0, 3, (rows // 16 if tiles else rows, K // 16))
        s = np.repeat(np.array((0.5, 1.0, 2.0))[pick], 16, axis=1)
        v = np.stack((grid[codes & 15], grid[codes >> 4]), axis=-1).reshape(rows, K)
        v = v * (np.repeat(s, 16, axis=0) if tiles else s)
        return torch.from_numpy(codes).cuda(), torch.from_numpy(np.array((0x30, 0x38, 0x40), np.uint8)[pick]).cuda(), v

    ca, sa, va = operand(M, "a" in tiled)
    cb, sb, vb = operand(N, "b" in tiled)
    want = va @ vb.T
    assert (np.abs(va) @ np.abs(vb).T).max() < 2.0 ** 20
    one = torch.ones(1, dtype=torch.float32, device="cuda")
    flags = (B.GEMM_A_TILE_SCALES if "a" in tiled else 0) | (B.GEMM_B_TILE_SCALES if "b" in tiled else 0)
    got = B.nvfp4_46_gemm(ca, sa, one, cb, sb, one, out_dtype=B.OUT_F32, flags=flags)
    got16 = B.nvfp4_46_gemm(ca, sa, one, cb, sb, one, out_dtype=B.OUT_BF16, flags=flags)
    assert torch.equal(got16.cpu(), torch.from_numpy(want.astype(np.float32)).to(torch.bfloat16))
    assert np.array_equal(got.cpu().numpy().astype(np.float64), want)
