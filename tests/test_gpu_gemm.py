"""GPU: the NVFP4 x NVFP4 matrix product against the CPU oracle, through the C ABI.

The operands are expanded exactly and every product is exact; the matrix unit accumulates in
fp32 in its own order.  Any fp32 summation of K exact products differs from the exact sum by
at most (K - 1) 2^-24 sum|a b| (1 + O(K 2^-24)); the bound used is twice that, 2 K 2^-24, so
that a matrix unit that truncates instead of rounding its partial sums still passes.  On top
come the rounding of alpha_a * alpha_b and of the scaled result (2 * 2^-24 relative) and of
the output (half an ulp: at most 2^-24 for fp32 and 2^-8 for BF16, relative to the result).  Where every partial sum
is exactly representable the comparison is bit for bit."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2512_02010_amd import binding as B
from paper_2512_02010_amd import workloads as wl
from tests import _host_model as hm

pytestmark = pytest.mark.gpu


def _log(msg):
    print(msg, flush=True)


def _operand(name, rows, K, **kw):
    """(codes, scales, alpha) of a synthetic tensor quantized by the oracle."""
    bits = wl.bf16_bits(wl.make(name, rows, K))
    alpha = ref.tensor_scale(bits)
    codes, scales, _ = ref.quantize(bits, alpha, **kw)
    return codes, scales, alpha


def _dev(a):
    return torch.from_numpy(a).cuda()


def _alpha(a):
    return torch.tensor([a], dtype=torch.float32, device="cuda")


def _bf16_to_f64(t):
    return t.float().double().cpu().numpy()


def _tolerance(c_ref, c_abs, K, out_dtype):
    out_eps = 2.0 ** -24 if out_dtype == B.OUT_F32 else 2.0 ** -8
    return 2.0 * K * 2.0 ** -24 * c_abs + (out_eps + 2.0 ** -22) * np.abs(c_ref) + 1e-300


def check_gemm(A, Bm, out_dtype, tag):
    (ca, sa, aa), (cb, sb, ab) = A, Bm
    M, N, K = ca.shape[0], cb.shape[0], ca.shape[1] * 2
    _log(f"gemm case {tag} M={M} N={N} K={K} out_dtype={out_dtype}")
    c_ref, c_abs = ref.gemm(ca, sa, aa, cb, sb, ab, want_abs=True)
    got = B.nvfp4_46_gemm(_dev(ca), _dev(sa), _alpha(aa), _dev(cb), _dev(sb), _alpha(ab),
                          out_dtype=out_dtype)
    torch.cuda.synchronize()
    g = got.double().cpu().numpy() if out_dtype == B.OUT_F32 else _bf16_to_f64(got)
    assert g.shape == (M, N)
    err = np.abs(g - c_ref)
    tol = _tolerance(c_ref, c_abs, K, out_dtype)
    bad = np.argwhere(err > tol)
    assert len(bad) == 0, (tag, len(bad), bad[:4].tolist(), g[tuple(bad[0])], c_ref[tuple(bad[0])])
    # the bound is far from tight: typical errors sit near sqrt(K) 2^-24
    _log(f"  max err / tol = {float((err / tol).max()):.3f}")
    return g, c_ref


SHAPES = [(32, 32, 32), (1, 1, 64), (100, 70, 160), (256, 256, 128), (257, 255, 384),
          (300, 520, 1056), (512, 768, 2048), (200, 300, 256),
          # few rows of A and K a multiple of 256: up to 32 rows the kernels that stream B (up to 16 the
          # 16-row one), then 32 x 32 tiles
          (1, 40, 256), (16, 32, 512), (33, 100, 1024), (64, 1000, 2304), (100, 96, 768),
          (128, 257, 512), (129, 64, 512),
          (7, 45, 256), (16, 64, 768), (9, 1000, 2304), (3, 17, 4096), (17, 33, 256),
          # more rows of A, ragged tiles
          (257, 255, 768), (384, 300, 256), (511, 40, 1024), (513, 40, 512)]


@pytest.mark.parametrize("out_dtype", [B.OUT_F32, B.OUT_BF16])
@pytest.mark.parametrize("shape", SHAPES)
def test_gemm_matches_oracle(shape, out_dtype):
    M, N, K = shape
    check_gemm(_operand("c3", M, K), _operand("c2", N, K), out_dtype, "c3xc2")


@pytest.mark.parametrize("shape", [(64, 96, 256), (130, 260, 1120)])
def test_gemm_wide_range_operands(shape):
    # gradients with rows spread over many octaves (scale bytes down to subnormal E4M3)
    # against a weight matrix with outlier columns; stochastic rounding on the gradient side
    M, N, K = shape
    A = _operand("c5", M, K, rounding=ref.SR, sr_seed=wl.C5_SR_SEED)
    g, c_ref = check_gemm(A, _operand("c2", N, K), B.OUT_F32, "c5xc2")
    if M >= 128:
        assert (A[1] < 8).any()      # subnormal scale bytes do occur in this operand


def test_gemm_is_exact_when_every_partial_sum_is_representable():
    """Scale 1, codes on small multiples of 0.5: every product is a multiple of 0.25 below
    36, every partial sum a multiple of 0.25 below 2^22, so fp32 accumulation is exact in any
    order and the result must equal the oracle's bit for bit (alpha = 1)."""
    rng = np.random.default_rng(46)
    M, N, K = 160, 288, 1024
    ca = rng.integers(0, 256, (M, K // 2), dtype=np.uint8)
    cb = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    sa = rng.choice(np.array([0x30, 0x38, 0x40], np.uint8), (M, K // 16))    # 0.5, 1, 2
    sb = rng.choice(np.array([0x38, 0x40, 0x48], np.uint8), (N, K // 16))    # 1, 2, 4
    c_ref = ref.gemm(ca, sa, 1.0, cb, sb, 1.0)
    assert np.array_equal(c_ref, c_ref.astype(np.float32).astype(np.float64))
    got = B.nvfp4_46_gemm(_dev(ca), _dev(sa), _alpha(1.0), _dev(cb), _dev(sb), _alpha(1.0),
                          out_dtype=B.OUT_F32)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), c_ref)
    # and the BF16 output is the round-to-nearest-even of those exact values
    got16 = B.nvfp4_46_gemm(_dev(ca), _dev(sa), _alpha(1.0), _dev(cb), _dev(sb), _alpha(1.0),
                            out_dtype=B.OUT_BF16)
    want16 = torch.from_numpy(c_ref.astype(np.float32)).to(torch.bfloat16)
    assert torch.equal(got16.cpu(), want16)


@pytest.mark.parametrize("M", [1, 5, 16, 17, 30, 64, 128, 200, 512])
def test_small_batch_gemm_is_exact_when_every_partial_sum_is_representable(M):
    """The same argument for few rows of A (the 16-row and 32-row streaming kernels, then 32 x 32 tiles):
    scales 0.5 .. 4, so every sum is exact in fp32 in any order."""
    rng = np.random.default_rng(4600 + M)
    N, K = 77, 768
    ca = rng.integers(0, 256, (M, K // 2), dtype=np.uint8)
    cb = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    sa = rng.choice(np.array([0x30, 0x38, 0x40], np.uint8), (M, K // 16))
    sb = rng.choice(np.array([0x38, 0x40, 0x48], np.uint8), (N, K // 16))
    c_ref = ref.gemm(ca, sa, 1.0, cb, sb, 1.0)
    assert np.array_equal(c_ref, c_ref.astype(np.float32).astype(np.float64))
    got = B.nvfp4_46_gemm(_dev(ca), _dev(sa), _alpha(1.0), _dev(cb), _dev(sb), _alpha(1.0),
                          out_dtype=B.OUT_F32)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), c_ref)


# Every kernel that is picked by the sizes, at the edges of its tiles and of its chunks of the
# contraction axis (128 to 512 indices), with K whole and, where it may be, ragged; the operands
# in `tiled` carry one scale line per 16 rows.
TILE_SHAPES = {
    "tile32": [(1, 1, 32, ""), (31, 33, 64, ""), (48, 64, 512, "ab"), (33, 32, 544, "b"),
               (250, 997, 1056, ""), (7, 9001, 4128, ""), (2111, 31, 992, ""), (66, 4100, 8192, "")],
    "tile64x32": [(304, 848, 96, "ab"), (301, 833, 256, ""), (320, 831, 288, "a"), (17000, 31, 992, "")],
    "tile64": [(701, 799, 32, ""), (705, 769, 512, ""), (704, 784, 800, "ab"), (64, 17008, 96, "ab"),
               (1100, 1500, 4128, "")],          # (operands past one die's L2: the tiles in strips, the last narrower)
    "tile64long": [(129, 4203, 8192, ""), (144, 4208, 8224, "ab"), (705, 1300, 9696, "")],
    "tile128": [(1901, 1920, 288, "b"), (1793, 1921, 256, ""), (100, 28677, 320, ""), (1904, 1920, 768, "ab"),
                (1901, 1928, 992, ""), (1793, 1921, 1888, "")],
    "tile256x128": [(2177, 2945, 96, ""), (2192, 2945, 416, "a"), (2177, 2947, 928, ""), (1344, 13184, 128, "ab"),
                    (1338, 13184, 1824, "b")],
    # the kernels that stream B: 16 rows, 32 rows, 64 rows
    "skinny": [(16, 1008, 512, "ab"), (5, 4099, 768, ""), (32, 64, 512, "ab"), (31, 4099, 256, ""),
               (33, 4100, 256, ""), (50, 8203, 768, ""), (64, 4112, 768, "ab"), (48, 16384, 256, "a"),
               (63, 5008, 512, "b")],
    # 256 x 256 tiles by copies: one, two and three chunks (test_gemm_large_tiles.py has more)
    "dma": [(3300, 3400, 128, ""), (3300, 3400, 256, ""), (3311, 3393, 384, ""), (3312, 3400, 256, "a"),
            (3300, 3408, 384, "b"), (3312, 3408, 128, "ab")]}
TILE_SHAPES = [(kernel, *size) for kernel, sizes in TILE_SHAPES.items() for size in sizes]


@pytest.mark.parametrize("kernel,M,N,K,tiled", TILE_SHAPES)
def test_tile_shapes_are_exact_when_every_partial_sum_is_representable(kernel, M, N, K, tiled):
    """Scales 0.5 .. 4 as above: every product is a multiple of 1/8, and the magnitudes of an element's
    products add up to less than 2^21 (checked), so all partial sums are exact in fp32 (2^21 / 2^-3 =
    2^24) in any order and the result is the oracle's bit for bit."""
    assert (hm.choose_gemm(M, N, K), hm.choose_gemm(M, N, K, f32=True)) == (kernel, kernel)
    _log(f"gemm {kernel} case M={M} N={N} K={K} tiled={tiled!r}")
    rng = np.random.default_rng(M * 7919 + N * 31 + K)
    ca = rng.integers(0, 256, (M, K // 2), dtype=np.uint8)
    cb = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    la, lb = (M // 16 if "a" in tiled else M), (N // 16 if "b" in tiled else N)
    sa = rng.choice(np.array([0x30, 0x38, 0x40], np.uint8), (la, K // 16))
    sb = rng.choice(np.array([0x38, 0x40, 0x48], np.uint8), (lb, K // 16))
    flags = (B.GEMM_A_TILE_SCALES if "a" in tiled else 0) | (B.GEMM_B_TILE_SCALES if "b" in tiled else 0)
    got = B.nvfp4_46_gemm(_dev(ca), _dev(sa), _alpha(1.0), _dev(cb), _dev(sb), _alpha(1.0),
                          out_dtype=B.OUT_F32, flags=flags)
    # (the products of decoded values; float64 sums of multiples of 1/8 below 2^21 are exact too)
    grid = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])
    value = {0x30: 0.5, 0x38: 1.0, 0x40: 2.0, 0x48: 4.0}

    def decoded(codes, scales, lines):
        v = np.stack((grid[codes & 15], grid[codes >> 4]), axis=-1).reshape(codes.shape[0], -1)
        s = np.repeat(np.vectorize(value.get)(scales), 16, axis=1)
        return v * (np.repeat(s, 16, axis=0) if lines != codes.shape[0] else s)

    da, db = decoded(ca, sa, la), decoded(cb, sb, lb)
    want = da @ db.T
    assert (np.abs(da) @ np.abs(db).T).max() < 2.0 ** 21
    assert np.array_equal(got.cpu().numpy().astype(np.float64), want)
    got16 = B.nvfp4_46_gemm(_dev(ca), _dev(sa), _alpha(1.0), _dev(cb), _dev(sb), _alpha(1.0),
                            out_dtype=B.OUT_BF16, flags=flags)
    assert torch.equal(got16.cpu(), torch.from_numpy(want.astype(np.float32)).to(torch.bfloat16))


def test_small_batch_gemm_with_tile_scaled_operands():
    """Sixteen rows of A and a B operand, both quantized in 16x16 tiles (one scale line per
    16 rows), through the 16-row kernel; and the same B against 32 rows of A."""
    K, N = 512, 48
    for M in (16, 32):
        ops, ref_ops = [], []
        for rows, name in ((M, "c3"), (N, "c2")):
            bits = wl.bf16_bits(wl.make(name, rows, K, seed=7100 + rows))
            a = ref.tensor_scale(bits)
            c, s, _, _ = ref.quantize_2d(bits, a)
            ref_ops += [c, s, a]
            ops += [_dev(c), _dev(s), _alpha(a)]
        flags = B.GEMM_A_TILE_SCALES | B.GEMM_B_TILE_SCALES
        c_ref, c_abs = ref.gemm(*ref_ops, want_abs=True, tiles_a=True, tiles_b=True)
        got = B.nvfp4_46_gemm(*ops, out_dtype=B.OUT_F32, flags=flags).double().cpu().numpy()
        assert (np.abs(got - c_ref) <= _tolerance(c_ref, c_abs, K, B.OUT_F32)).all(), M


def test_gemm_every_scale_byte_and_code():
    """Each of the 127 scale bytes 0x00..0x7E and all sixteen codes, one at a time against a
    unit operand: C[m][n] = 16 * value(code) * value(scale) exactly."""
    K = 32
    ca = np.zeros((127 * 16, K // 2), np.uint8)
    sa = np.zeros((127 * 16, K // 16), np.uint8)
    for s in range(127):
        for c in range(16):
            ca[s * 16 + c, :8] = c | (c << 4)        # sixteen copies of code c in block 0
            sa[s * 16 + c, 0] = s
    cb = np.full((40, K // 2), 0x22, np.uint8)       # all 1.0
    sb = np.full((40, K // 16), 0x38, np.uint8)
    c_ref = ref.gemm(ca, sa, 1.0, cb, sb, 1.0)
    got = B.nvfp4_46_gemm(_dev(ca), _dev(sa), _alpha(1.0), _dev(cb), _dev(sb), _alpha(1.0),
                          out_dtype=B.OUT_F32).cpu().numpy().astype(np.float64)
    assert np.array_equal(got, c_ref)
    assert got[0x7E * 16 + 7, 0] == 16 * 6 * 448 and got[1 * 16 + 1, 3] == 16 * 0.5 * 2.0 ** -9


def test_gemm_is_reproducible_and_runs_on_a_side_stream():
    A, Bm = _operand("c1", 300, 512), _operand("c4", 200, 512)
    args = [_dev(A[0]), _dev(A[1]), _alpha(A[2]), _dev(Bm[0]), _dev(Bm[1]), _alpha(Bm[2])]
    first = B.nvfp4_46_gemm(*args, out_dtype=B.OUT_F32)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        again = [B.nvfp4_46_gemm(*args, out_dtype=B.OUT_F32, stream=s) for _ in range(3)]
    s.synchronize()
    for o in again:
        assert torch.equal(o, first)


def test_gemm_error_paths():
    A = _operand("c1", 32, 64)
    args = [_dev(A[0]), _dev(A[1]), _alpha(A[2]), _dev(A[0]), _dev(A[1]), _alpha(A[2])]
    out = torch.full((32, 32), 7.0, dtype=torch.float32, device="cuda")
    assert B.gemm_raw(*args, 32, 32, 48, B.OUT_F32, out) == 2          # K % 32 != 0
    assert B.gemm_raw(*args, 0, 32, 64, B.OUT_F32, out) == 2
    assert B.gemm_raw(*args, 32, 32, 64, 2, out) == 4
    assert B.gemm_raw(args[0], None, *args[2:], 32, 32, 64, B.OUT_F32, out) == 1
    assert B.gemm_raw(*args, 32, 32, 64, B.OUT_F32, out.data_ptr() + 4) == 3
    torch.cuda.synchronize()
    assert bool((out == 7.0).all())


def test_gemm_full_size_sampled():
    """8192 x 8192 x 8192 (activations c3-like rows against the c2 weight matrix) in the
    configuration the benchmark times; the oracle recomputes 96 x 96 sampled outputs."""
    K = 8192
    A = _operand("c3", 8192, K)
    Bm = _operand("c2", 8192, K)
    got = B.nvfp4_46_gemm(_dev(A[0]), _dev(A[1]), _alpha(A[2]), _dev(Bm[0]), _dev(Bm[1]),
                          _alpha(Bm[2]), out_dtype=B.OUT_BF16)
    torch.cuda.synchronize()
    rng = np.random.default_rng(8192)
    rows = np.sort(np.concatenate([rng.choice(8192, 90, replace=False), [0, 255, 256, 4095, 8191, 31]]))
    cols = np.sort(np.concatenate([rng.choice(8192, 90, replace=False), [0, 127, 128, 4096, 8191, 63]]))
    c_ref, c_abs = ref.gemm(np.ascontiguousarray(A[0][rows]), np.ascontiguousarray(A[1][rows]),
                            A[2], np.ascontiguousarray(Bm[0][cols]),
                            np.ascontiguousarray(Bm[1][cols]), Bm[2], want_abs=True)
    g = _bf16_to_f64(got[torch.from_numpy(rows).cuda()][:, torch.from_numpy(cols).cuda()])
    err = np.abs(g - c_ref)
    tol = _tolerance(c_ref, c_abs, K, B.OUT_BF16)
    assert (err <= tol).all(), float((err / tol).max())
    _log(f"  full size: max err / tol = {float((err / tol).max()):.3f}")


def test_linear_layer_three_products_of_figure_3():
    """FPROP, DGRAD and WGRAD of one linear layer (Fig. 3), each as quantize -> NVFP4 product on
    the GPU, against the oracle's quantize -> product; the operand that a product needs along
    its other axis is the quantizer's columnwise output.  Gradients use stochastic rounding,
    the weight-gradient operands the random Hadamard transform (which cancels in the product
    because both operands carry the same signs along the contraction axis)."""
    T, K, N = 192, 256, 160                       # tokens, in features, out features
    x = wl.make("c3", T, K)
    w = wl.make("c2", N, K)
    dy = wl.make("c5", T, N)
    SR_SEED, RHT_SEED = wl.C5_SR_SEED, wl.C5_RHT_SEED

    def both_sides(t, layout, **kw):
        """Quantize on the GPU and with the oracle; returns (gpu operand, oracle operand)."""
        bits, td = wl.bf16_bits(t), t.cuda()
        rht = kw.get("rht", 0)
        a_gpu = B.nvfp4_46_tensor_scale(td, layout=layout, rht=rht, rht_seed=kw.get("rht_seed", 0))
        a_ref = ref.tensor_scale(bits, layout=layout, rht=rht, rht_seed=kw.get("rht_seed", 0))
        assert a_gpu.item() == a_ref
        o = B.nvfp4_46_quantize(td, a_gpu, layout=layout, **kw)
        sfx = "row" if layout == B.ROWWISE else "col"
        c_ref, s_ref, _ = ref.quantize(bits, a_ref, layout=layout, **kw)
        assert np.array_equal(o[f"codes_{sfx}"].cpu().numpy(), c_ref)
        return (o[f"codes_{sfx}"], o[f"scales_{sfx}"], a_gpu), (c_ref, s_ref, a_ref)

    def product(A, Bm, exact, what, rel):
        (ga, ra), (gb, rb) = A, Bm
        got = B.nvfp4_46_gemm(*ga, *gb, out_dtype=B.OUT_F32).double().cpu().numpy()
        c_ref, c_abs = ref.gemm(*ra, *rb, want_abs=True)
        Kc = ra[0].shape[1] * 2
        assert (np.abs(got - c_ref) <= _tolerance(c_ref, c_abs, Kc, B.OUT_F32)).all(), what
        err = np.sqrt(((got - exact) ** 2).mean()) / np.sqrt((exact ** 2).mean())
        _log(f"  {what}: relative RMS error against the unquantized product {err:.3f}")
        assert err < rel, (what, err)

    xd, wd, dyd = x.double().numpy(), w.double().numpy(), dy.double().numpy()
    sr = dict(rounding=B.SR, sr_seed=SR_SEED)
    rht = dict(rht=1, rht_seed=RHT_SEED)
    # FPROP  y = x w^T          (contraction over K: x rowwise, w rowwise)
    product(both_sides(x, B.ROWWISE), both_sides(w, B.ROWWISE), xd @ wd.T, "FPROP", 0.25)
    # DGRAD  dx = dy w          (over N: dy rowwise with SR, w columnwise)
    product(both_sides(dy, B.ROWWISE, **sr), both_sides(w, B.COLWISE), dyd @ wd, "DGRAD", 0.25)
    # WGRAD  dw = dy^T x        (over T: dy columnwise with RHT + SR, x columnwise with RHT)
    product(both_sides(dy, B.COLWISE, **sr, **rht), both_sides(x, B.COLWISE, **rht), dyd.T @ xd,
            "WGRAD", 0.25)


@pytest.mark.parametrize("M,N,K", [(320, 272, 512), (320, 272, 544),        # small tiles, K whole and ragged
                                   (20, 272, 512), (3300, 3400, 256)])       # streaming B; 256 x 256 tiles
def test_gemm_can_be_captured_in_a_graph_and_replayed(M, N, K):
    A, Bm = _operand("c3", M, K), _operand("c2", N, K)
    args = [_dev(A[0]), _dev(A[1]), _alpha(A[2]), _dev(Bm[0]), _dev(Bm[1]), _alpha(Bm[2])]
    out = torch.empty((M, N), dtype=torch.float32, device="cuda")
    want = B.nvfp4_46_gemm(*args, out_dtype=B.OUT_F32).clone()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        B.nvfp4_46_gemm(*args, out_dtype=B.OUT_F32, out=out, stream=s)     # warm-up
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        B.nvfp4_46_gemm(*args, out_dtype=B.OUT_F32, out=out, stream=torch.cuda.current_stream())
    for _ in range(3):
        out.zero_()                     # eager work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


@pytest.mark.parametrize("K", [256, 416])      # whole chunks of 256, and none
def test_gemm_with_weights_quantized_in_16x16_tiles(K):
    """FPROP and DGRAD with a weight matrix quantized once in 16x16 tiles (Section 4.1): the
    row packing multiplies activations, the packing for W^T multiplies gradients, and the
    product only has to be told that the operand's scales come one line per 16 rows."""
    T, N = 200, 320
    w = wl.make("c2", N, K)
    wb, wd = wl.bf16_bits(w), w.cuda()
    aw = B.nvfp4_46_tensor_scale(wd)
    a_w = float(aw.item())
    qw = B.nvfp4_46_quantize(wd, aw, layout=B.BOTH, block2d=1)
    c_ref, s_ref, f_ref, _ = ref.quantize_2d(wb, a_w)
    cc_ref, sc_ref, _ = ref.repack_2d_columnwise(c_ref, s_ref, f_ref)
    assert np.array_equal(qw["codes_row"].cpu().numpy(), c_ref)
    assert np.array_equal(qw["codes_col"].cpu().numpy(), cc_ref)

    def check(A, codes_w, scales_w, ref_w, flags_gpu, what, **tiles):
        got = B.nvfp4_46_gemm(_dev(A[0]), _dev(A[1]), _alpha(A[2]), codes_w, scales_w, aw,
                              out_dtype=B.OUT_F32, flags=flags_gpu).double().cpu().numpy()
        c, c_abs = ref.gemm(A[0], A[1], A[2], ref_w[0], ref_w[1], a_w, want_abs=True, **tiles)
        Kc = A[0].shape[1] * 2
        assert (np.abs(got - c) <= _tolerance(c, c_abs, Kc, B.OUT_F32)).all(), what
        return got

    x = _operand("c3", T, K)
    y = check(x, qw["codes_row"], qw["scales_row"], (c_ref, s_ref), B.GEMM_B_TILE_SCALES, "FPROP",
              tiles_b=True)
    assert y.shape == (T, N)
    dy = _operand("c5", T, N, rounding=ref.SR, sr_seed=wl.C5_SR_SEED)
    dx = check(dy, qw["codes_col"], qw["scales_col"], (cc_ref, sc_ref), B.GEMM_B_TILE_SCALES,
               "DGRAD", tiles_b=True)
    assert dx.shape == (T, K)
    # the tile-scaled operand on the A side
    got = B.nvfp4_46_gemm(qw["codes_row"], qw["scales_row"], aw, _dev(x[0]), _dev(x[1]),
                          _alpha(x[2]), out_dtype=B.OUT_F32, flags=B.GEMM_A_TILE_SCALES)
    c, c_abs = ref.gemm(c_ref, s_ref, a_w, x[0], x[1], x[2], want_abs=True, tiles_a=True)
    assert (np.abs(got.double().cpu().numpy() - c) <= _tolerance(c, c_abs, K, B.OUT_F32)).all()


def test_gemm_flag_validation():
    A = _operand("c1", 40, 64)
    args = [_dev(A[0]), _dev(A[1]), _alpha(A[2]), _dev(A[0]), _dev(A[1]), _alpha(A[2])]
    out = torch.empty((40, 40), dtype=torch.float32, device="cuda")
    assert B.gemm_raw(*args, 40, 40, 64, B.OUT_F32, out, flags=4) == 4
    assert B.gemm_raw(*args, 40, 40, 64, B.OUT_F32, out, flags=B.GEMM_A_TILE_SCALES) == 2   # 40 % 16


def test_gemm_seeded_sweep_of_shapes():
    """Twenty drawn (M, N, K, output type, tile-scale flags) combinations."""
    rng = np.random.default_rng(4647)
    for i in range(20):
        flags = int(rng.integers(0, 4))
        M = int(rng.integers(1, 38)) * 16 if flags & 1 else int(rng.integers(1, 600))
        N = int(rng.integers(1, 38)) * 16 if flags & 2 else int(rng.integers(1, 600))
        K = int(rng.integers(1, 24)) * 32
        out_dtype = int(rng.integers(0, 2))
        ops, ref_ops = [], []
        for rows, tiled, name in ((M, flags & 1, "c3"), (N, flags & 2, "c2")):
            bits = wl.bf16_bits(wl.make(name, rows, K, seed=7000 + i))
            a = ref.tensor_scale(bits)
            if tiled:
                c, s, _, _ = ref.quantize_2d(bits, a)
            else:
                c, s, _ = ref.quantize(bits, a)
            ref_ops += [c, s, a]
            ops += [_dev(c), _dev(s), _alpha(a)]
        _log(f"gemm sweep {i}: M={M} N={N} K={K} out_dtype={out_dtype} flags={flags}")
        c_ref, c_abs = ref.gemm(*ref_ops, want_abs=True, tiles_a=bool(flags & 1),
                                tiles_b=bool(flags & 2))
        got = B.nvfp4_46_gemm(*ops, out_dtype=out_dtype, flags=flags)
        g = got.double().cpu().numpy() if out_dtype == B.OUT_F32 else _bf16_to_f64(got)
        assert (np.abs(g - c_ref) <= _tolerance(c_ref, c_abs, K, out_dtype)).all(), i


def test_gemm_operand_larger_than_four_gibibytes():
    """A [262,192][32,768]: 4.3 GB of codes, so byte offsets into A pass 2^32 (random codes and
    moderate scale bytes drawn on the GPU); rows from the start, from around the 2^32-byte
    mark and from the end are recomputed by the oracle."""
    M, N, K = 262192, 200, 32768
    g = torch.Generator(device="cuda")
    g.manual_seed(4651)
    u8 = dict(dtype=torch.uint8, device="cuda", generator=g)
    ca = torch.randint(0, 256, (M, K // 2), **u8)
    sa = torch.randint(0x28, 0x48, (M, K // 16), **u8)
    cb = torch.randint(0, 256, (N, K // 2), **u8)
    sb = torch.randint(0x28, 0x48, (N, K // 16), **u8)
    al = _alpha(0.5)
    got = B.nvfp4_46_gemm(ca, sa, al, cb, sb, al, out_dtype=B.OUT_F32)
    torch.cuda.synchronize()
    mark = 2 ** 32 // (K // 2)                                 # first row past 2^32 bytes
    rows = np.array([0, 1, 255, 256, mark - 1, mark, mark + 1, M - 129, M - 2, M - 1])
    idx = torch.from_numpy(rows).cuda()
    c_ref, c_abs = ref.gemm(ca[idx].cpu().numpy(), sa[idx].cpu().numpy(), 0.5, cb.cpu().numpy(),
                            sb.cpu().numpy(), 0.5, want_abs=True)
    gsel = got[idx].double().cpu().numpy()
    assert (np.abs(gsel - c_ref) <= _tolerance(c_ref, c_abs, K, B.OUT_F32)).all()


@pytest.mark.parametrize("tail", [32, 128])
@pytest.mark.parametrize("M,N", [(3, 5), (257, 258)])
def test_gemm_with_a_contraction_axis_past_the_32_bit_offsets(M, N, tail):
    """K = 2^24 + 32 (a last chunk of one unit) and 2^24 + 128 (a whole one): the kernel that stages chunks
    through registers, which no smaller K takes.  The codes are 0 but for 4096 indices, the last 64 and
    some around every power of two among them; scales 1 and multiples of 0.25 below 2^22: exact in any
    order."""
    K = (1 << 24) + tail
    assert hm.choose_gemm(M, N, K) == "staged"
    _log(f"gemm staged case M={M} N={N} K={K}")
    rng = np.random.default_rng(4653 + tail)
    special = [k + d for k in 2 ** np.arange(1, 25) for d in (-1, 0, 1) if k + d < K]
    at = np.unique(np.concatenate([rng.integers(0, K, 4096 - 160), special, np.arange(K - 64, K)]))
    codes, ops = {}, []
    for name, rows in (("a", M), ("b", N)):
        codes[name] = rng.integers(0, 16, (rows, len(at)), dtype=np.uint8)
        c = torch.zeros((rows, K // 2), dtype=torch.uint8, device="cuda")
        for parity in (0, 1):                    # even index: low nibble
            pick = at % 2 == parity
            c[:, torch.from_numpy(at[pick] // 2).cuda()] += _dev(codes[name][:, pick] << (4 * parity))
        ops += [c, torch.full((rows, K // 16), 0x38, dtype=torch.uint8, device="cuda"), _alpha(1.0)]
    grid = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6])
    da, db = grid[codes["a"]], grid[codes["b"]]
    assert (np.abs(da) @ np.abs(db).T).max() < 2.0 ** 22
    for out_dtype in (B.OUT_F32, B.OUT_BF16):
        got = B.nvfp4_46_gemm(*ops, out_dtype=out_dtype)
        want = torch.from_numpy((da @ db.T).astype(np.float32))
        assert torch.equal(got.cpu(), want if out_dtype == B.OUT_F32 else want.to(torch.bfloat16))


def test_gemm_with_more_columns_than_a_launch_of_small_tiles_holds():
    """One row of A against 2^28 + 96 rows of B, K = 32: in 32 x 32 tiles the launch would need 2^32 lanes.
    Every scale is 1, so each element is a sum of 32 multiples of 0.25, exact in any order."""
    N, K = (1 << 28) + 96, 32
    g = torch.Generator(device="cuda")
    g.manual_seed(4652)
    ca = torch.randint(0, 256, (1, K // 2), dtype=torch.uint8, device="cuda", generator=g)
    cb = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=g)
    sa = torch.full((1, K // 16), 0x38, dtype=torch.uint8, device="cuda")
    sb = torch.full((N, K // 16), 0x38, dtype=torch.uint8, device="cuda")
    _log(f"gemm case M=1 N={N} K={K}")
    got = B.nvfp4_46_gemm(ca, sa, _alpha(1.0), cb, sb, _alpha(1.0), out_dtype=B.OUT_F32)
    torch.cuda.synchronize()
    cols = np.concatenate([np.arange(0, N, 99991), [255, 256, N - 257, N - 2, N - 1]])
    rows = cb[torch.from_numpy(cols).cuda()].cpu().numpy()
    want = ref.gemm(ca.cpu().numpy(), sa.cpu().numpy(), 1.0, rows, np.full((len(cols), K // 16), 0x38, np.uint8), 1.0)
    assert np.array_equal(got[0, torch.from_numpy(cols).cuda()].double().cpu().numpy(), want[0])


@pytest.mark.parametrize("block2d", [True, False])
def test_linear_layer_module(block2d):
    """paper_2512_02010_amd.linear strings the library calls together as Fig. 3 does; each
    product must approximate the unquantized one to within NVFP4's quantization noise, and
    FPROP must equal the same calls made by hand."""
    from paper_2512_02010_amd import linear
    T, K, N = 256, 512, 384
    x = wl.make("c3", T, K).cuda()
    w = wl.make("c2", N, K, dtype=torch.float32).cuda()
    dy = wl.make("c1", T, N).cuda()
    qw = linear.quantize_weight(w, block2d=block2d)
    y = linear.fprop(x, qw)
    dx = linear.dgrad(dy, qw, sr_seed=wl.C5_SR_SEED)
    dw = linear.wgrad(dy, x, sr_seed=wl.C5_SR_SEED, rht_seed=wl.C5_RHT_SEED)
    assert y.shape == (T, N) and y.dtype == torch.bfloat16
    assert dx.shape == (T, K) and dw.shape == (N, K) and dw.dtype == torch.float32

    def rel(got, want):
        return float(((got.double() - want) ** 2).mean().sqrt() / (want ** 2).mean().sqrt())

    xd, wd, gd = x.double(), w.double(), dy.double()
    errs = {"FPROP": rel(y, xd @ wd.T), "DGRAD": rel(dx, gd @ wd), "WGRAD": rel(dw, gd.T @ xd)}
    _log(f"  linear layer (block2d={block2d}): relative RMS errors {errs}")
    assert all(e < 0.2 for e in errs.values()), errs

    ax = B.nvfp4_46_tensor_scale(x)
    qx = B.nvfp4_46_quantize(x, ax)
    by_hand = B.nvfp4_46_gemm(qx["codes_row"], qx["scales_row"], ax, qw["codes_row"],
                              qw["scales_row"], qw["alpha"],
                              flags=B.GEMM_B_TILE_SCALES if block2d else 0)
    assert torch.equal(by_hand, y)

    # the same step with the one-launch tensor scales (one workspace for all five)
    ws = B.new_workspace()
    qw2 = linear.quantize_weight(w, block2d=block2d, workspace=ws)
    assert torch.equal(qw2["alpha"], qw["alpha"]) and torch.equal(qw2["codes_col"], qw["codes_col"])
    assert torch.equal(linear.fprop(x, qw2, workspace=ws), y)
    assert torch.equal(linear.dgrad(dy, qw2, sr_seed=wl.C5_SR_SEED, workspace=ws), dx)
    assert torch.equal(linear.wgrad(dy, x, sr_seed=wl.C5_SR_SEED, rht_seed=wl.C5_RHT_SEED,
                                    workspace=ws), dw)
    assert not bool(ws.any())            # left zeroed
