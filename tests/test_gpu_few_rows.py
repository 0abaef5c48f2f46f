"""GPU: scale, codes and product of a few rows in one launch, against the oracle and against the calls one by one."""
import threading

import numpy as np
import pytest
import torch

from oracle import ref
from paper_2512_02010_amd import binding as B
from paper_2512_02010_amd import linear as L
from paper_2512_02010_amd import workloads as wl
from tests.test_gpu_gemm import _bf16_to_f64, _dev, _alpha, _tolerance

pytestmark = pytest.mark.gpu


def _weight(N, K, tiles):
    bits = wl.bf16_bits(wl.make("c2", N, K))
    alpha = ref.tensor_scale(bits)
    codes, scales = (ref.quantize_2d if tiles else ref.quantize)(bits, alpha)[:2]
    return codes, scales, alpha


# rows: one, an odd number, a whole instruction tile; K: below one chunk of 256, ragged, whole chunks, more chunks
# than the eight waves hold at once (a second turn of the ring, waves without a chunk), the most values there may be;
# N: less than a workgroup's columns, ragged, and either side of the wider workgroups (256 of 16 columns)
@pytest.mark.parametrize("M,K", [(1, 32), (1, 256), (3, 160), (16, 96), (5, 2048), (14, 2048), (1, 4384), (6, 4640), (1, 16384),
                                 (1, 28672)])
@pytest.mark.parametrize("N,tiles", [(1, False), (17, False), (48, True), (160, True)])
def test_few_rows_match_the_oracle(M, K, N, tiles):
    cb, sb, ab = _weight(N, K, tiles)
    bits = wl.bf16_bits(wl.make("c3", M, K))
    aa = ref.tensor_scale(bits)
    ca, sa, _ = ref.quantize(bits, aa)
    sb_rows = sb.repeat(16, axis=0) if tiles else sb
    want, total = ref.gemm(ca, sa, aa, cb, sb_rows, ab, want_abs=True)
    x = wl.make("c3", M, K).cuda()
    flags = B.GEMM_B_TILE_SCALES if tiles else 0
    got = B.product_of_rows(x, _dev(cb), _dev(sb), _alpha(ab), flags)
    assert got is not None and got.shape == (M, N) and got.dtype == torch.bfloat16
    err = abs(_bf16_to_f64(got) - want)
    assert (err <= _tolerance(want, total, K, B.OUT_BF16)).all(), err.max()


# the wider workgroups (more than 256 of 16 columns) along a longer K: a second stage of the ring (more than eight chunks of 256), its
# refill (more than sixteen), whole and ragged chunks, a workgroup cut by the edge
@pytest.mark.parametrize("M,K,N,tiles", [(1, 2080, 4097, False), (3, 2048, 8192, True), (3, 4640, 8192, False), (5, 4096, 4112, True),
                                         (3, 8192, 8192, True), (1, 8224, 4128, False), (1, 16384, 4097, False),
                                         (1, 28672, 4112, True)])
def test_few_rows_against_wide_weights(M, K, N, tiles):
    rng = np.random.default_rng(M * 7919 + N * 31 + K)
    cb = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    sb = rng.integers(0x20, 0x48, (N // 16 if tiles else N, K // 16), dtype=np.uint8)
    ab = np.float32(0.01)
    bits = wl.bf16_bits(wl.make("c3", M, K))
    aa = ref.tensor_scale(bits)
    ca, sa, _ = ref.quantize(bits, aa)
    want, total = ref.gemm(ca, sa, aa, cb, sb.repeat(16, axis=0) if tiles else sb, ab, want_abs=True)
    print(f"few rows case M={M} K={K} N={N} tiles={tiles}", flush=True)
    got = B.product_of_rows(wl.make("c3", M, K).cuda(), _dev(cb), _dev(sb), _alpha(ab), B.GEMM_B_TILE_SCALES if tiles else 0)
    assert got is not None and got.shape == (M, N)
    err = abs(_bf16_to_f64(got) - want)
    assert (err <= _tolerance(want, total, K, B.OUT_BF16)).all(), err.max()


def test_two_threads_with_different_sizes():
    """One kernel, two sizes of LDS, two threads on streams of their own."""
    qw = [L.quantize_weight(wl.make("c2", 5120, cols).cuda()) for cols in (256, 1792)]
    xs = [wl.make("c1", rows, cols).cuda() for rows, cols in ((1, 256), (16, 1792))]
    want = [L.fprop(x, w) for x, w in zip(xs, qw)]
    torch.cuda.synchronize()
    got = [[], []]

    def calls(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(100):
                got[i].append(L.fprop(xs[i], qw[i]))
        s.synchronize()

    threads = [threading.Thread(target=calls, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(got[i]) == 100 and all(torch.equal(y, want[i]) for y in got[i]), i


@pytest.mark.parametrize("N", [4096, 4097, 8192])
def test_wide_weights_match_the_calls_one_by_one(N):
    """Whole chunks: the same sums in the same order but for the number of waves, one rounding to BF16 apart."""
    w = wl.make("c2", N, 512).cuda()
    qw = L.quantize_weight(w) if N % 16 == 0 else dict(B.nvfp4_46_scale_quantize(w), block2d=False)
    x = wl.make("c3", 16, 512).cuda()
    q = B.nvfp4_46_scale_quantize(x)
    flags = B.GEMM_B_TILE_SCALES if qw["block2d"] else 0
    exact = B.nvfp4_46_gemm(q["codes_row"], q["scales_row"], q["alpha"], qw["codes_row"], qw["scales_row"], qw["alpha"],
                            out_dtype=B.OUT_F32, flags=flags)
    y = L.fprop(x, qw)
    assert ((y.float() - exact).abs() <= exact.abs() * 2.0 ** -8 + exact.abs().max() * 2.0 ** -18).all()


def _one_by_one(x, qw, **kw):
    """The forward pass by the two calls that it was made of."""
    q = B.nvfp4_46_scale_quantize(x, **kw)
    flags = B.GEMM_B_TILE_SCALES if qw["block2d"] else 0
    return B.nvfp4_46_gemm(q["codes_row"], q["scales_row"], q["alpha"], qw["codes_row"], qw["scales_row"], qw["alpha"],
                           flags=flags)


# either side of what takes one launch: rows, values, columns; BF16 and fp32, another selection rule
@pytest.mark.parametrize("rows,cols,out", [(16, 256, 64), (17, 256, 64), (7, 4096, 64), (8, 4096, 64), (2, 256, 8192),
                                           (2, 256, 8208)])
def test_either_side_of_one_launch(rows, cols, out):
    qw = L.quantize_weight(wl.make("c2", out, cols).cuda())
    x = wl.make("c3", rows, cols).cuda()
    assert torch.equal(L.fprop(x, qw), _one_by_one(x, qw))
    assert torch.equal(L.fprop(x.float(), qw), _one_by_one(x.float(), qw))
    assert torch.equal(L.fprop(x, qw, select=B.SEL_46_MAE), _one_by_one(x, qw, select=B.SEL_46_MAE))
    assert not L.fprop(torch.zeros_like(x), qw).any()


def test_what_is_left_to_the_calls_one_by_one():
    qw = L.quantize_weight(wl.make("c2", 64, 256).cuda())
    args = qw["codes_row"], qw["scales_row"], qw["alpha"], B.GEMM_B_TILE_SCALES
    x = wl.make("c1", 16, 256).cuda()
    assert B.product_of_rows(x, *args) is not None
    small = torch.zeros(16, dtype=torch.uint8, device="cuda")
    for other in (wl.make("c1", 16, 512).cuda()[:, ::2],                # not contiguous
                  wl.make("c1", 16, 512).cuda(),                        # another K
                  x.half(), x.reshape(-1), x.cpu()):
        assert B.product_of_rows(other, *args) is None
    assert B.product_of_rows(x, *args, workspace=small) is None
    assert B.product_of_rows(x, *args[:3], 0) is None                   # scales of another shape than these flags say
    with pytest.raises(B.Nvfp4Error):
        L.fprop(wl.make("c1", 64, 256).cuda(), qw, workspace=small)
    with pytest.raises(AssertionError):
        L.fprop(x.half(), qw)


def test_few_rows_on_a_side_stream_and_in_a_graph():
    qw = L.quantize_weight(wl.make("c2", 96, 512).cuda())
    x = wl.make("c1", 8, 512).cuda()
    want = L.fprop(x, qw).clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        assert torch.equal(L.fprop(x, qw, stream=s), want)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = L.fprop(x, qw)
    for scale in (1.0, 2.0, -4.0):                                      # exact: a power of two scales x's own scale
        x.copy_(wl.make("c1", 8, 512).cuda() * scale)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, L.fprop(x, qw)) and torch.equal(y, want * scale)
