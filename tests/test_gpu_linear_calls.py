"""GPU: the products of a linear layer in one call each against the library calls that they stand for, bit for bit."""
import pytest
import torch

from paper_2512_02010_amd import binding as B
from paper_2512_02010_amd import linear as L
from paper_2512_02010_amd import workloads as wl

pytestmark = pytest.mark.gpu

SR_SEED, RHT_SEED = wl.C5_SR_SEED, wl.C5_RHT_SEED


def _columnwise(t, **kw):
    q = B.nvfp4_46_scale_quantize(t, layout=B.COLWISE, rht=1, rht_seed=RHT_SEED, **kw)
    return q["codes_col"], q["scales_col"], q["alpha"]


def _wgrad(dy, x, select=B.SEL_46_MSE):
    return B.nvfp4_46_gemm(*_columnwise(dy, rounding=B.SR, sr_seed=SR_SEED, select=select), *_columnwise(x, select=select),
                           out_dtype=B.OUT_F32)


# tokens x features of dy and of x: one tile, fewer tiles than dies, neither a multiple of the other, tall, wide, either
# side of four bytes per lane for the maxima, and more than goes in pairs (192 MiB)
@pytest.mark.parametrize("T,N,K", [(32, 8, 16), (64, 128, 128), (96, 1000, 24), (736, 264, 1032), (4096, 64, 48), (64, 4096, 256),
                                   (1024, 2048, 2048), (1024, 2048, 2056), (2048, 4096, 4096), (16384, 6144, 256)])
@pytest.mark.parametrize("with_workspace", [True, False])
def test_weight_gradient_matches_the_calls_one_by_one(T, N, K, with_workspace):
    torch.manual_seed(T)
    dy = (torch.randn(T, N, device="cuda") * torch.randn(T, 1, device="cuda").mul(2.0).exp() * 1e-3).bfloat16()
    x = torch.randn(T, K, device="cuda").bfloat16()
    ws = B.new_workspace() if with_workspace else None
    want = _wgrad(dy, x)
    for _ in range(2):                                   # the words are left zero
        assert torch.equal(L.wgrad(dy, x, SR_SEED, RHT_SEED, workspace=ws), want)
    if ws is not None:
        assert not ws.any()


@pytest.mark.parametrize("select", [B.SEL_FORCE6, B.SEL_FORCE4, B.SEL_46_MAE, B.SEL_46_ABSMAX])
def test_weight_gradient_with_every_rule(select):
    dy, x = wl.make("c5", 160, 272).cuda(), wl.make("c3", 160, 144).cuda()
    assert torch.equal(L.wgrad(dy, x, SR_SEED, RHT_SEED, select=select), _wgrad(dy, x, select))


def test_weight_gradient_on_another_stream_in_a_graph_and_of_other_types():
    dy, x = wl.make("c5", 256, 512).cuda(), wl.make("c3", 256, 384).cuda()
    want = _wgrad(dy, x)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    for kw in (dict(), dict(workspace=B.new_workspace()), dict(stream=s)):
        with torch.cuda.stream(s):
            got = L.wgrad(dy, x, SR_SEED, RHT_SEED, **kw)
        s.synchronize()
        assert torch.equal(got, want)
    ws, graph = B.new_workspace(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = L.wgrad(dy, x, SR_SEED, RHT_SEED, workspace=ws)
    for seed in (1, 2, 3):
        dy.copy_(wl.make("c5", 256, 512).cuda() * seed)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, _wgrad(dy, x))
    assert torch.equal(L.wgrad(dy.float(), x, SR_SEED, RHT_SEED), _wgrad(dy.float(), x))
    with pytest.raises(AssertionError):
        L.wgrad(dy, x[:128], SR_SEED, RHT_SEED)


@pytest.mark.parametrize("block2d", [True, False])
def test_input_gradient_matches_the_calls_one_by_one(block2d):
    qw = L.quantize_weight(wl.make("c2", 288, 160, dtype=torch.float32).cuda(), block2d=block2d)
    dy = wl.make("c5", 48, 288).cuda()
    q = B.nvfp4_46_scale_quantize(dy, rounding=B.SR, sr_seed=SR_SEED)
    want = B.nvfp4_46_gemm(q["codes_row"], q["scales_row"], q["alpha"], qw["codes_col"], qw["scales_col"], qw["alpha"],
                           flags=B.GEMM_B_TILE_SCALES if block2d else 0)
    assert torch.equal(L.dgrad(dy, qw, SR_SEED), want)
    assert torch.equal(L.dgrad(dy, qw, SR_SEED, workspace=B.new_workspace()), want)
