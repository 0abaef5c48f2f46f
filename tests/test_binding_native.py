"""The native side of the binding (csrc/python.cpp): what it refuses (CPU), and that outputs which it allocates
itself hold what the same calls leave in outputs of a caller's allocator (GPU)."""
import numpy as np
import pytest
import torch

from paper_2512_02010_amd import binding as B
from paper_2512_02010_amd import linear as L


def test_refusals_without_a_device():
    x = torch.zeros((16, 16), dtype=torch.bfloat16)
    for call, error in (
            (lambda: B.nvfp4_46_tensor_scale(x), AssertionError),                       # not on a device
            (lambda: B.nvfp4_46_tensor_scale(x.double()), AssertionError),
            (lambda: B.nvfp4_46_tensor_scale(x[0]), AssertionError),
            (lambda: B.nvfp4_46_tensor_scale(None), AttributeError),
            (lambda: B.nvfp4_46_tensor_scale_ws(x, None, out=16), AttributeError),
            (lambda: B.nvfp4_46_tensor_scale(x, rht="1"), TypeError),
            (lambda: B.nvfp4_46_gemm(x, x, x, x, x, x), AssertionError),                 # scales of another shape
            (lambda: B.nvfp4_46_quantize(x, 16, out={}), KeyError)):
        with pytest.raises(error):
            call()
    with pytest.raises(B.Nvfp4Error) as e:
        B.nvfp4_46_dequantize(16, 16, 16, 16, 17, out=16, stream=0)
    assert e.value.status == 2 and "nvfp4_46_dequantize: NVFP4_ERR_SHAPE" in str(e.value)


class _Index:
    def __init__(self, value):
        self.value = value

    def __index__(self):
        return self.value


@pytest.mark.parametrize("as_int", [np.int64, np.uint8, torch.tensor, _Index])
def test_integers_of_other_types(as_int):
    """Every integer argument may be anything with __index__, as NumPy's integers (a drawn seed) are; the calls end
    at what is wrong with them afterwards: tensors that are on no device, a shape."""
    x, one = torch.zeros((16, 16), dtype=torch.bfloat16), as_int(1)
    for call in (lambda: B.nvfp4_46_tensor_scale(x, layout=one, rht=one, rht_seed=one, fp8_max=256, out=16),
                 lambda: B.nvfp4_46_tensor_scale_ws(x, x, layout=one, rht=one, rht_seed=one, out=16),
                 lambda: B.nvfp4_46_quantize(x, 16, layout=one, rounding=one, select=one, rht=one, sr_seed=one,
                                             rht_seed=one, block2d=one),
                 lambda: B.nvfp4_46_scale_quantize(x, None, layout=one, rounding=one, select=one, rht=one,
                                                   sr_seed=one, rht_seed=one, block2d=one),
                 lambda: B.nvfp4_46_fake_quant(x, 16, layout=one, rounding=one, select=one, rht=one, sr_seed=one,
                                               rht_seed=one, block2d=one, out=16)):
        with pytest.raises(AssertionError, match="device tensors"):
            call()
    with pytest.raises(B.Nvfp4Error) as e:
        B.nvfp4_46_dequantize(16, 16, 16, one, one, layout=one, out=16, stream=0)
    assert e.value.status == 2


def _calls():
    g = torch.Generator(device="cuda")
    g.manual_seed(4670)
    x = torch.randn((64, 160), generator=g, device="cuda").bfloat16()
    w = torch.randn((96, 160), generator=g, device="cuda")
    ws = B.new_workspace()
    alpha = B.nvfp4_46_tensor_scale(x)
    yield lambda: B.nvfp4_46_tensor_scale(x, layout=B.COLWISE, rht=1, rht_seed=-3, fp8_max=448)
    yield lambda: B.nvfp4_46_tensor_scale_ws(w, ws)
    for layout in (B.ROWWISE, B.COLWISE, B.BOTH):
        for choice in (False, True):
            yield lambda: B.nvfp4_46_quantize(x, alpha, layout=layout, want_choice=choice, rounding=B.SR,
                                              sr_seed=np.uint64((1 << 64) - 5))
    yield lambda: B.nvfp4_46_quantize(w, alpha, layout=B.BOTH, block2d=1)
    yield lambda: B.nvfp4_46_scale_quantize(w, ws, layout=B.BOTH, block2d=1, want_choice=False)
    yield lambda: B.nvfp4_46_scale_quantize(x)
    yield lambda: B.nvfp4_46_fake_quant(w, alpha, layout=B.COLWISE, select=B.SEL_46_MAE)
    q = B.nvfp4_46_quantize(x, alpha)
    yield lambda: B.nvfp4_46_dequantize(q["codes_row"], q["scales_row"], alpha, 64, 160)
    for out in (B.OUT_BF16, B.OUT_F32):
        yield lambda: B.nvfp4_46_gemm(q["codes_row"], q["scales_row"], alpha, q["codes_row"], q["scales_row"],
                                      alpha, out_dtype=out)
    yield lambda: L.fprop(x, L.quantize_weight(w, workspace=ws), workspace=ws)


@pytest.mark.gpu
def test_outputs_allocated_natively(monkeypatch):
    def run(call):
        r = call()
        return list(r.items()) if isinstance(r, dict) else [("", r)]

    for i, call in enumerate(_calls()):
        print(f"native allocation case {i}", flush=True)
        want = run(call)
        with monkeypatch.context() as m:
            m.setattr(B, "OUTPUT_ALLOCATOR", B._device_empty)
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            got = [run(call)]
            with torch.cuda.stream(side):
                got.append(run(call))
            torch.cuda.synchronize()
        for g in got:
            assert [k for k, _ in g] == [k for k, _ in want]
            for (name, a), (_, b) in zip(g, want):
                if b is None:
                    assert a is None, name
                else:
                    assert a.shape == b.shape and a.dtype == b.dtype and a.device == b.device, name
                    assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name


@pytest.mark.gpu
def test_given_outputs_and_statuses(monkeypatch):
    monkeypatch.setattr(B, "OUTPUT_ALLOCATOR", B._device_empty)
    x = torch.ones((32, 32), dtype=torch.bfloat16, device="cuda")
    alpha = torch.empty(1, dtype=torch.float32, device="cuda")
    assert B.nvfp4_46_tensor_scale(x, out=alpha) is alpha
    out = B.alloc_outputs(32, 32, B.ROWWISE, x.device)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    assert B.nvfp4_46_quantize(x, alpha, out=out, stream=s) is out
    s.synchronize()
    assert torch.equal(out["codes_row"], B.nvfp4_46_quantize(x, alpha, stream=0)["codes_row"])
    for call, status in ((lambda: B.nvfp4_46_quantize(x, alpha, layout=4), 4),
                         (lambda: B.nvfp4_46_quantize(x[:, :24].contiguous(), alpha), 2),
                         (lambda: B.nvfp4_46_quantize(x, None), 1),
                         (lambda: B.nvfp4_46_tensor_scale_ws(x, torch.zeros(16, dtype=torch.uint8, device="cuda")), 4),
                         (lambda: B.nvfp4_46_fake_quant(x, alpha, layout=B.BOTH), 4)):
        with pytest.raises(B.Nvfp4Error) as e:
            call()
        assert e.value.status == status
    with pytest.raises(AssertionError):
        B.nvfp4_46_quantize(x.t()[::2], alpha)
