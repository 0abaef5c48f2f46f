"""The native side of the binding (csrc/python.cpp): what it refuses (CPU), and that outputs which it allocates
itself hold what the same calls leave in outputs of a caller's allocator (GPU)."""
import ctypes as C
import importlib.machinery
import importlib.util
import shutil

import numpy as np
import pytest
import torch

from paper_2512_02010_amd import binding as B
from paper_2512_02010_amd import build
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


def test_module_builds_without_a_host_compiler(monkeypatch, tmp_path):
    """Whoever can compile the library can compile the module."""
    which = shutil.which
    monkeypatch.delenv("CXX", raising=False)
    monkeypatch.setattr(shutil, "which", lambda name, *a, **k: None if name in ("g++", "c++") else which(name, *a, **k))
    so = build.build_python(tmp_path / "nvfp4_46_python.so")
    loader = importlib.machinery.ExtensionFileLoader("nvfp4_46_python", str(so))
    module = importlib.util.module_from_spec(importlib.util.spec_from_loader("nvfp4_46_python", loader))
    loader.exec_module(module)
    assert all(callable(getattr(module, name)) for name in B.NATIVE_ENTRY_POINTS)


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


class _Like:
    """Not a tensor, but with a tensor's attributes (on a pretended device, if it is on none)."""
    is_cuda = True

    def __init__(self, t):
        self.t = t

    def __getattr__(self, name):
        return getattr(self.t, name)


class _Mind(torch.Tensor):
    """A subclass that answers for itself where its memory is."""
    is_cuda = True

    def data_ptr(self):
        return super().data_ptr() + 64


@pytest.fixture
def calls_seen():
    """The module connected to entry points that only note their name, arguments and what `watch` says at that time."""
    module, seen, kept = B.native(), [], []
    watch = {"now": lambda: None}

    def noting(name, argtypes):
        def note(*a):
            seen.append((name, a, watch["now"]()))
            return 0
        kept.append(C.CFUNCTYPE(C.c_int, *argtypes)(note))
        return C.cast(kept[-1], C.c_void_p).value

    L = B.lib()
    real = [getattr(L, "nvfp4_46_" + name) for name in B.NATIVE_ENTRY_POINTS]
    types = [[C.c_void_p if t is C.POINTER(B.Params) else t for t in f.argtypes] for f in real]
    module.connect(B.Nvfp4Error, B._device_empty, *map(noting, B.NATIVE_ENTRY_POINTS, types))
    try:
        yield seen, watch
    finally:
        module.connect(B.Nvfp4Error, B._device_empty, *(C.cast(f, C.c_void_p).value for f in real))


@pytest.mark.parametrize("like", [_Like, lambda t: t.as_subclass(_Mind)])
def test_objects_with_a_tensors_attributes(like, calls_seen):
    seen, _ = calls_seen
    t = [torch.zeros(s, dtype=d) for s, d in (((32, 48), torch.bfloat16), ((1,), torch.float32), ((32, 24), torch.uint8),
                                              ((32, 3), torch.uint8), ((64,), torch.uint8), ((32, 48), torch.float32))]
    x, alpha, codes, scales, ws, out = (like(v) for v in t)
    px, pa, pc, ps, pw, po = (v.data_ptr() for v in (x, alpha, codes, scales, ws, out))
    assert (px == t[0].data_ptr()) == (like is _Like)
    full = dict(codes_row=codes, scales_row=scales, choice_row=None, codes_col=None, scales_col=None, choice_col=None)
    assert B.nvfp4_46_tensor_scale(x, out=alpha, stream=0) is alpha
    assert B.nvfp4_46_tensor_scale_ws(x, ws, out=alpha, stream=0) is alpha
    assert B.nvfp4_46_quantize(x, alpha, out=full, stream=0) is full
    assert B.nvfp4_46_dequantize(codes, scales, alpha, 32, 48, out=out, stream=0) is out
    assert B.nvfp4_46_fake_quant(x, alpha, out=out, stream=0) is out
    # (as operands 32 x 48 of a product of that contraction length: the scales' shape is right, the library is not asked)
    assert B.nvfp4_46_gemm(codes, scales, alpha, codes, scales, alpha, out=out, stream=0) is out
    assert [name for name, _, _ in seen] == ["tensor_scale", "tensor_scale_ws", "quantize", "dequantize", "fake_quant", "gemm"]
    a = [a for _, a, _ in seen]
    assert (a[0][0], a[0][2]) == (px, pa)
    assert (a[1][0], a[1][2], a[1][3], a[1][4]) == (px, pa, pw, 64)
    assert (a[2][0], a[2][2], a[2][3], a[2][4], a[2][5]) == (px, pa, pc, ps, None)
    assert a[3][:7] == (pc, ps, pa, 32, 48, 1, po)
    assert (a[4][0], a[4][2], a[4][3]) == (px, pa, po)
    assert a[5][:11] == (pc, ps, pa, pc, ps, pa, 32, 32, 48, 0, 0) and a[5][11] == po
    for call in (lambda: B.nvfp4_46_tensor_scale(like(t[0][0])), lambda: B.nvfp4_46_tensor_scale(like(t[2])),
                 lambda: B.nvfp4_46_quantize(like(t[0].t()), alpha, out=full),
                 lambda: B.nvfp4_46_gemm(codes, codes, alpha, codes, scales, alpha, out=out)):
        with pytest.raises(AssertionError):
            call()
    with pytest.raises(AttributeError):
        B.nvfp4_46_tensor_scale_ws(x, 16, out=alpha)


def test_outputs_that_a_mapping_makes_live_until_the_launch(calls_seen):
    """A mapping may make what it returns; nothing else holds it while the call runs without the lock."""
    seen, watch = calls_seen
    gone = []

    class Made(_Like):
        def __del__(self):
            gone.append(self)

    class Mapping:
        def __init__(self):
            self.alpha = None

        def __getitem__(self, name):
            return Made(torch.zeros((16, 8), dtype=torch.uint8))

        def __setitem__(self, name, value):
            self.alpha = value

    watch["now"] = lambda: len(gone)
    x, alpha = _Like(torch.zeros((16, 16), dtype=torch.bfloat16)), _Like(torch.zeros(1))
    B.nvfp4_46_quantize(x, alpha, out=Mapping(), stream=0)
    B.native().scale_quantize(x, None, alpha, Mapping(), True, 0, 1, 0, 0, 0, 0, 0, 256.0, 0)
    assert [now for _, _, now in seen] == [0, 6] and len(gone) == 12
    assert len(set(a for a in seen[0][1][3:9])) == 6       # (six outputs, none in another's memory)


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
    # (outputs like an object that is only like a tensor)
    yield lambda: B.nvfp4_46_tensor_scale(_Like(x))
    yield lambda: B.nvfp4_46_quantize(_Like(x), _Like(alpha), layout=B.BOTH)
    yield lambda: B.nvfp4_46_fake_quant(_Like(x), _Like(alpha))
    yield lambda: B.nvfp4_46_gemm(*(_Like(v) for v in (q["codes_row"], q["scales_row"], alpha) * 2))


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
@pytest.mark.parametrize("given", [False, True])
def test_launches_on_the_stream_that_is_meant(monkeypatch, given):
    """Each call is made while the stream it belongs to is still busy with what comes before its inputs (some
    milliseconds of products, then a copy into x): launched on any other stream it would read the inputs of before.
    `given`: the stream is named in the call instead of being the current one."""
    monkeypatch.setattr(B, "OUTPUT_ALLOCATOR", B._device_empty)
    g = torch.Generator(device="cuda")
    g.manual_seed(4671)
    new = torch.randn((64, 160), generator=g, device="cuda").bfloat16()
    alpha = B.nvfp4_46_tensor_scale(new)
    q = B.nvfp4_46_quantize(new, alpha)
    busy = torch.randn((4096, 4096), generator=g, device="cuda")
    ws, side = B.new_workspace(), torch.cuda.Stream()
    x, a, codes, scales = (torch.zeros_like(t) for t in (new, alpha, q["codes_row"], q["scales_row"]))
    for i, call in enumerate((lambda **s: B.nvfp4_46_tensor_scale(x, **s),
                              lambda **s: B.nvfp4_46_tensor_scale_ws(x, ws, **s),
                              lambda **s: B.nvfp4_46_quantize(x, a, **s)["codes_row"],
                              lambda **s: B.nvfp4_46_scale_quantize(x, ws, **s)["codes_row"],
                              lambda **s: B.nvfp4_46_fake_quant(x, a, **s),
                              lambda **s: B.nvfp4_46_dequantize(codes, scales, a, 64, 160, **s),
                              lambda **s: B.nvfp4_46_gemm(codes, scales, a, codes, scales, a, **s))):
        print(f"stream case {i}", flush=True)
        for t, n in ((x, new), (a, alpha), (codes, q["codes_row"]), (scales, q["scales_row"])):
            t.copy_(n)
        want = call().clone()
        for t in (x, a, codes, scales):
            t.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(4):
                busy @ busy
            for t, n in ((x, new), (a, alpha), (codes, q["codes_row"]), (scales, q["scales_row"])):
                t.copy_(n)
            if not given:
                got = call()
        if given:
            got = call(stream=side)
        busy_then = not side.query()
        torch.cuda.synchronize()
        assert busy_then and torch.equal(got.view(torch.uint8), want.view(torch.uint8)), i


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
