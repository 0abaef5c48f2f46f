"""CPU: which HIP calls the library's host code makes (no device is involved, see _hip_calls.py)."""
from . import _hip_calls


def test_limits_of_dynamic_lds_are_the_kernels_own():
    """A kernel's limit of dynamic LDS is one for all threads of the process: whatever the size of a call, it sets the
    same, or a thread that is about to launch with more would be refused."""
    calls = _hip_calls.run("""
sizes = [(M, N, K) for M, K in ((1, 32), (1, 512), (16, 512), (7, 4096), (16, 1792), (5, 5728), (1, 28672)) for N in (64, 4096, 4097, 8192)]
for M, N, K in sizes:
    assert L.nvfp4_46_few_rows(P, 256.0, P, P, P, M, N, K, 0, P, None) == 0
for M, N, K in ((16, 8192, 8192), (32, 8192, 8192), (64, 8192, 8192), (64, 4096, 4096), (128, 4096, 4096), (200, 4096, 4096),
                (300, 2000, 1056), (300, 2000, 1312), (128, 8192, 8192), (1000, 4096, 992), (1000, 4096, 4096), (1000, 4096, 4128),
                (2048, 4096, 4096), (2048, 4096, 4128), (8192, 8192, 8192), (8192, 8192, 8160), (2048, 4095, 992), (2048, 4095, 768)):
    for out in (0, 1):
        assert L.nvfp4_46_gemm(P, P, P, P, P, P, M, N, K, out, 0, P, None) == 0
result = calls()
""")
    limits, launches = {}, {}
    for kind, kernel, lds, _, _ in calls:
        if kind in ("set_attribute", "launch"):
            (limits if kind == "set_attribute" else launches).setdefault(kernel, set()).add(lds)
    assert limits.keys() == launches.keys() and len(limits) > 20
    assert any(len(sizes) > 5 for sizes in launches.values())          # k_few_rows' own need varies
    for kernel, sizes in launches.items():
        assert len(limits[kernel]) == 1 and max(sizes) <= min(limits[kernel]), (limits[kernel], sizes)


def test_refused_calls_make_no_hip_call():
    made = _hip_calls.run("""
bad = [params(0, 1024), params(16, 1000), params(16, 1024, layout=0), params(16, 1024, fp8_max=0.0), params(24, 1024, layout=2)]
for p in bad:
    assert L.nvfp4_46_tensor_scale(P, p, P, None) != 0
    assert L.nvfp4_46_scale_quantize(P, p, P, None, 0, P, P, None, None, None, None, None) != 0
assert L.nvfp4_46_tensor_scale(P + 2, params(16, 1024), P, None) != 0
assert L.nvfp4_46_tensor_scale(None, params(16, 1024), P, None) != 0
assert L.nvfp4_46_tensor_scale(P, params(16, 1024), None, None) != 0
assert L.nvfp4_46_wgrad_operands(P, P, 24, 64, 64, 0, 1, 2, P, P, P, P, P, P, None, 0, None) != 0
result = calls()
""")
    assert made == []


def test_the_default_stream_is_only_asked_for_words_that_are_used():
    """Calls that run the same kernels on every stream make the same HIP calls on every stream: no lookup of scratch
    words that nobody uses (a host-bound call pays for it)."""
    default, other = _hip_calls.run("""
def on(stream):
    assert L.nvfp4_46_tensor_scale(P, params(64, 1024), P, stream) == 0                       # one workgroup
    assert L.nvfp4_46_tensor_scale(P, params(16, 1024, x_dtype=B.X_F32), P, stream) == 0
    assert L.nvfp4_46_scale_quantize(P, params(256, 1024), P, None, 0, P, P, None, None, P, None, stream) == 0   # one launch
    assert L.nvfp4_46_tensor_scale_ws(P, params(4096, 4096), P, P, 4352, stream) == 0
    assert L.nvfp4_46_scale_quantize(P, params(4096, 4096, layout=2, rht=1), P, P, 4352, None, None, P, P, None, None, stream) == 0
    assert L.nvfp4_46_wgrad_operands(P, P, 16384, 6144, 256, 0, 1, 2, P, P, P, P, P, P, P, 4352, stream) == 0    # one after the other
    return [c[:4] for c in calls()]
on(None)                                      # (the first calls ask for the compute units)
result = on(None), on(1 << 12)
""")
    assert default == other and len(default) >= 6


def test_a_small_tensors_scale_is_one_bare_launch():
    """512 KiB on the default stream: one workgroup, and no question to the runtime besides."""
    small, larger = _hip_calls.run("""
assert L.nvfp4_46_tensor_scale(P, params(256, 1024), P, None) == 0
small = [(c[0], c[3]) for c in calls()]
assert L.nvfp4_46_tensor_scale(P, params(320, 1024), P, None) == 0
result = small, [(c[0], c[3]) for c in calls() if c[0] == "launch"]
""")
    assert small == [["launch", 1]] and len(larger) == 1 and larger[0][1] > 1


def test_words_of_the_default_stream_are_looked_up_once():
    kinds = _hip_calls.run("""
for _ in range(3):
    assert L.nvfp4_46_tensor_scale(P, params(4096, 4096), P, None) == 0
result = [c[0] for c in calls()]
""")
    assert kinds.count("symbol_address") == 1 and kinds.count("launch") == 3


def test_compute_units_are_asked_for_once_per_launch():
    """(an attribute of the device costs the host a tenth of a microsecond, small calls are bound by the host)"""
    calls = _hip_calls.run("""
q = lambda **kw: L.nvfp4_46_quantize(P, params(1024, 2048, **kw), P, *((P, P) if kw.get("layout", 1) & 1 else (None, None)),
                                     *((P, P) if kw.get("layout", 1) & 2 else (None, None)), None, None, None)
result = []
for call in (lambda: q(), lambda: q(rounding=1, rht=1), lambda: q(layout=2), lambda: q(layout=3), lambda: q(block2d=1),
             lambda: q(layout=3, block2d=1), lambda: L.nvfp4_46_fake_quant(P, params(1024, 2048, block2d=1), P, P, None),
             lambda: L.nvfp4_46_dequantize(P, P, P, 1024, 2048, 1, P, None),
             lambda: L.nvfp4_46_tensor_scale_ws(P, params(1024, 2048, layout=2, rht=1), P, P, 4352, None),
             lambda: L.nvfp4_46_wgrad_operands(P, P, 256, 512, 384, 0, 1, 2, P, P, P, P, P, P, P, 4352, None)):
    assert call() == 0
    result.append([c[0] for c in calls()])
""")
    for kinds in calls:
        assert kinds.count("device_attribute") <= 1 <= kinds.count("launch"), kinds


def test_compute_units_are_kept_for_a_device():
    """They do not change; before they were kept every call asked for them."""
    kinds = _hip_calls.run("""
for _ in range(5):
    assert L.nvfp4_46_tensor_scale(P, params(4096, 4096), P, None) == 0
    assert L.nvfp4_46_quantize(P, params(4096, 4096), P, P, P, None, None, None, None, None) == 0
    assert L.nvfp4_46_quantize(P, params(4096, 4096, layout=3, block2d=1), P, P, P, P, P, None, None, None) == 0
    assert L.nvfp4_46_dequantize(P, P, P, 4096, 4096, 1, P, None) == 0
result = [c[0] for c in calls()]
""")
    assert kinds.count("launch") == 20 and kinds.count("device_attribute") <= 4, kinds


def test_rounds_of_the_rowwise_transform():
    """With the transform an eighth of the rounds goes to one-round workgroups, which leaves fewer workgroups; not where one
    fp32 candidate is rounded to nearest, which waits for memory (6144 x 6144 3.7 % slower with an eighth)."""
    grids = _hip_calls.run("""
result = []
for kw in (dict(select=1), dict(select=2), dict(select=0), dict(select=1, x_dtype=B.X_BF16), dict(select=1, rounding=1)):
    kw = dict(dict(x_dtype=B.X_F32, rht=1), **kw)
    for rht in (0, 1):
        assert L.nvfp4_46_quantize(P, params(6144, 6144, **dict(kw, rht=rht)), P, P, P, None, None, None, None, None) == 0
    result.append([c[3] for c in calls() if c[0] == "launch"])
""")
    for plain, transformed in grids[:2]:
        assert transformed == plain
    for plain, transformed in grids[2:]:
        assert transformed < plain


def test_maximum_after_the_rowwise_transform():
    """BF16: one kernel where a workgroup has at most two rounds of 256 blocks (two workgroups per compute unit), another beyond."""
    kernels = _hip_calls.run("""
result = []
for rows, cols in ((16, 1024), (2048, 2048), (2064, 2048), (2560, 2048), (8192, 8192)):
    assert L.nvfp4_46_tensor_scale_ws(P, params(rows, cols, rht=1), P, P, 4352, None) == 0
    result.append([c[1] for c in calls() if c[0] == "launch"])
""")
    small, large = kernels[0], kernels[-1]
    assert small != large and kernels == [small, small, large, large, large]
