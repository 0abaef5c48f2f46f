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
