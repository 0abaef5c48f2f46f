"""CPU-side checks of the C-ABI library: it loads, exports what the header declares,
and its host-side argument validation returns the documented codes without touching
the GPU (every call below fails validation before any HIP call)."""
import ctypes as C
import re
import subprocess
from pathlib import Path

import pytest

from paper_2512_02010_amd import binding as B
from paper_2512_02010_amd import build

ROOT = Path(__file__).resolve().parent.parent
HEADER = (ROOT / "include" / "nvfp4_46.h").read_text()
FUSED_HEADER = (ROOT / "include" / "nvfp4_46_fused.h").read_text()


def _declared(header=HEADER + FUSED_HEADER):
    names = re.findall(r"^(?:int|const char \*)\s*(nvfp4_46_\w+)\s*\(", header, flags=re.M)
    return sorted(set(names))


def test_every_header_is_covered():
    assert sorted(p.name for p in (ROOT / "include").glob("*.h")) == ["nvfp4_46.h", "nvfp4_46_fused.h"]
    assert _declared(FUSED_HEADER) == ["nvfp4_46_scale_quantize"]


def test_library_exports_every_declared_symbol():
    L = B.lib()
    names = _declared()
    assert len(_declared(HEADER)) == 14 and len(names) == 15
    assert sorted(B.EXPORTS) == names
    for n in names:
        assert hasattr(L, n), n


def test_what_the_library_exports_besides_is_declared():
    """Two entry points for the package's own Python module (csrc/layer.hpp, which that module is built with); not more."""
    names = set(re.findall(r" T (nvfp4_46_\w+)$", subprocess.run(["nm", "-D", "--defined-only", str(B.library_path())], text=True,
                                                                capture_output=True, check=True).stdout, flags=re.M))
    layer = set(_declared((ROOT / "paper_2512_02010_amd" / "csrc" / "layer.hpp").read_text()))
    assert layer == {"nvfp4_46_" + name for name in B.LAYER_ENTRY_POINTS}
    assert names == layer | set(B.EXPORTS)


def test_the_default_stream_is_one_for_all_threads(tmp_path):
    """Scratch words are lent to calls on the default stream; the sources do not compile with one per thread."""
    source = tmp_path / "one.hip"
    source.write_text('#include "launch.hpp"\n')
    base = [build.hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-fsyntax-only",
            f"-I{build.ROOT / 'include'}", f"-I{build.PKG / 'csrc'}", str(source)]
    assert subprocess.run(base, capture_output=True).returncode == 0
    per_thread = subprocess.run([*base, "-fgpu-default-stream=per-thread"], capture_output=True, text=True)
    assert per_thread.returncode != 0 and "legacy default stream" in per_thread.stderr


def test_params_struct_layout_matches_header():
    assert C.sizeof(B.Params) == 64
    offs = {f[0]: getattr(B.Params, f[0]).offset for f in B.Params._fields_}
    assert offs == {"rows": 0, "cols": 8, "layout": 16, "rounding": 20, "select": 24, "rht": 28,
                    "sr_seed": 32, "rht_seed": 40, "fp8_max": 48, "block2d": 52,
                    "x_dtype": 56}
    # enum values quoted in the header
    for name, val in (("NVFP4_ROWWISE", 1), ("NVFP4_COLWISE", 2), ("NVFP4_RTN", 0), ("NVFP4_SR", 1), ("NVFP4_SR_AFTER_RTN_SELECT", 2),
                      ("NVFP4_SEL_46_MSE", 0), ("NVFP4_SEL_FORCE6", 1), ("NVFP4_SEL_FORCE4", 2),
                      ("NVFP4_SEL_46_MAE", 3), ("NVFP4_SEL_46_ABSMAX", 4), ("NVFP4_X_BF16", 0),
                      ("NVFP4_X_F32", 1)):
        assert re.search(rf"{name} = {val}\b", HEADER), name


def test_status_strings():
    for code in range(7):
        s = B.status_string(code)
        assert isinstance(s, str) and s
    assert B.status_string(0) == "ok" and "unknown" in B.status_string(99)


P = 0x10000      # a fake, 16-byte aligned, never dereferenced "device pointer"


def _q(params, x=P, alpha=P, cr=P, sr=P, cc=None, sc=None, hr=None, hc=None):
    return B.quantize_raw(x, params, alpha, cr, sr, cc, sc, hr, hc, stream=0)


def test_quantize_validation_codes():
    ok = B.make_params(32, 64)
    assert _q(None) == 1 and _q(ok, x=None) == 1 and _q(ok, alpha=None) == 1
    assert _q(ok, cr=None) == 1 and _q(ok, sr=None) == 1
    assert _q(B.make_params(0, 64)) == 2 and _q(B.make_params(32, -16)) == 2
    assert _q(B.make_params(32, 72)) == 2                       # cols % 16 != 0, rowwise
    assert _q(B.make_params(40, 64, layout=B.COLWISE), cr=None, sr=None, cc=P, sc=P) == 2
    assert _q(B.make_params(32, 36, layout=B.COLWISE), cr=None, sr=None, cc=P, sc=P) == 2
    assert _q(ok, x=P + 2) == 3 and _q(ok, cr=P + 8) == 3 and _q(ok, hr=P + 1) == 3
    assert _q(B.make_params(32, 64, layout=0)) == 4 and _q(B.make_params(32, 64, layout=4)) == 4
    assert _q(B.make_params(32, 64, rounding=3)) == 4 and _q(B.make_params(32, 64, select=5)) == 4
    assert _q(B.make_params(32, 64, rht=2)) == 4
    assert _q(B.make_params(32, 64, x_dtype=2)) == 4
    assert _q(B.make_params(32, 64, fp8_max=0.0)) == 4
    assert _q(B.make_params(32, 64, fp8_max=449.0)) == 4
    assert _q(B.make_params(32, 64, fp8_max=float("nan"))) == 4
    bad = B.make_params(32, 64)
    bad.block2d = 2
    assert _q(bad) == 4
    # 16x16 tiles: both dims multiples of 16, no transform
    assert _q(B.make_params(40, 64, block2d=1)) == 2
    assert _q(B.make_params(32, 64, block2d=1, rht=1)) == 5
    # 2D blocks packed for the transposed matrix only: row outputs are then not allowed
    assert _q(B.make_params(32, 64, layout=B.COLWISE, block2d=1), cr=P, sr=P, cc=P, sc=P) == 4
    # outputs for a layout that was not asked for
    assert _q(ok, cc=P, sc=P) == 4 and _q(ok, hc=P) == 4
    # columnwise requested but its outputs are missing
    assert _q(B.make_params(32, 64, layout=B.BOTH)) == 1
    # the transform with both orientations is refused
    assert _q(B.make_params(32, 64, layout=B.BOTH, rht=1), cc=P, sc=P) == 5
    # over-large shapes
    assert _q(B.make_params(1 << 32, 64)) == 2 and _q(B.make_params(1 << 30, 1 << 12)) == 2


def test_other_entry_points_validation_codes():
    ok = B.make_params(32, 64)
    assert B.tensor_scale_raw(P, ok, None, stream=0) == 1
    assert B.tensor_scale_raw(None, ok, P, stream=0) == 1
    assert B.tensor_scale_raw(P, B.make_params(32, 60), P, stream=0) == 2
    assert B.tensor_scale_raw(P + 4, ok, P, stream=0) == 3
    assert B.tensor_scale_raw(P, B.make_params(32, 64, layout=B.BOTH, rht=1), P, stream=0) == 5
    assert B.fake_quant_raw(P, ok, P, None, stream=0) == 1
    assert B.fake_quant_raw(P, B.make_params(32, 64, layout=B.BOTH), P, P, stream=0) == 4
    assert B.fake_quant_raw(P, ok, P, P + 6, stream=0) == 3
    assert B.dequantize_raw(None, P, P, 32, 64, B.ROWWISE, P, stream=0) == 1
    assert B.dequantize_raw(P, P, P, 32, 64, B.BOTH, P, stream=0) == 4
    assert B.dequantize_raw(P, P, P, 40, 64, B.BLOCK2D, P, stream=0) == 2
    assert B.dequantize_raw(P, P, P, 32, 40, B.ROWWISE, P, stream=0) == 2
    assert B.dequantize_raw(P, P, P, 24, 64, B.COLWISE, P, stream=0) == 2
    assert B.dequantize_raw(P, P + 3, P, 32, 64, B.ROWWISE, P, stream=0) == 3
    assert B.tensor_scale_ws_raw(P, ok, P, None, 4352, stream=0) == 1
    assert B.tensor_scale_ws_raw(P, ok, P, P, 4096, stream=0) == 4
    assert B.tensor_scale_ws_raw(P, ok, P, P + 4, 4352, stream=0) == 3
    assert B.tensor_scale_ws_raw(P, ok, None, P, 4352, stream=0) == 1
    L = B.lib()
    assert L.nvfp4_46_debug_e2m1_rtn_range(0, 16, None, None) == 1
    assert L.nvfp4_46_debug_e4m3_range(0, 0, C.c_void_p(P), None) == 2


def _sq(params, x=P, alpha=P, ws=P, ws_bytes=4352, cr=P, sr=P, cc=None, sc=None, hr=None, hc=None):
    return B.scale_quantize_raw(x, params, alpha, ws, ws_bytes, cr, sr, cc, sc, hr, hc, stream=0)


def test_joined_call_has_the_errors_of_its_two_calls():
    """nvfp4_46_scale_quantize refuses what nvfp4_46_tensor_scale(_ws) or nvfp4_46_quantize would; where
    several arguments are wrong, with the status of the call, and the check, that comes first."""
    ok = B.make_params(32, 64)
    both = B.make_params(32, 64, layout=B.BOTH)
    for ws, n in ((P, 4352), (None, 0)):
        w = dict(ws=ws, ws_bytes=n)
        assert _sq(None, **w) == 1 and _sq(ok, x=None, **w) == 1 and _sq(ok, alpha=None, **w) == 1
        assert _sq(B.make_params(0, 64), **w) == 2 and _sq(B.make_params(32, 72), **w) == 2
        assert _sq(B.make_params(1 << 30, 1 << 12), **w) == 2
        assert _sq(B.make_params(40, 64, block2d=1), **w) == 2
        assert _sq(ok, x=P + 2, **w) == 3
        assert _sq(B.make_params(32, 64, layout=0), **w) == 4 and _sq(B.make_params(32, 64, select=9), **w) == 4
        assert _sq(B.make_params(32, 64, fp8_max=0.0), **w) == 4
        assert _sq(B.make_params(32, 64, layout=B.BOTH, rht=1), cc=P, sc=P, **w) == 5
        assert _sq(B.make_params(32, 64, block2d=1, rht=1), **w) == 5
        # the quantizer's own checks
        assert _sq(ok, cr=None, **w) == 1 and _sq(ok, sr=None, **w) == 1 and _sq(both, **w) == 1
        assert _sq(ok, cr=P + 8, **w) == 3 and _sq(ok, hr=P + 1, **w) == 3
        assert _sq(ok, cc=P, sc=P, **w) == 4 and _sq(ok, hc=P, **w) == 4
        # ... come after those of the tensor scale
        assert _sq(B.make_params(32, 72), cr=None, **w) == 2 and _sq(ok, x=P + 2, cc=P, sc=P, **w) == 3
    # the workspace, and its checks first
    assert _sq(ok, ws_bytes=4096) == 4 and _sq(ok, ws=P + 4) == 3
    for more in (dict(x=None), dict(alpha=None), dict(cr=None), dict(x=P + 2)):
        assert _sq(ok, ws_bytes=4096, **more) == B.tensor_scale_ws_raw(P, ok, None, P, 4096, stream=0) == 4
        assert _sq(ok, ws=P + 4, **more) == B.tensor_scale_ws_raw(P, ok, None, P + 4, 4352, stream=0) == 3


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setenv("NVFP4_46_LIB", str(tmp_path / "nope.so"))
    monkeypatch.setattr(B, "_lib", None)
    with pytest.raises(FileNotFoundError):
        B.lib()


def test_every_hip_source_is_part_of_the_build():
    from pathlib import Path
    from paper_2512_02010_amd import build
    sources = {p.name for p in (Path(build.PKG) / "csrc").glob("*.hip")}
    assert sources == {Path(u[0]).name for u in build.UNITS}
    # each part number of a source compiled in parts appears exactly once
    for name in ("nvfp4_46.hip", "gemm.hip"):
        parts = sorted(list(u[1].values())[0] for u in build.UNITS if Path(u[0]).name == name)
        assert parts == list(range(7)), (name, parts)
