"""The kernels' per-block code compiled for the host (tests/host_model/), behind ctypes.

Test infrastructure.  ``csrc/block.hpp`` and ``csrc/codec.hpp`` -- the code every quantizing
kernel runs per block -- and ``csrc/gemm_shapes.hpp``, ``csrc/small_tensors.hpp`` and ``csrc/tile_shapes.hpp`` -- the
host side's choices of kernel -- are compiled with the host compiler, the gfx950 conversion
instructions replaced by plain definitions of what they compute, so that CPU tests can put
the GPU path's block logic next to the oracle on inputs of any range without a GPU.
"""
from __future__ import annotations

import ctypes as C
import os
import shutil
import subprocess
from pathlib import Path

import numpy as np

_HERE = Path(__file__).resolve().parent / "host_model"
_ROOT = _HERE.parent.parent
_CSRC = _ROOT / "paper_2512_02010_amd" / "csrc"
_SO = _HERE / "_build" / "libhost_model.so"
_SOURCES = [_HERE / "model.cpp", _HERE / "gfx950_on_host.hpp", _CSRC / "block.hpp", _CSRC / "codec.hpp",
            _CSRC / "gemm_shapes.hpp", _CSRC / "small_tensors.hpp", _CSRC / "tile_shapes.hpp"]

RTN, SR, SR_AFTER_RTN_SELECT = 0, 1, 2

# enum GemmKernel
GEMM_KERNELS = ("staged", "dma", "skinny", "tile32", "tile64x32", "tile64", "tile64long",
                "tile128", "tile256x128", "dma256x128", "dma128")


def _compiler() -> str:
    for cand in ("/opt/rocm/llvm/bin/clang++", shutil.which("amdclang++"), shutil.which("clang++")):
        if cand and Path(cand).exists():
            return cand
    raise RuntimeError("no clang++ found (the headers use clang vector extensions)")


def build(force: bool = False) -> Path:
    newest = max(p.stat().st_mtime for p in _SOURCES)
    if _SO.exists() and not force and _SO.stat().st_mtime >= newest:
        return _SO
    _SO.parent.mkdir(parents=True, exist_ok=True)
    tmp = _SO.with_suffix(f".tmp{os.getpid()}.so")
    # one rounding per operation, as in the device build; no fast-math, denormals kept
    subprocess.run([_compiler(), "-x", "c++", "-std=c++17", "-O1", "-fPIC", "-shared",
                    "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{_CSRC}", f"-I{_ROOT / 'include'}", str(_HERE / "model.cpp"), "-o", str(tmp)],
                   check=True)
    os.replace(tmp, _SO)
    return _SO


_lib = None


def lib() -> C.CDLL:
    global _lib
    if _lib is None:
        L = C.CDLL(str(build()))
        f32p, u32p, u8p = C.POINTER(C.c_float), C.POINTER(C.c_uint32), C.POINTER(C.c_uint8)
        L.hm_quantize_blocks.restype = None
        L.hm_quantize_blocks.argtypes = [f32p, f32p, C.c_int64, C.c_float, C.c_int, C.c_int, u32p,
                                         u8p, u8p]
        L.hm_second_passes.restype = C.c_int
        L.hm_second_passes.argtypes = []
        L.hm_tile_decision.restype = C.c_int
        L.hm_tile_decision.argtypes = [f32p, f32p, C.c_float, C.c_int, u8p, u8p, C.POINTER(C.c_int)]
        L.hm_e2m1_sr.restype = None
        L.hm_e2m1_sr.argtypes = [f32p, f32p, C.c_int64, u8p, u8p]
        L.hm_block_scale.restype = C.c_int
        L.hm_block_scale.argtypes = [C.c_float, C.c_float, C.c_int, C.c_int]
        L.hm_philox.restype = None
        L.hm_philox.argtypes = [u32p, C.c_uint32, C.c_uint32, u32p]
        L.hm_sr_words_in_wave.restype = None
        L.hm_sr_words_in_wave.argtypes = [C.c_uint64, C.c_uint64, C.c_int, u32p]
        L.hm_rht_sign_word_of_wave.restype = C.c_uint32
        L.hm_rht_sign_word_of_wave.argtypes = [C.c_uint64, C.c_uint64]
        L.hm_rht16.restype = None
        L.hm_rht16.argtypes = [f32p, C.c_uint32]
        L.hm_choose_gemm.restype = C.c_int
        L.hm_choose_gemm.argtypes = [C.c_int64, C.c_int64, C.c_int64, C.c_int]
        L.hm_gemm_lanes.restype = C.c_int64
        L.hm_gemm_lanes.argtypes = [C.c_int, C.c_int64, C.c_int64]
        L.hm_scale_in_one_workgroup.restype = C.c_int
        L.hm_scale_in_one_workgroup.argtypes = [C.c_int64, C.c_int]
        L.hm_scale_in_one_workgroup_lent.restype = C.c_int
        L.hm_scale_in_one_workgroup_lent.argtypes = [C.c_int64]
        L.hm_scale_and_codes_in_one_launch.restype = C.c_int
        L.hm_scale_and_codes_in_one_launch.argtypes = [C.c_int64, C.c_int]
        L.hm_scale_by_words.restype = C.c_int
        L.hm_scale_by_words.argtypes = [C.c_int64, C.c_int]
        L.hm_tile_map.restype = None
        L.hm_tile_map.argtypes = [C.c_int64, C.c_int64, C.POINTER(C.c_int64)]
        L.hm_tile_unit_rows.restype = C.c_int
        L.hm_tile_unit_rows.argtypes = [C.c_int64, C.c_int64, C.c_int, C.c_int64]
        L.hm_tile_shape.restype = None
        L.hm_tile_shape.argtypes = [C.c_int, C.POINTER(C.c_int32)]
        _lib = L
    return _lib


def _p(a, ctype):
    return None if a is None else a.ctypes.data_as(C.POINTER(ctype))


def quantize_blocks(v: np.ndarray, alpha: float, rounding: int = RTN, select: int = 0,
                    u: np.ndarray | None = None):
    """v: [n][16] float32 (u likewise, for stochastic rounding).  Returns (codes [n][8] uint8
    in the library's nibble order, scale bytes [n], choices [n])."""
    v = np.ascontiguousarray(v, dtype=np.float32)
    n = v.shape[0]
    assert v.shape == (n, 16)
    if u is not None:
        u = np.ascontiguousarray(u, dtype=np.float32)
        assert u.shape == v.shape
    codes = np.zeros((n, 2), np.uint32)
    scale = np.zeros(n, np.uint8)
    four = np.zeros(n, np.uint8)
    lib().hm_quantize_blocks(_p(v, C.c_float), _p(u, C.c_float), n, alpha, rounding, select,
                             _p(codes, C.c_uint32), _p(scale, C.c_uint8), _p(four, C.c_uint8))
    return codes.view(np.uint8).reshape(n, 8), scale, four


def second_passes() -> int:
    """Blocks so far that the estimate pass could not decide (redone with the defined errors)."""
    return lib().hm_second_passes()


def tile_decision(v: np.ndarray, alpha: float, rounding: int = RTN, u: np.ndarray | None = None):
    """v: [16][16] float32, one tile.  Returns (four, scale6, scale4, took_defined_path)."""
    v = np.ascontiguousarray(v, dtype=np.float32)
    assert v.shape == (16, 16)
    if u is not None:
        u = np.ascontiguousarray(u, dtype=np.float32)
    s6, s4, path = C.c_uint8(), C.c_uint8(), C.c_int()
    four = lib().hm_tile_decision(_p(v, C.c_float), _p(u, C.c_float), alpha, rounding, C.byref(s6),
                                  C.byref(s4), C.byref(path))
    return four, s6.value, s4.value, path.value


def e2m1_sr(y: np.ndarray, u: np.ndarray):
    """(codes by the software rule, codes by the conversion instruction | 0x80 where the
    kernels would redo the block in software)."""
    y = np.ascontiguousarray(y, dtype=np.float32)
    u = np.ascontiguousarray(u, dtype=np.float32)
    out = np.zeros(y.shape, np.uint8)
    fast = np.zeros(y.shape, np.uint8)
    lib().hm_e2m1_sr(_p(y, C.c_float), _p(u, C.c_float), y.size, _p(out, C.c_uint8), _p(fast, C.c_uint8))
    return out, fast


def block_scale(b: float, alpha: float, M: int) -> int:
    """The byte for one M as the always-6 / always-4 kernels compute it."""
    return lib().hm_block_scale(b, alpha, M, 0)


def block_scale_pair(b: float, alpha: float):
    """(S6, S4) as the 4/6 kernels compute them, in one go."""
    r = lib().hm_block_scale(b, alpha, 6, 1)
    return r & 0xFF, r >> 8


def philox(ctr, key):
    c = (C.c_uint32 * 4)(*ctr)
    o = (C.c_uint32 * 4)()
    lib().hm_philox(c, key[0], key[1], o)
    return tuple(int(x) for x in o)


def sr_words_in_wave(seed: int, q: int, groups: int):
    """The stochastic-rounding words of elements 4 q .. 4 (q + groups) - 1, by the wave's generator."""
    o = (C.c_uint32 * (4 * groups))()
    lib().hm_sr_words_in_wave(seed, q, groups, o)
    return [int(x) for x in o]


def rht_sign_word_of_wave(seed: int, B: int) -> int:
    return lib().hm_rht_sign_word_of_wave(seed, B)


def rht16(v, sign_word: int) -> np.ndarray:
    a = np.array(v, dtype=np.float32).copy()
    lib().hm_rht16(_p(a, C.c_float), sign_word)
    return a


def choose_gemm(M: int, N: int, K: int, f32: bool = False) -> str:
    """Name of the kernel that nvfp4_46_gemm runs for an M x N x K product (C in BF16, or fp32)."""
    return GEMM_KERNELS[lib().hm_choose_gemm(M, N, K, f32)]


def gemm_lanes(kernel: str, M: int, N: int) -> int:
    return lib().hm_gemm_lanes(GEMM_KERNELS.index(kernel), M, N)


def tile_shape(kernel: str):
    """(BM, BN, threads, LDS bytes) of a tile shape of k_gemm_tile."""
    v = (C.c_int32 * 4)()
    lib().hm_tile_shape(GEMM_KERNELS.index(kernel), v)
    return tuple(v)


def scale_in_one_workgroup(nbytes: int, has_scratch: bool) -> bool:
    return bool(lib().hm_scale_in_one_workgroup(nbytes, has_scratch))


def scale_in_one_workgroup_lent(nbytes: int) -> bool:
    """... on the default stream, without a workspace."""
    return bool(lib().hm_scale_in_one_workgroup_lent(nbytes))


def scale_and_codes_in_one_launch(nbytes: int, has_scratch: bool) -> bool:
    return bool(lib().hm_scale_and_codes_in_one_launch(nbytes, has_scratch))


def scale_by_words(words: int, xf32: bool) -> bool:
    return bool(lib().hm_scale_by_words(words, xf32))


def tile_map(rows: int, cols: int):
    """(super-tile width, height, workgroups) of the tiled kernels' launch."""
    v = (C.c_int64 * 3)()
    lib().hm_tile_map(rows, cols, v)
    return tuple(v)


def tile_unit_rows(rows: int, cols: int, xf32: bool, compute_units: int = 256) -> int:
    """Tile rows of the units in which a tensor gets both packings of its 16x16 tiles."""
    return lib().hm_tile_unit_rows(rows, cols, xf32, compute_units)
