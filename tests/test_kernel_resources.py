"""CPU: register and scratch budgets of the kernels, read from the compiler's resource report.

hipcc cross-compiles for gfx950 without a GPU.  Two properties are pinned here because the
code silently depends on them:
  - the rowwise 4/6 kernel fits 64 vector registers (8 waves per SIMD) without spilling --
    the reason the rare undecided block is redone from memory instead of kept in registers;
  - the matrix-product kernels that wait for their asynchronous global -> LDS copies with
    hand-counted `s_waitcnt vmcnt(N)` use no scratch memory: a spill would add vector-memory
    instructions of the compiler's own and make those counts too small.
"""
import functools
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2512_02010_amd import build

from . import _host_model as hm


@functools.lru_cache(maxsize=None)
def _report(source: str, part_macro: str, part: int):
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    r = subprocess.run([build.hipcc(), *flags, f"-I{build.ROOT / 'include'}", f"-I{build.PKG / 'csrc'}",
                        f"-D{part_macro}={part}", "-Rpass-analysis=kernel-resource-usage", "-c",
                        str(build.PKG / "csrc" / source), "-o", "/dev/null"],
                       capture_output=True, text=True, check=True)
    kernels, cur = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = kernels.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+(VGPRs|AGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]|LDS Size \[bytes/block\]): (\d+)", line)
        if m and cur is not None:
            cur[m.group(1).split(" ")[0]] = int(m.group(2))
    return kernels


def test_register_and_scratch_budgets():
    jobs = [("nvfp4_46.hip", "NVFP4_46_PART", 1), ("gemm.hip", "NVFP4_46_GEMM_PART", 5),
            ("gemm.hip", "NVFP4_46_GEMM_PART", 6)]
    with ThreadPoolExecutor(3) as pool:
        quant, dma, skinny = pool.map(lambda j: _report(*j), jobs)
    # k_flat<BF16 input, round to nearest, 4/6 by squared error, no transform, codes out>
    flat = [v for k, v in quant.items() if "6k_flatILb0ELi0ELi0ELb0ELi0E" in k]
    assert len(flat) == 1
    assert flat[0]["ScratchSize"] == 0 and flat[0]["VGPRs"] <= 64 and flat[0]["Occupancy"] == 8, flat[0]
    assert all(v["ScratchSize"] == 0 for v in quant.values())       # no quantizer kernel spills
    for kernels, name in ((dma, "k_gemm_dma"), (skinny, "k_gemm_skinny")):
        mine = {k: v for k, v in kernels.items() if name in k}
        assert len(mine) >= 2, (name, list(kernels))
        assert all(v["ScratchSize"] == 0 for v in mine.values()), mine


def test_tile_kernel_budgets():
    """k_gemm_tile counts its copies by hand too, and its small shapes leave room for four waves per SIMD in
    registers (the compiler's figure, which does not know the dynamic LDS of the next test)."""
    tile = {k: v for k, v in _report("gemm.hip", "NVFP4_46_GEMM_PART", 6).items() if "k_gemm_tile" in k}
    assert len(tile) == 6 * 4, list(tile)          # six shapes x (K whole or ragged) x output type
    assert all(v["ScratchSize"] == 0 for v in tile.values()), tile
    assert all(v["Occupancy"] >= (2 if "ILi4ELi2E" in k else 4) for k, v in tile.items()), tile


def test_budgets_of_the_kernels_beside_them():
    """k_few_rows and k_gemm_scales_first count their copies by hand as well, the second with room for four waves per SIMD;
    k_tile_pair has the registers and the LDS of its stochastic half."""
    products = _report("gemm.hip", "NVFP4_46_GEMM_PART", 6)
    few = {k: v for k, v in products.items() if "k_few_rows" in k}
    first = {k: v for k, v in products.items() if "k_gemm_scales_first" in k}
    assert len(few) == 2 and len(first) == 2, list(products)
    assert all(v["ScratchSize"] == 0 for v in (*few.values(), *first.values())), (few, first)
    assert all(v["Occupancy"] >= 4 for v in first.values()), first
    quant = _report("nvfp4_46.hip", "NVFP4_46_PART", 2)
    pair = {re.search(r"k_tile_pairILi(\d)E", k).group(1): v for k, v in quant.items() if "k_tile_pair" in k}
    tile = {re.search(r"6k_tileILb0ELi1ELi(\d)E", k).group(1): v for k, v in quant.items()
            if re.search(r"6k_tileILb0ELi1ELi\dELb1ELb0ELi0E", k)}        # SR, transform, columnwise codes
    assert sorted(pair) == sorted(tile) == list("01234")
    for select, v in pair.items():
        assert v["ScratchSize"] == 0 and v["LDS"] == tile[select]["LDS"], (select, v, tile[select])
        assert v["Occupancy"] >= tile[select]["Occupancy"] - 1, (select, v, tile[select])


def test_tile_kernel_workgroups_per_compute_unit():
    """What the LDS that each shape asks for at launch (stages or partial sums, the larger) leaves of a
    compute unit's 160 KiB."""
    fits = {k: 160 * 1024 // hm.tile_shape(k)[3] for k in hm.GEMM_KERNELS if k.startswith("tile")}
    assert fits == {"tile32": 4, "tile64x32": 5, "tile64": 3, "tile64long": 1, "tile128": 1,
                    "tile256x128": 1}, fits
    waves = {k: fits[k] * hm.tile_shape(k)[2] // 64 / 4 for k in fits}         # per SIMD, by LDS alone
    assert waves == {"tile32": 8, "tile64x32": 5, "tile64": 3, "tile64long": 2, "tile128": 4,
                     "tile256x128": 2}, waves


def test_fp32_stochastic_fake_quant_leaves_room_for_four_workgroups():
    """The random words of a tile take 32 KiB of LDS.  Next to fp32 fake-quant's own 32 KiB they would leave
    two workgroups per compute unit, which pays only where registers allow no third: under the
    squared-error rule, and with the transform under the other two that compare errors."""
    tile = {k: v for k, v in _report("nvfp4_46.hip", "NVFP4_46_PART", 5).items() if "6k_tileI" in k}
    assert len(tile) == 5 * 5, list(tile)          # five selection rules x five variants
    for name, v in tile.items():
        m = re.search(r"6k_tileILb(\d)ELi(\d)ELi(\d)ELb(\d)ELb(\d)ELi(\d)E", name)
        xf32, rounding, select, rht, want_row, out = map(int, m.groups())
        assert (xf32, rounding) == (1, 1) and v["ScratchSize"] == 0
        if out == 1:                               # kOutFake
            words = select == 0 or (rht == 1 and select in (3, 4))
            assert (v["LDS"] > 160 * 1024 // 4) == words, (name, v)
            assert words or v["Occupancy"] == 3, (name, v)


@functools.lru_cache(maxsize=None)
def _assembly(part: int) -> str:
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    return subprocess.run([build.hipcc(), *flags, f"-I{build.ROOT / 'include'}", f"-I{build.PKG / 'csrc'}",
                           f"-DNVFP4_46_PART={part}", "--offload-device-only", "-S", str(build.PKG / "csrc" / "nvfp4_46.hip"),
                           "-o", "-"], capture_output=True, text=True, check=True).stdout


def test_loads_of_a_tile_go_out_together():
    """k_tile's lanes load their share of the tile (two row blocks, 16 bytes at a time) before they wait for any of it: a
    wait in between, which the compiler put there to move a register of a piece that is zero outside the
    tensor, cost fp32 fake-quant along the columns 7 to 11 %."""
    asm = _assembly(4)                             # fp32, round to nearest
    bodies = re.findall(r"^_ZN\S+6k_tileILb1ELi0ELi\dELb\dELb(\d)ELi(\d)E\S+:(.*?)^\.Lfunc_end", asm, flags=re.M | re.S)
    staged = [body for want_row, out, body in bodies if (want_row, out) != ("0", "0")]     # the others load no tile
    assert len(bodies) == 5 * 5 and len(staged) == 5 * 3
    for body in staged:
        ops = re.findall(r"global_load_dwordx4|s_waitcnt [^\n]*vmcnt", body)
        first = ops.index("global_load_dwordx4")
        assert ops[first:first + 8] == ["global_load_dwordx4"] * 8, ops[:12]


def test_packed_sign_flips_are_the_squared_error_rules():
    """BF16 pairs are flipped before they are unpacked where that saves registers for a wave more; under the other rules it was 1 to
    6 % slower.  The masks' LDS tells which a kernel does: 8 KiB, or 16 for one mask per value."""
    with ThreadPoolExecutor(2) as pool:
        kernels = [k for r in pool.map(lambda part: _report("nvfp4_46.hip", "NVFP4_46_PART", part), (1, 2)) for k in r.items()]
    seen = 0
    for name, v in kernels:
        m = re.search(r"6k_flatILb0ELi(\d)ELi(\d)ELb1ELi(\d)E", name)
        if not m:
            continue
        rounding, select, out = map(int, m.groups())
        assert v["LDS"] == 2048 + (8192 if select == 0 else 16384) + (8192 if out == 1 else 0), (name, v)
        seen += 1
    assert seen == 2 * 5 * 2, seen                 # round to nearest and stochastic, five rules, codes and fake-quant


def test_stochastic_rounding_of_the_rowwise_kernel():
    """Under the rules of absolute errors both candidates are rounded by the conversion instruction (on the subnormal grid 2 to 6 %
    slower), under the squared-error rule, and one candidate, on the subnormal grid."""
    bodies = re.findall(r"^_ZN\S+6k_flatILb0ELi1ELi(\d)ELb\dELi[01]E\S+:(.*?)^\.Lfunc_end", _assembly(2), flags=re.M | re.S)
    assert len(bodies) == 5 * 4                    # five rules x transform or not x codes and fake-quant
    for select, body in bodies:
        assert ("v_cvt_scalef32_sr_pk_fp4_f32" in body) == (select in "34"), select
