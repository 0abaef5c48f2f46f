"""CPU: the kernels' per-block code, compiled for the host, against the oracle.

`tests/host_model/` compiles csrc/block.hpp and csrc/codec.hpp -- block scales by
multiplication with an exactness guard, both candidates, the 4-vs-6 decision from error
estimates with a fallback to the defined errors (Table 3 lines 1-14), stochastic rounding,
Philox, the Hadamard butterflies -- with the host compiler.  These tests need no GPU and
reach input ranges where a shortcut of the kernel could silently differ from the definition:
the fp32-subnormal range of the squared errors (Table 3 lines 6 / 12), the rounding
boundaries of the E4M3 block scale (Eq. (2)), exact ties (Table 3 line 13).
"""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2512_02010_amd import workloads as wl
from tests import _host_model as hm

SR_SEED, RHT_SEED = wl.C5_SR_SEED, wl.C5_RHT_SEED


def _blocks(x: torch.Tensor) -> np.ndarray:
    return x.float().numpy().reshape(-1, 16)


def _uniforms(rows, cols, seed=SR_SEED) -> np.ndarray:
    """The oracle's uniform of every element (Philox keyed by the flat element index)."""
    u = np.array([ref.sr_uniform(seed, g) for g in range(rows * cols)], np.float32)
    return u.reshape(-1, 16)


def _compare(x: torch.Tensor, rounding=ref.RTN, select=ref.SEL_46_MSE, tag=""):
    xb = wl.host_array(x)
    rows, cols = x.shape
    alpha = ref.tensor_scale(xb)
    c, s, f = ref.quantize(xb, alpha, rounding=rounding, select=select, sr_seed=SR_SEED)
    u = _uniforms(rows, cols) if rounding != ref.RTN else None
    mc, ms, mf = hm.quantize_blocks(_blocks(x), alpha, rounding, select, u)
    bad_s = int((ms.reshape(s.shape) != s).sum())
    bad_f = int((mf.reshape(f.shape) != f).sum())
    bad_c = int((mc.reshape(c.shape) != c).any(axis=1).sum())
    assert (bad_s, bad_f, bad_c) == (0, 0, 0), (tag, rounding, select, bad_s, bad_f, bad_c)
    return f


@pytest.mark.parametrize("rounding", [ref.RTN, ref.SR, ref.SR_AFTER_RTN_SELECT])
@pytest.mark.parametrize("select", [ref.SEL_46_MSE, ref.SEL_FORCE6, ref.SEL_FORCE4, ref.SEL_46_MAE,
                                    ref.SEL_46_ABSMAX])
def test_block_code_matches_oracle_on_the_workloads(rounding, select):
    for name in ("c1", "c2", "c3", "c5"):
        _compare(wl.make(name, 48, 256), rounding, select, name)


@pytest.mark.parametrize("kind", wl.ADVERSARIAL_KINDS + ("decision_stress",))
def test_block_code_matches_oracle_on_adversarial_tensors(kind):
    for dt in (torch.bfloat16, torch.float32):
        x = wl.adversarial(kind, 32, 128, dtype=dt)
        _compare(x, ref.RTN, tag=kind)
        _compare(x, ref.SR, tag=kind)


@pytest.mark.parametrize("rounding", [ref.RTN, ref.SR])
def test_decision_where_squared_errors_are_subnormal(rounding):
    """N(0,1) * 2^e for e = -40 ... -90: from about 2^-58 down the squared errors are fp32
    subnormals, where the relative-error bound behind the kernel's estimate-based decision
    does not hold (an estimate may be off by a whole subnormal step while the tolerance has
    underflowed to zero); the decision must still be the defined one, ties going to 6."""
    g = torch.Generator().manual_seed(5)
    base = torch.randn((64, 256), generator=g)
    seen_four = 0
    for e in range(-40, -92, -2):
        x = (base * 2.0 ** e).to(torch.bfloat16)
        assert float(x.abs().max()) >= 2.0 ** -89          # the contract of the tensor scale
        f = _compare(x, rounding, tag=f"2^{e}")
        seen_four += int(f.sum())
        _compare((base * 2.0 ** e).contiguous(), rounding, tag=f"fp32 2^{e}")
    assert seen_four > 1000


def test_subnormal_range_inputs_really_reach_near_ties():
    # the sweep above is only worth something if the two errors there are close or equal for
    # many blocks while not all being zero
    x = wl.adversarial("sq_underflow_72", 64, 256)
    xb = wl.bf16_bits(x)
    alpha = ref.tensor_scale(xb)
    E6, E4 = ref.block_errors(xb, alpha)
    tiny = np.float32(2.0 ** -126)
    assert (E6 < tiny).all() and (E4 < tiny).all()           # all subnormal ...
    assert (E6 > 0).mean() > 0.8 and (E4 > 0).mean() > 0.8   # ... and most of them not zero
    assert (E6 == E4).sum() > 50                             # exact ties occur
    near = (E6 != E4) & (np.abs(E6 - E4) <= np.float32(4 * 2.0 ** -149))
    assert near.sum() > 100                                  # and differences of a few steps
    f = ref.quantize(xb, alpha)[2]
    assert 0.05 < f.mean() < 0.95


@pytest.mark.parametrize("rounding", [ref.RTN, ref.SR])
def test_tile_decision_matches_oracle(rounding):
    """The 16x16-tile decision (sum of sixteen row estimates, fallback to the defined errors)
    on ordinary tensors, on near-tie patterns and where the squared errors are subnormal."""
    cases = [wl.make("c2", 64, 128), wl.make("c4", 64, 128),
             wl.adversarial("decision_stress", 64, 128)]
    cases += [wl.adversarial(k, 64, 128, dtype=dt) for k in wl.ADVERSARIAL_KINDS
              if k.startswith("sq_underflow") for dt in (torch.bfloat16, torch.float32)]
    defined_path = 0
    for x in cases:
        xb = wl.host_array(x)
        rows, cols = x.shape
        alpha = ref.tensor_scale(xb)
        _, s_ref, f_ref, _ = ref.quantize_2d(xb, alpha, rounding=rounding, sr_seed=SR_SEED)
        xf = x.float().numpy()
        u = _uniforms(rows, cols).reshape(rows, cols) if rounding == ref.SR else None
        for tr in range(rows // 16):
            for tc in range(cols // 16):
                sl = (slice(16 * tr, 16 * tr + 16), slice(16 * tc, 16 * tc + 16))
                four, s6, s4, path = hm.tile_decision(xf[sl], alpha, rounding,
                                                      None if u is None else u[sl])
                defined_path += path
                assert four == f_ref[tr, tc], (tr, tc, four, path)
                assert (s4 if four else s6) == s_ref[tr, tc]
    assert defined_path > 0


def test_block_scale_shortcut_is_exact_around_every_rounding_boundary():
    """Eq. (2): the kernel takes the E4M3 byte of b * fl(1/(alpha*M)) unless that product is
    close to a rounding boundary, where it divides.  Probe both sides of every boundary of the
    E4M3 cast, for several alpha whose reciprocals round in different directions."""
    rng = np.random.default_rng(11)
    alphas = [1.0, 1.0 / 3.0, 0.7, 1000.0 / 1536.0, 2.0 ** -40 * 1.37, 3.1e7]
    n = 0
    for alpha in alphas:
        a32 = float(np.float32(alpha))
        for M in (6, 4):
            c = float(np.float32(np.float32(a32) * np.float32(M)))
            for byte in range(0, 0x7E):
                lo, hi = ref.e4m3_decode(byte), ref.e4m3_decode(byte + 1)
                mid = 0.5 * (lo + hi)                      # exact in double
                b0 = np.float32(mid * c)
                for step in range(-6, 7):                  # fp32 neighbours of the boundary's pre-image
                    b = b0
                    for _ in range(abs(step)):
                        b = np.nextafter(b, np.float32(np.inf if step > 0 else 0), dtype=np.float32)
                    if not (b > 0):
                        continue
                    assert hm.block_scale(float(b), a32, M) == ref.block_scale(float(b), a32, float(M))
                    assert hm.block_scale_pair(float(b), a32) == (ref.block_scale(float(b), a32, 6.0),
                                                                 ref.block_scale(float(b), a32, 4.0))
                    n += 1
            for b in rng.lognormal(0.0, 3.0, 300).astype(np.float32):
                assert hm.block_scale(float(b * c), a32, M) == ref.block_scale(float(b * c), a32, float(M))
                assert hm.block_scale_pair(float(b * c), a32) == (ref.block_scale(float(b * c), a32, 6.0),
                                                                 ref.block_scale(float(b * c), a32, 4.0))
    assert n > 15000


def test_stochastic_rounding_rule_matches_oracle():
    rng = np.random.default_rng(3)
    y = np.concatenate([rng.uniform(-7, 7, 20000), rng.normal(0, 0.3, 20000),
                        np.array([0.0, -0.0, 0.25, 0.5, 5.999, 6.0, 6.5, 1e-30, -1e30])]).astype(np.float32)
    u = rng.integers(0, 1 << 24, y.size).astype(np.float32) * np.float32(2.0 ** -24)
    # thresholds hit exactly: u == (|y| - lo) / (hi - lo) must round down, one step below up
    yy = np.array([0.125, 0.625, 1.75, 2.25, 3.5, 5.0, -0.375, -4.5], np.float32)
    pp = np.array([0.25, 0.25, 0.5, 0.25, 0.5, 0.5, 0.75, 0.25], np.float32)
    y = np.concatenate([y, yy, yy, yy])
    u = np.concatenate([u, pp, pp - np.float32(2.0 ** -24), np.zeros_like(pp)])
    got, fast = hm.e2m1_sr(y, u)
    want = np.array([ref.e2m1_sr(float(a), float(b)) for a, b in zip(y, u)], np.uint8)
    assert np.array_equal(got, want)
    # the conversion instruction (as described in host_model/gfx950_on_host.hpp): every code
    # the kernels would keep is the oracle's, and they keep nearly all
    trusted = (fast & 0x80) == 0
    assert np.array_equal(fast[trusted], want[trusted])
    assert trusted.mean() > 0.999


def test_fast_stochastic_rounding_flags_every_case_it_gets_wrong():
    """Below 1 the conversion instruction cuts the value to a multiple of 2^-23 before it
    compares; the kernels must notice every (y, u) for which that changes the answer."""
    rng = np.random.default_rng(4)
    n = 300000
    a = np.concatenate([rng.uniform(0, 0.5, n // 3), 2.0 ** rng.uniform(-40, -1, n // 3),
                        rng.uniform(0.5, 1.0, n // 3)]).astype(np.float32)
    a = np.minimum(a, np.float32(0.99999994))
    # u around the threshold p = frac(2|y|): k = floor(p 2^24) + d
    p = 2.0 * a.astype(np.float64)
    p -= np.floor(p)
    k = np.floor(p * 2.0 ** 24).astype(np.int64) + rng.integers(-8, 9, n)
    k = np.clip(k, 0, (1 << 24) - 1)
    u = k.astype(np.float32) * np.float32(2.0 ** -24)
    y = a * rng.choice(np.array([-1.0, 1.0], np.float32), n)
    got, fast = hm.e2m1_sr(y, u)
    want = np.array([ref.e2m1_sr(float(p_), float(q)) for p_, q in zip(y, u)], np.uint8)
    assert np.array_equal(got, want)
    trusted = (fast & 0x80) == 0
    assert np.array_equal(fast[trusted], want[trusted])
    wrong = (fast & 0x0F) != want
    for sel in (a < 0.5, a >= 0.5):      # the cases exist in both ranges and are all flagged
        assert (wrong & sel).sum() > 1000 and not (wrong & trusted & sel).any()
    # ... and from 1 up the instruction's answer is the rule's, flagged or not
    y2 = (rng.uniform(1.0, 7.0, n) * rng.choice([-1.0, 1.0], n)).astype(np.float32)
    frac = (y2.view(np.uint32) & 0x3FFFFF).astype(np.int64)
    k2 = np.clip((frac << 2) + rng.integers(-8, 9, n), 0, (1 << 24) - 1)
    u2 = k2.astype(np.float32) * np.float32(2.0 ** -24)
    got2, fast2 = hm.e2m1_sr(y2, u2)
    want2 = np.array([ref.e2m1_sr(float(p_), float(q)) for p_, q in zip(y2, u2)], np.uint8)
    assert np.array_equal(got2, want2) and np.array_equal(fast2 & 0x0F, want2)


def test_philox_and_hadamard_match_oracle():
    rng = np.random.default_rng(5)
    for _ in range(200):
        ctr = [int(v) for v in rng.integers(0, 1 << 32, 4)]
        key = [int(v) for v in rng.integers(0, 1 << 32, 2)]
        assert hm.philox(ctr, key) == ref.philox4x32_10(ctr, key)
    for _ in range(200):
        v = (rng.normal(0, 1, 16) * 2.0 ** rng.integers(-30, 30)).astype(np.float32)
        sw = int(rng.integers(0, 1 << 32))
        assert np.array_equal(hm.rht16(v, sw).view(np.uint32), ref.rht16(v, sw).view(np.uint32))


def test_generators_of_a_wave_match_oracle():
    """The stochastic-rounding words and sign words drawn with part of the arithmetic on the scalar unit, for upper
    counter words other than 0 as well (tensors of more than 2^34 elements), and next to a carry."""
    rng = np.random.default_rng(6)
    for i in range(300):
        seed = int(rng.integers(0, 1 << 64, dtype=np.uint64))
        hi = (0, 1, int(rng.integers(0, 1 << 29)))[i % 3]      # (element numbers have 63 bits)
        lo = (0, (1 << 32) - 4, int(rng.integers(0, (1 << 32) - 4)))[i // 3 % 3]
        q, key = (hi << 32) | lo, (seed & 0xFFFFFFFF, seed >> 32)
        for groups in (1, 2, 4):
            want = [w for j in range(groups) for w in ref.philox4x32_10((lo + j, hi, 0, 0), key)]
            assert hm.sr_words_in_wave(seed, q, groups) == want, (seed, q, groups)
        for j, w in enumerate(want[:8]):
            assert ref.sr_uniform(seed, 4 * q + j) == np.float32((w >> 8) * 2.0 ** -24)
        B = (hi << 32) | lo
        assert hm.rht_sign_word_of_wave(seed, B) == ref.rht_sign_word(seed, B)


def _uniform_at_threshold(y: float, d: int):
    """The uniform d steps of 2^-24 from where the rounding of |y| < 1 turns (there the conversion
    instruction, which compares two bits less, may answer differently); None outside [0, 1)."""
    a = abs(float(y))
    if not 0.0 < a < 1.0:
        return None
    k = int(np.floor(a * 2.0 ** 25)) - (1 << 24 if a >= 0.5 else 0) + d
    return np.float32(k * 2.0 ** -24) if 0 <= k < 1 << 24 else None


@pytest.mark.parametrize("rounding", [ref.SR, ref.SR_AFTER_RTN_SELECT])
def test_near_ties_with_an_element_at_its_rounding_threshold(rounding):
    """Blocks whose two candidates' errors are within a few fp32 steps of a tie, with one uniform within
    four steps of the threshold that its element has under the scale to 4 or to 6.  The first pass
    cannot decide them, and the scale that the defined errors choose may be the one under which the
    instruction's answer is not the rule's."""
    from tests._near_ties import block_crossings
    from tests.test_oracle_order_transcriptions import _tree_of_halves
    alpha = np.float32(1.0) / np.float32(1536.0)
    rng = np.random.default_rng(4698)
    base = rng.integers(0, 1 << 24, (4096, 16)).astype(np.float32) * np.float32(2.0 ** -24)
    near = (dict(rounding=ref.SR, uniforms=lambda k: base[k], samples=24, elements=4)
            if rounding == ref.SR else {})
    blocks, us, ys = [], [], []
    for k, (v, i, first, S6, S4) in enumerate(
            block_crossings(3000 if near else 300, 4699, _tree_of_halves, float(alpha), **near)):
        for step in (-3, -1, 0, 1, 2, 4):
            w = v.copy()
            w[i] = np.uint32(first + step).view(np.float32)
            for S in (S6, S4):
                y = w * (np.float32(1.0) / (np.float32(ref.e4m3_decode(S)) * alpha))
                for e in rng.permutation(16)[:6]:
                    u = base[k].copy()
                    at = _uniform_at_threshold(y[e], int(rng.integers(-4, 3)))
                    if e != i and at is not None:
                        u[e] = at
                        blocks.append(w)
                        us.append(u)
                        ys.append((y[e], at, S == S4))
    v, u = np.stack(blocks), np.stack(us)
    passes = hm.second_passes()
    codes, scale, four = hm.quantize_blocks(v, float(alpha), rounding, ref.SEL_46_MSE, u)
    assert hm.second_passes() - passes > 0.5 * len(v)
    # how many have the element at risk under the scale that is chosen, and would come out wrong by the instruction
    y, at, under4 = (np.array(a) for a in zip(*ys))
    rule, fast = hm.e2m1_sr(y.astype(np.float32), at.astype(np.float32))
    wrong = ((fast & 0x0F) != rule) & (under4 == (four == 1))
    assert (wrong & (four == 1)).sum() > 100 and (wrong & (four == 0)).sum() > 100, (len(v), wrong.sum())
    bad = 0
    for n in range(len(v)):
        want = ref.quantize_block(v[n], float(alpha), rounding, ref.SEL_46_MSE, u[n])
        got = np.stack((codes[n] & 15, codes[n] >> 4), axis=1).reshape(16)
        bad += not (np.array_equal(got, want["codes"]) and scale[n] == want["S"] and four[n] == want["four"])
    assert bad == 0, (bad, len(v))


@pytest.mark.parametrize("select", [ref.SEL_46_MSE, ref.SEL_FORCE6, ref.SEL_FORCE4, ref.SEL_46_MAE, ref.SEL_46_ABSMAX])
@pytest.mark.parametrize("fit", ["tiny", "subnormal", "own", "saturated", "huge"])
def test_stochastic_rounding_under_scales_at_the_ends_of_their_range(select, fit):
    """Stochastic rounding takes its codes from sums on fp32's subnormal grid and one error estimate in units
    of the scale: block maxima about the smallest scale byte (both bytes 0, one of them 0, both 1 and
    up), the tensor's own range, and an alpha so small that bytes saturate and magnitudes lie far above 6."""
    rng = np.random.default_rng(4707)
    alpha = np.float32(0.37 * 2.0 ** -9)
    lo, hi = {"tiny": (-13, -8), "subnormal": (-9, -4), "own": (0, 8.5), "saturated": (8, 11), "huge": (11, 60)}[fit]
    n = 1500
    b = (np.float32(alpha) * 6.0 * 2.0 ** rng.uniform(lo, hi, (n, 1))).astype(np.float32)
    v = (b * rng.uniform(-1, 1, (n, 16)) ** 3).astype(np.float32)
    v[np.arange(n), rng.integers(0, 16, n)] = b[:, 0]
    v[rng.random((n, 16)) < 0.1] *= np.float32(0.0)                    # zeros of both signs
    u = (rng.integers(0, 1 << 24, (n, 16)) * 2.0 ** -24).astype(np.float32)
    u[rng.random((n, 16)) < 0.02] = 0.0                                # the uniform that rounds all but grid values up
    codes, scale, four = hm.quantize_blocks(v, float(alpha), ref.SR, select, u)
    zero_scales = chose_four = 0
    for k in range(n):
        want = ref.quantize_block(v[k], float(alpha), ref.SR, select, u[k])
        got = np.stack((codes[k] & 15, codes[k] >> 4), axis=1).reshape(16)
        assert np.array_equal(got, want["codes"]) and scale[k] == want["S"] and four[k] == want["four"], (k, v[k])
        zero_scales += scale[k] == 0
        chose_four += int(four[k])
    if select == ref.SEL_46_MSE and fit != "huge":
        assert 0 < chose_four < n
    if fit == "tiny":
        assert 0 < zero_scales < n
