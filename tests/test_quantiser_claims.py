"""Host-side pin of the arithmetic claim behind the quantiser that the fused prologues apply to 16-bit activations
(paper: Appendix table of quantisation configurations, per-token symmetric int4 activations; q = clamp(round(y / S))).

The kernels do not divide: they round y (1/S) + 1536 once, to a multiple of 2^-13, and that to an integer by a second addition.
The claim is that for y with at most 11 significant bits (fp16, bf16) and S an fp16 number this gives, after
clamping, exactly the integer that rounding the correctly rounded binary32 quotient y / S gives -- ties included -- and that
a reciprocal that is off by one unit in the last place does not change that.  The check below evaluates both sides with
numpy on every finite fp16 input (and the bf16 inputs of 52 exponents) for several hundred scales.  The fused multiply-adds
are evaluated in binary64, where the products and the first sum are exact.

Nor do they divide for S itself: the product of the clipping ratio and the maximum is multiplied by the seventh and corrected by its
exact residual, and that quotient is rounded to binary32 before it is rounded to fp16.
"""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2502_15779_amd import _build


def _fma32(a, b, c):
    """Binary32 fused multiply-add of binary32 arrays, through binary64 (exact product; see the module text)."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


def _kernel_side(y, rs):
    """The code by two additions: y (1/S) + 1536 snaps to a multiple of 2^-13, the second one rounds it to an integer."""
    v = _fma32(y, np.float32(rs), np.float32(1536.0))
    code = (v + np.float32(12582912.0 - 1536.0 + 8.0)).astype(np.float32)
    return (np.clip(code, np.float32(12582912.0), np.float32(12582927.0)) - np.float32(12582920.0)).astype(np.int32)


def _definition(y, s):
    return np.clip(np.rint((y / np.float32(s)).astype(np.float32)), -8, 7).astype(np.int32)


def _scales():
    rng = np.random.default_rng(20250215)
    bits = np.concatenate([rng.integers(1, 0x7C00, size=300, dtype=np.int64),        # anywhere, subnormals included
                           rng.integers(0x2C00, 0x4400, size=200, dtype=np.int64),    # around the scales of real layers
                           np.array([1, 2, 0x03FF, 0x0400, 0x3400, 0x3C00, 0x3C01, 0x3BFF, 0x7BFF], dtype=np.int64)])
    return bits.astype(np.uint16).view(np.float16).astype(np.float32)


def _reciprocal(s, ulp):
    rs = np.float32(1.0) / np.float32(s)
    return rs if ulp == 0 else np.nextafter(rs, np.float32(np.inf) if ulp > 0 else np.float32(0.0), dtype=np.float32)


@pytest.mark.parametrize("ulp", [0, -1, 1])
def test_snapped_quotient_rounds_like_the_division_for_every_fp16_input(ulp):
    y_all = np.arange(0x10000, dtype=np.uint32).astype(np.uint16).view(np.float16)
    y = y_all[np.isfinite(y_all)].astype(np.float32)
    ties = 0
    for s in _scales():
        got, want = _kernel_side(y, _reciprocal(s, ulp)), _definition(y, s)
        assert np.array_equal(got, want), (float(s), y[got != want][:4])
        t = y.astype(np.float64) / np.float64(s)
        ties += int(np.count_nonzero((np.abs(t) < 8.5) & (np.abs(t - np.floor(t)) == 0.5)))
    assert ties > 1000       # the sweep really does sit on rounding ties, a couple of thousand times


@pytest.mark.parametrize("ulp", [0, -1, 1])
def test_snapped_quotient_rounds_like_the_division_for_bf16_inputs(ulp):
    # bf16 numbers: the upper 16 bits of a binary32, every mantissa of the exponents that matter
    hi = np.arange(0x3000, 0x4A00, dtype=np.uint32)
    y = (np.concatenate([hi, hi | 0x8000]) << 16).view(np.float32)
    for s in _scales():
        got, want = _kernel_side(y, _reciprocal(s, ulp)), _definition(y, s)
        assert np.array_equal(got, want), (float(s), y[got != want][:4])


def test_plain_reciprocal_product_does_not_round_like_the_division():
    """The pin has teeth: rounded by itself, the product y * (1/S) lands on the wrong side of some ties."""
    allbits = np.arange(0x10000, dtype=np.uint32).astype(np.uint16)
    y_all = allbits.view(np.float16)
    y_all = y_all[np.isfinite(y_all)].astype(np.float32)
    wrong = 0
    for s in _scales()[300:400]:
        y = y_all[np.abs(y_all) <= np.float32(40.0) * s]
        rs = np.float32(1.0) / np.float32(s)
        plain = np.clip(np.rint((y * rs).astype(np.float32)), -8, 7).astype(np.int32)
        wrong += int(np.count_nonzero(plain != _definition(y, s)))
    assert wrong > 0


# ---- the scale ----
def test_the_scale_is_the_rounded_quotient_by_seven():
    rng = np.random.default_rng(3)
    p = np.concatenate([rng.integers(0x00800000, 0x7F800000, size=400000), np.arange(0x3F800000, 0x40800000, 37),
                        np.array([0x7F7FFFFF, 0x477FE000, 0x33800000, 0x00800000])]).astype(np.uint32).view(np.float32)
    with np.errstate(under="ignore"):
        seventh = np.float32(0.142857149243354797363)
        q0 = (p * seventh).astype(np.float32)
        raw = _fma32(_fma32(-q0, np.float32(7.0), p), seventh, q0)
        want = (p / np.float32(7.0)).astype(np.float32)
    big = p >= np.float32(2.0 ** -110)
    assert np.array_equal(raw[big], want[big]) and np.all(np.abs(raw[~big]) < 2.0 ** -100)


def _quotients_on_midpoints_of_halves():
    """Binary32 maxima 7 m / 2048, m odd: their seventh is exactly half way between two halves (eleven bits and one)."""
    return (7.0 * np.arange(2049, 4096, 2) / 2048.0).astype(np.float32)


def test_the_scale_is_the_half_of_the_binary32_quotient():
    """Product, quotient and half are rounded one after the other, as the oracle does; rounding the quotient to a half in one step
    gives other scales, so a compiled kernel must not merge the two."""
    known = [(1.0, 0x3FC34A00, 0x32FA), (0.9, 0x3FDD5CE4, 0x331E)]
    for clip, bits, half in known:
        a = np.array([bits], np.uint32).view(np.float32)
        assert oracle.quantize_act(np.repeat(a, 32).reshape(1, 32), clip)[1][0] == half
    a = _quotients_on_midpoints_of_halves()
    scale = oracle.quantize_act(np.repeat(a[:, None], 32, axis=1), 1.0)[1]
    assert np.array_equal(scale, (a / np.float32(7.0)).astype(np.float32).astype(np.float16).view(np.uint16))
    seventh = np.float32(0.142857149243354797363)
    q0 = (a * seventh).astype(np.float32)
    once = (_fma32(-q0, np.float32(7.0), a).astype(np.float64) * np.float64(seventh) + q0).astype(np.float16).view(np.uint16)
    assert np.count_nonzero(once != scale) > 100


def test_the_compiled_scale_is_rounded_to_binary32_before_the_half(tmp_path):
    src = tmp_path / "scale.hip"
    src.write_text('#include "rcp_internal.hpp"\n'
                   "__global__ void scale(const float* a, float clip, uint16_t* s)\n"
                   "{ s[threadIdx.x] = rcp::scale_bits_from_amax(a[threadIdx.x], clip); }\n")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + _build.COMPILE_FLAGS
    cmd += ["-I", os.path.join(_build.ROOT, "include"), "-I", _build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(tmp_path / "scale.s")]
    subprocess.run(cmd, check=True, capture_output=True)
    text = (tmp_path / "scale.s").read_text()
    assert "v_cvt_f16_f32" in text and "mixlo" not in text and "mixhi" not in text
