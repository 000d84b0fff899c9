"""The window around bf16 rounding ties inside which jet_fused.hip's silu_grad_mul leaves its binary32 product to
binary64: a CPU model of the function, with the hardware's 2^y and reciprocal off by up to one ulp either way."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

f = np.float32
SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_14243_amd", "csrc", "jet_fused.hip")


def _window():
    m = re.findall(r"const float window = ([\d.]+)f \+ ([\d.]+)f \* fabsf\(gom\)", open(SRC).read())
    assert len(m) == 1
    return float(m[0][0]), float(m[0][1])


def _const(name):
    m = re.findall(rf"\b{name} = (0x[0-9a-fp.+-]+)f", open(SRC).read())
    assert len(set(m)) == 1
    return f(float.fromhex(m[0]))


@pytest.mark.parametrize("rcp", [-1, 0, 1])
@pytest.mark.parametrize("exp2", [-1, 0, 1])
def test_the_window_covers_the_error_of_the_binary32_product(exp2, rcp):
    """da r w against da silu'(g) for every bf16 g with |g| <= 80 and a product above 2^-100.  A relative error d is
    at most d 2^24 ulps of the product wherever its significand lies; one more covers the rounding by da."""
    a, b = _window()
    c_hi, c_lo, ln2 = _const("c_hi"), _const("c_lo"), _const("ln2")
    bits = np.arange(0, 0x42A1, dtype=np.uint32)
    g = (np.concatenate([bits, bits | 0x8000]) << 16).view(f)
    off = lambda v, n: v if n == 0 else np.nextafter(v, f(np.inf * n))
    x = g.astype(np.longdouble)
    s = 1 / (1 + np.exp(-x))
    exact = s * (1 + x * (1 - s))

    y = -g * c_hi
    assert np.array_equal(y.astype(np.float64), -g.astype(np.float64) * float(c_hi))     # the leading product is exact
    p2 = off(np.exp2(y.astype(np.longdouble)).astype(f), exp2)
    e = (p2.astype(np.float64) * ((-g * c_lo) * ln2).astype(np.float64) + p2.astype(np.float64)).astype(f)
    r = off((1.0 / (f(1) + e).astype(np.float64)).astype(f), rcp)
    gom = g * (e * r)
    w = f(1) + gom
    rw = r * w
    used = np.abs(rw) >= f(2.0 ** -100)
    ulps = np.abs((rw.astype(np.longdouble) - exact) / exact).astype(np.float64)[used] * 2.0 ** 24 + 1.0
    # the device forms |gom| / |w| with a reciprocal of its own: 2^-22 of it at most
    window = a + b * (np.abs(gom) / np.abs(w)).astype(np.float64)[used] * (1 - 2.0 ** -22)
    worst = float(np.max(ulps / window))
    print(f"exp2 {exp2:+d} ulp, rcp {rcp:+d} ulp: {worst:.2f} of the window at g = {float(g[used][np.argmax(ulps / window)])}")
    assert used.sum() > 33000 and worst < 1.0


@pytest.mark.parametrize("rcp", [-1, 0, 1])
@pytest.mark.parametrize("exp2", [-1, 0, 1])
def test_no_intermediate_value_is_subnormal(exp2, rcp):
    """The window's bound is one of relative errors: for every bf16 g with |g| <= 80, e, r, e r, g e r, w and r w are normal
    binary32 numbers (or the zero of g = 0), and r w has the sign of silu'(g) and its error within the window."""
    a, b = _window()
    c_hi, c_lo, ln2 = _const("c_hi"), _const("c_lo"), _const("ln2")
    bits = np.arange(0, 0x42A1, dtype=np.uint32)
    g = (np.concatenate([bits, bits | 0x8000]) << 16).view(f)
    off = lambda v, n: v if n == 0 else np.nextafter(v, f(np.inf * n))
    p2 = off(np.exp2((-g * c_hi).astype(np.longdouble)).astype(f), exp2)
    e = (p2.astype(np.float64) * ((-g * c_lo) * ln2).astype(np.float64) + p2.astype(np.float64)).astype(f)
    r = off((1.0 / (f(1) + e).astype(np.float64)).astype(f), rcp)
    om = e * r
    gom = g * om
    w = f(1) + gom
    rw = r * w
    for name, v in (("e", e), ("r", r), ("om", om), ("w", w), ("rw", rw)):
        assert np.abs(v).min() >= 2.0 ** -126, name
    assert (np.abs(gom[np.abs(g) >= 2.0 ** -120]) >= 2.0 ** -126).all()      # below, w is 1 whatever gom is
    x = g.astype(np.longdouble)
    s = 1 / (1 + np.exp(-x))
    exact = s * (1 + x * (1 - s))
    assert np.array_equal(np.signbit(rw), np.signbit(exact))
    ulps = np.abs((rw.astype(np.longdouble) - exact) / exact).astype(np.float64) * 2.0 ** 24 + 1.0
    window = a + b * (np.abs(gom) / np.abs(w)).astype(np.float64) * (1 - 2.0 ** -22)
    assert float(np.max(ulps / window)) < 1.0 and float(window.max()) < 32768.0


def test_zero_and_normal_products_stay_in_binary32(tmp_path):
    """The condition of the source, compiled here: what goes to binary64 is a product near a tie, below the normal range or of a
    gate beyond 80 -- not a zero gradient of either sign, which whole rows of masked tokens have."""
    src = open(SRC).read()
    cond = re.findall(r"\n    sure = (.*);\n    return prod;", src)
    limit = re.findall(r"\bkSiluRange = ([\d.]+)f", src)
    assert len(cond) == 1 and len(limit) == 1
    cpp, so = tmp_path / "sure.cpp", tmp_path / "sure.so"
    cpp.write_text(f"""#include <math.h>
static const float kSiluRange = {limit[0]}f;
extern "C" int sure(float g, float da, float prod, float dist, float window) {{ return {cond[0]}; }}
""")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", str(cpp), "-o", str(so)], check=True)
    fn = ctypes.CDLL(str(so)).sure
    fn.argtypes = [ctypes.c_float] * 5
    for sign in (1.0, -1.0):
        assert fn(1.0, 0.0 * sign, 0.0 * sign, 32768.0, 40.0)
        assert fn(-80.0, 0.0 * sign, 0.0 * sign, 32768.0, 40.0)
        assert fn(1.0, sign * 2.0 ** -124, sign * 2.0 ** -124, 32768.0, 40.0)
        assert not fn(1.0, sign * 2.0 ** -130, sign * 2.0 ** -130, 32768.0, 40.0)
        assert not fn(sign * 80.5, 1.0, 1.0, 32768.0, 40.0)
        assert not fn(sign * 80.5, 0.0, 0.0, 32768.0, 40.0)
        assert not fn(1.0, sign, sign, 39.0, 40.0)
