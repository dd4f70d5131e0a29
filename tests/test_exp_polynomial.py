"""The softmax exponential of the INT8 attention kernels (csrc/attention.hip, exp_nonpos) is a binary64 polynomial
whose result is rounded to binary32; the rounding is the correct one only if the polynomial is accurate far beyond a
binary32 ulp.  This test reads the constants out of the kernel source and replays the function on the CPU with every
fused multiply-add evaluated exactly (rational arithmetic, one rounding), against a 60-digit exponential."""
import math
import os
import random
import re
import struct
from decimal import Decimal, getcontext
from fractions import Fraction

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_2209_09130_amd", "csrc", "attention.hip")


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))          # Fraction -> float rounds to nearest even


def constants():
    text = open(SRC).read()
    body = text[text.index("double exp_nonpos(double x)"):]
    body = body[:body.index("return __builtin_ldexp")]
    num = r"-?(?:0x[0-9a-fA-F.]+p[-+]?\d+|\d+\.\d+(?:e[-+]?\d+)?)"
    lits = [float.fromhex(t) if "0x" in t else float(t) for t in re.findall(num, body)]
    # in source order: log2 e, the shift (twice: added, then taken off), the two parts of -ln 2, the coefficients
    log2e, shift, shift_again, ln2_hi, ln2_lo = lits[:5]
    assert shift_again == shift
    poly = lits[5:]
    return log2e, shift, ln2_hi, ln2_lo, poly


def exp_nonpos(x, log2e, shift, ln2_hi, ln2_lo, poly):
    shifted = fma(x, log2e, shift)
    k = shifted - shift
    r = fma(k, ln2_hi, x)
    r = fma(k, ln2_lo, r)
    p = poly[0]
    for c in poly[1:]:
        p = fma(p, r, c)
    return math.ldexp(p, int(k)), r


def test_exponential_polynomial_is_accurate_far_beyond_a_binary32_ulp():
    getcontext().prec = 60
    log2e, shift, ln2_hi, ln2_lo, poly = constants()
    assert shift == 1.5 * 2.0 ** 52 and abs(log2e - 1 / math.log(2)) < 1e-15
    assert abs(-(ln2_hi + ln2_lo) - math.log(2)) < 1e-16 and poly[-1] == 1.0 and poly[-2] == 1.0
    f32 = lambda v: struct.unpack("f", struct.pack("f", v))[0]
    rnd = random.Random(11)
    xs = [f32(-rnd.random() * 100) for _ in range(4000)] + [f32(-rnd.random() * 0.7) for _ in range(1500)] + [0.0]
    xs += [f32(-(k + 0.5) * math.log(2)) for k in range(0, 140, 3)]           # the ends of the reduced range
    xs += [-745.0, -700.25, -87.5]
    worst, r_max = 0.0, 0.0
    for x in xs:
        y, r = exp_nonpos(x, log2e, shift, ln2_hi, ln2_lo, poly)
        exact = Fraction(str(Decimal(x).exp()))
        if exact > Fraction(1, 2 ** 1000):                                   # normal results
            worst = max(worst, float(abs(Fraction(y) - exact) / exact))
        r_max = max(r_max, abs(r))
    assert r_max <= 0.34665, r_max                                            # the interval the polynomial was fitted on
    assert worst < 2.0 ** -49, math.log2(worst)
    assert exp_nonpos(0.0, log2e, shift, ln2_hi, ln2_lo, poly)[0] == 1.0
    # far below the range of binary32 the scaling flushes to zero, as the exponential does
    assert exp_nonpos(-1.0e9, log2e, shift, ln2_hi, ln2_lo, poly)[0] == 0.0


NUM = r"-?(?:0x[0-9a-fA-F.]+p[-+]?\d+|\d+\.\d+(?:e[-+]?\d+)?)"


def table_exponential():
    """exp_nonpos(float, table) of the kernel source as a function of x that returns (exp(x), f), with the powers of two
    (csrc/exp2_table.h) checked on the way."""
    getcontext().prec = 60
    text = open(os.path.join(os.path.dirname(SRC), "exp2_table.h")).read()
    entries = [int(t, 16) for t in re.findall(r"0x([0-9a-f]{16})", text)]
    assert len(entries) == 256
    ln2 = Decimal(2).ln()
    power = lambda k: struct.unpack("<d", struct.pack("<Q", entries[k & 255] + ((k << 12) << 32) & (2 ** 64 - 1)))[0]
    for j in range(256):
        assert power(j) == float((ln2 * j / 256).exp())
    assert power(-256 * 150) == 2.0 ** -150 and power(-256 * 149 + 255) == math.ldexp(power(255), -149)
    body = open(SRC).read()
    body = body[body.index("float exp_nonpos(float x, const ExpTable &table)"):]
    body = body[:body.index("const double scale")]
    lits = [float.fromhex(t) if "0x" in t else float(t) for t in re.findall(NUM, body)]
    floor, rate, shift, rate_again, shift_again = lits[:5]
    # the further parts of 256 / ln 2 (far below the polynomial's coefficients) are added to f in the order they are written
    parts, poly = lits[5:-4], lits[-4:]
    assert floor == -104.0 and rate == rate_again == float(256 / ln2) and shift == shift_again == 1.5 * 2.0 ** 52
    assert all(part == float(256 / ln2 - Decimal(rate)) for part in parts) and len(parts) <= 1

    def table_exp(x):
        x = max(x, floor)
        shifted = fma(x, rate, shift)
        k = int(shifted - shift)
        f = fma(x, rate, -(shifted - shift))
        for part in parts:
            f = fma(x, part, f)
        q = poly[0]
        for c in poly[1:]:
            q = fma(q, f, c)
        scale = power(k)
        return fma(scale, f * q, scale), f

    return table_exp


f32 = lambda v: struct.unpack("f", struct.pack("f", v))[0]


def relative_error(y, x):
    return float(abs(Fraction(y) / Fraction(str(Decimal(x).exp())) - 1))


def test_table_exponential_is_accurate_far_beyond_a_binary32_ulp():
    """Half an ulp (2^-53) from the table entry, half an ulp from the last operation, 2^-58 from the polynomial and 2^-62 from
    rounding f q(f), which is below 2^-9: below 2^-51.9 together, over the whole range of arguments."""
    table_exp = table_exponential()
    rnd = random.Random(12)
    xs = [f32(-rnd.random() * 103.9) for _ in range(4000)] + [f32(-rnd.random() * 0.7) for _ in range(1500)] + [0.0, -104.0]
    xs += [f32(-(k + 0.5) * math.log(2) / 256) for k in range(0, 38000, 301)]        # the ends of the reduced range
    worst = 0.0
    for x in xs:
        y, f = table_exp(x)
        assert abs(f) <= 0.5001
        worst = max(worst, relative_error(y, x))
    assert worst < 2.0 ** -51.9, math.log2(worst)
    assert table_exp(0.0)[0] == 1.0
    assert f32(table_exp(-1.0e9)[0]) == 0.0                                   # below half of the smallest binary32 number


def test_table_exponential_is_no_less_accurate_than_the_polynomial_anywhere():
    """Kernels of either kind serve the same calls (by sequence length), so neither may lose accuracy in a part of the range:
    mean and largest error, range by range."""
    table_exp, consts = table_exponential(), constants()
    rnd = random.Random(13)
    for lo, hi in ((-0.7, 0.0), (-5.0, -0.7), (-20.0, -5.0), (-50.0, -20.0), (-80.0, -50.0), (-104.0, -80.0)):
        xs = [f32(rnd.uniform(lo, hi)) for _ in range(1200)]
        table = [relative_error(table_exp(x)[0], x) for x in xs]
        poly = [relative_error(exp_nonpos(x, *consts)[0], x) for x in xs]
        assert sum(table) <= sum(poly) and max(table) <= max(poly), (lo, hi, sum(table) / sum(poly), max(table) / max(poly))
