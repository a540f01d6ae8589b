"""The kernels' fast forms of the dyadic requantization (Sec. 3.2.1, Eq. 1:
the scales are applied after the integer accumulation, as a dyadic multiply
and shift; rounding half up and saturation to [-127, 127] are the readings
this implementation takes), checked on the CPU against the integer
definition q = sat(floor((v * m + 2^(s-1)) / 2^s)).

* Linear epilogues.  Per channel, c = b m + 2^(s-1) folds the bias and the
  rounding into one 64-bit addend, and the accumulator is first clamped to
  [lo, hi] = [-L - b, L - b] saturated to int32, with L = floor(130 * 2^s /
  |m|) + 1 (past L the result saturates anyway; no clamp when L would exceed
  2^30):

      q = sat(int32((clamp(acc) * m + c) >> s))

  claimed exact for every shift in [1, 62], any multiplier and any bias with
  acc + b inside int32 (the method's int32 accumulator): no intermediate
  leaves int64 and the shifted value stays inside int32.
* Attention scores, 64-bit form, stored biased:

      q + 128 = clamp(int32((acc * m + 2^(s-1) + 128 * 2^s) >> s), 1, 255),

  for |acc| <= 2^20 (a 64-channel head).  The int64 value is exact for
  s <= 54; the host takes this form when the shifted value provably fits in
  int32 (any s >= 32; smaller s when |m| 2^20 / 2^s is small enough).
"""
from fractions import Fraction
import math

import numpy as np
import pytest

I32 = (-(1 << 31), (1 << 31) - 1)
I64 = (-(1 << 63), (1 << 63) - 1)


def rq_exact(acc, m, s):
    v = (acc * m + (1 << (s - 1))) >> s
    return max(-127, min(127, v))


def in_range(v, r):
    return r[0] <= v <= r[1]


# ------------------------------------------------------- linear epilogue form
def clamp_bounds(m, b, s, margin=130):
    """[lo, hi] for the accumulator; None when no clamp is needed."""
    L = 2 if m == 0 else (margin << s) // abs(m) + 1
    if L >= 1 << 30:
        return None
    return max(-L - b, I32[0]), min(L - b, I32[1])


def rq_linear(acc, b, m, s, margin=130):
    bounds = clamp_bounds(m, b, s, margin)
    a = acc if bounds is None else max(bounds[0], min(bounds[1], acc))
    c = b * m + (1 << (s - 1))
    assert in_range(c, I64), "addend overflow"
    x = a * m + c
    assert in_range(x, I64), "int64 overflow"
    v = x >> s                       # arithmetic shift: the floor
    assert in_range(v, I32), "int32 overflow"
    return max(-127, min(127, v))


def linear_cases(m, s, b, rng, n=300, kmax=1536):
    """Random accumulators over a K = 1536 int8 dot product (kept so that
    acc + b fits int32), the clamp edges and every rounding and saturation
    boundary of acc + b."""
    amax = kmax * 127 * 127
    lo_ok, hi_ok = max(-amax, I32[0] - b), min(amax, I32[1] - b)
    accs = set(int(a) for a in rng.integers(lo_ok, hi_ok + 1, n))
    accs.update({0, 1, -1, lo_ok, hi_ok})
    bounds = clamp_bounds(m, b, s)
    if bounds is not None:
        for e in bounds:
            accs.update({e - 1, e, e + 1})
    if m != 0:
        for q in list(range(-130, 131, 5)) + [-128, -127, 126, 127, 128]:
            t = Fraction((2 * q + 1) << s, 2 * m) - b  # acc + b at q + 1/2
            for a in (math.floor(t) - 1, math.floor(t), math.ceil(t), math.ceil(t) + 1):
                accs.add(a)
    return sorted(a for a in accs if lo_ok <= a <= hi_ok)


LIN_PARAMS = [(1, 13, 0), (3, 1, -5), (1 << 29, 30, 12345), (-(1 << 30), 31, -(1 << 20)),
              (12345, 20, 77), ((1 << 30) - 12345, 43, (1 << 21) - 1),
              (-((1 << 29) + 5), 40, -((1 << 21) - 1)), ((1 << 31) - 1, 43, 1 << 15),
              ((1 << 31) - 1, 36, -(1 << 15)), ((1 << 29) + 3, 38, 32768),
              ((1 << 31) - 1, 62, (1 << 31) - (1 << 25)), (1, 62, 5), (-3, 53, -(1 << 30)),
              ((1 << 31) - 1, 1, 7), (0, 17, 1 << 30), ((1 << 30) + 1, 50, -(1 << 31) + (1 << 25))]


@pytest.mark.parametrize("m,s,b", LIN_PARAMS)
@pytest.mark.parametrize("margin", [129, 130])
def test_linear_form_is_exact(m, s, b, margin):
    """Any clamp bound L in [129 * 2^s / |m| + 1, 2^30] works (the kernel's
    fp32 estimate of 130 * 2^s / |m| lies there)."""
    rng = np.random.default_rng(abs(m) % 1000 + s + margin)
    for acc in linear_cases(m, s, b, rng):
        assert rq_linear(acc, b, m, s, margin) == rq_exact(acc + b, m, s), (acc, b, m, s)


def test_linear_form_random_parameters():
    rng = np.random.default_rng(7)
    for _ in range(120):
        s = int(rng.integers(1, 63))
        m = int(rng.integers(-(1 << 31) + 1, 1 << 31))
        b = int(rng.integers(-(1 << 31) + 1, 1 << 31))
        for acc in linear_cases(m, s, b, rng, n=40):
            assert rq_linear(acc, b, m, s) == rq_exact(acc + b, m, s), (acc, b, m, s)


def test_linear_form_domain():
    """The form holds for |acc + b| < 3 * 2^30, past int32, whatever the
    multiplier and shift (the split convolution adds int32 biases to sums that
    fill int32); at 2^32 the largest multiplier with a shift that needs no clamp
    leaves int64."""
    rng = np.random.default_rng(10)
    top = (3 << 30) - 1
    for s in range(1, 63):
        for m in [(1 << 31) - 1, -(1 << 30), 1, *(int(v) for v in rng.integers(1, 1 << 31, 4))]:
            for b in [(1 << 31) - 1, -(1 << 31), 1 << 30, 0]:
                for acc in [*I32, 0, top - b, -top - b, *(int(v) for v in rng.integers(*I32, 4))]:
                    if in_range(acc, I32) and abs(acc + b) <= top:
                        assert rq_linear(acc, b, m, s) == rq_exact(acc + b, m, s), (acc, b, m, s)
    with pytest.raises(AssertionError, match="int64 overflow"):
        rq_linear((1 << 31) - 2, (1 << 31) - 1, (1 << 31) - 1, 55)


def test_linear_clamp_is_needed():
    """Without the clamp a small shift with a large multiplier leaves int32
    after the shift (m = 2^31 - 1, s = 1, acc = 2^24 gives about 2^54)."""
    m, s, acc = (1 << 31) - 1, 1, 1 << 24
    v = (acc * m + (1 << (s - 1))) >> s
    assert not in_range(v, I32)
    assert rq_linear(acc, 0, m, s) == rq_exact(acc, m, s) == 127


# ---------------------------------------------------- wide split-convolution sums
def rq_wide(t, m, s):
    """The split convolution's requantization of a 64-bit sum through the two
    halves of t: u = floor(t m / 2^(s-1)), rounded by (u + 1) >> 1."""
    p = (t & 0xffffffff) * m
    h = (t >> 32) * m + (p >> 32)
    assert in_range(p, I64) and in_range(h, I64), "int64 overflow"
    if s > 32:
        u = h >> (s - 33)
    else:
        hc = max(-512, min(511, h))
        u = ((hc << 32) + (p & 0xffffffff)) >> (s - 1)
    assert in_range(u + 1, I64), "int64 overflow"
    return max(-127, min(127, (u + 1) >> 1))


def test_wide_sum_form_is_exact():
    """Every shift, multipliers from 1 to 2^31 - 1 of both signs, sums at every
    rounding and saturation boundary that int64 holds and at its ends."""
    rng = np.random.default_rng(9)
    for s in range(1, 63):
        for m in [1, -1, 3, (1 << 31) - 1, 1 - (1 << 31), -(1 << 30),
                  *(int(v) for v in rng.integers(-(1 << 31) + 1, 1 << 31, 3)), 0]:
            ts = {0, 1, -1, *I64, 1 << 32, (1 << 32) - 1, -(1 << 32)}
            ts.update(int(v) >> int(k) for v, k in zip(rng.integers(*I64, 20),
                                                       rng.integers(0, 40, 20)))
            if m:
                for q in [-512, -129, -128, -127, -126, -1, 0, 1, 126, 127, 128, 511, 512]:
                    t = math.floor(Fraction((2 * q + 1) << s, 2 * m))
                    ts.update({t - 1, t, t + 1, t + 2})
            for t in ts:
                if in_range(t, I64):
                    assert rq_wide(t, m, s) == rq_exact(t, m, s), (t, m, s)


# ------------------------------------------------------------ 64-bit score form
def score_scale(m, s):
    """The host's form of a score scale m / 2^s: a shift in [22, 54]."""
    while s < 32 and abs(m) < 1 << 30:
        m, s = 2 * m, s + 1
    if s < 22:
        return (-(1 << 30) if m < 0 else 1 << 30), 22
    return (0, 54) if s > 54 else (m, s)


def int32_word(v):
    return ((v + (1 << 31)) % (1 << 32)) - (1 << 31)


def rq_score_fast(acc, m, s):
    """A score by the kernel's one-shift form (the high word of the product
    from shift 32 on, the low word of its 64-bit shift below), checked against
    its form for either.  Scores are kept complemented: n = -q - 1."""
    c = -(1 << (s - 1)) - 1
    x = acc * -m + c
    assert in_range(x, I64), "int64 overflow"
    v = (x >> 32) >> (s - 32) if s >= 32 else int32_word(x >> s)
    k = max(32 - s, 0)
    xk = (acc << k) * -m + (c << k)
    assert in_range(acc << k, I32) and in_range(xk, I64), "scaled form: overflow"
    n, nk = (max(-128, min(126, w)) for w in (v, (xk >> 32) >> max(s - 32, 0)))
    assert n == nk, (acc, m, s)
    return ~n


def score_cases(m, s, rng, n=400):
    accs = set(int(a) for a in rng.integers(-(1 << 20), (1 << 20) + 1, n))
    accs.update({0, 1, -1, 1 << 20, -(1 << 20)})
    if m != 0:
        for q in list(range(-130, 131, 7)) + [-128, -127, 126, 127, 128]:
            t = Fraction((2 * q + 1) << s, 2 * m)
            for a in (math.floor(t) - 1, math.floor(t), math.ceil(t), math.ceil(t) + 1):
                if abs(a) <= 1 << 20:
                    accs.add(a)
    return sorted(accs)


SCORE_PARAMS = [(1, 13), (3, 1), (1 << 29, 30), ((1 << 30) + 1, 31), (-(1 << 30), 32),
                ((1 << 30) - 12345, 43), (-((1 << 29) + 5), 40), ((1 << 20) + 7, 22),
                ((1 << 31) - 1, 54), ((1 << 31) - 1, 32), (-((1 << 31) - 1), 33),
                ((1 << 10) - 1, 1)]


@pytest.mark.parametrize("m,s", SCORE_PARAMS)
def test_score_fast_form_is_exact(m, s):
    rng = np.random.default_rng(abs(m) % 997 + s)
    for acc in score_cases(m, s, rng):
        assert rq_score_fast(acc, *score_scale(m, s)) == rq_exact(acc, m, s), (acc, m, s)


def test_score_fast_random_parameters():
    """Every shift, multipliers from 0 to 2^31 - 1 of both signs."""
    rng = np.random.default_rng(8)
    for s in range(1, 63):
        for m in [0, 1, -1, (1 << 31) - 1, 1 - (1 << 31), 1 << 30, -(1 << 30), (1 << 29) + 1,
                  *(int(v) >> int(k) for v, k in zip(rng.integers(-(1 << 31) + 1, 1 << 31, 4),
                                                     rng.integers(0, 31, 4)))]:
            m2, s2 = score_scale(m, s)
            assert 22 <= s2 <= 54 and abs(m2) < 1 << 31
            for acc in score_cases(m, s, rng, n=30):
                assert rq_score_fast(acc, m2, s2) == rq_exact(acc, m, s), (acc, m, s)


def test_score_fast_condition_is_needed():
    """Scales that the host replaces would fail as they stand: m = 2^30, s = 12
    and acc = 2^20 give 2^38, whose low word is 0, and past s = 54 the int64
    sum overflows."""
    assert int32_word((((1 << 20) * -(1 << 30)) - (1 << 11) - 1) >> 12) == -1
    assert rq_exact(1 << 20, 1 << 30, 12) == 127
    with pytest.raises(AssertionError, match="overflow"):
        rq_score_fast(1 << 20, (1 << 31) - 1, 64)


# ------------------------------------------------------ probabilities by one multiply
def p_form(I0, k_inter, k_out, m_p, s_d, n):
    """The attention host's rule for rows of n keys: 0 one multiply, 1 that and
    a shift, 2 the general form."""
    E = I0 << k_inter
    if s_d >= 0:
        if s_d > k_inter or (s_d < k_out and (E >> s_d) < 1 << k_out):
            return 2
        return 0 if s_d < k_out else 1
    if E < 1 << k_out or m_p + k_out > 30 or E > 1 << (30 - m_p):
        return 2
    return 0 if (n * E).bit_length() + m_p - 31 < k_out else 1


def test_one_multiply_probabilities_are_exact():
    """Every exponential of rows whose sum lies anywhere in [E, n E], E =
    ShiftExp(0), by the host's form against min(floor(e F / 2^sh), cap)."""
    rng = np.random.default_rng(12)
    seen = [0, 0, 0]
    for _ in range(6000):
        I0 = int(rng.integers(1, 1 << int(rng.integers(1, 15))))
        k_inter, k_out = int(rng.choice([16, 16, 4, int(rng.integers(1, 17))])), \
            int(rng.choice([8, 8, int(rng.integers(2, 9))]))
        m_p = int(rng.choice([4, 4, int(rng.integers(0, 32))]))
        s_d = int(rng.choice([-1, -1, int(rng.integers(0, 32))]))
        n, E = int(rng.integers(1, 2049)), I0 << k_inter
        form = p_form(I0, k_inter, k_out, m_p, s_d, n)
        seen[form] += 1
        if form == 2:
            continue
        cap = (1 << (k_out - 1)) - 1
        sums = {E, n * E, *(int(E * (n ** v)) for v in rng.random(6))}
        for p2 in (31, 32, 35 - m_p, (E * n).bit_length() - 1):
            sums.update(v for v in ((1 << max(p2, 0)) - 1, 1 << max(p2, 0)) if E <= v <= n * E)
        for S in sums:
            sd = s_d if s_d >= 0 else max(0, (S - 1).bit_length() + m_p - 31)
            F = ((1 << 31) - 1) // max(1, min(S >> sd, (1 << 31) - 1))
            sh = min(32 - k_out + sd, 63)
            assert sh >= 32 or F < 1 << sh
            Fs = F << (32 - sh) if sh < 32 else F
            assert Fs < 1 << 32 and (form == 1 or sh < 32)
            # the largest value, one that may be the row's only other one, and any
            for e in {E, E >> 1, S - E if S - E < E else 0, int(rng.integers(0, E + 1))}:
                got = ((e * Fs) >> 32) >> max(sh - 32, 0)
                assert got == min((e * F) >> sh, cap), (I0, k_inter, k_out, m_p, s_d, S, e)
    assert min(seen) > 300, seen
