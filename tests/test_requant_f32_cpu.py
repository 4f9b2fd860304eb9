"""The requants of the tile kernels, checked on the CPU against the definition
clamp(floor(x), 0, qmax), x = (u M + 2^(sh-1)) 2^-sh with u = t + bias (+ the
identity shortcut): one fma rounding towards minus infinity, in fp32 (|u|, M <
2^24) and in fp64 (every parameter), and the 2-bit form by FP4 conversions
(shifts up to 21).  The first two tests hold the fma's rounding to nearest
against them: y = RN(x) gives min(trunc(y), 3) up to a shift of 22 and fails past
it, which is why the kernels set the rounding mode.  x is exact in float64 there
(|u M| < 2^48) and numpy's float64 -> float32 conversion rounds it once to
nearest even, as an fma does."""
import numpy as np


def _definition(u, m, sh):
    num = u * m + (1 << (sh - 1))
    return np.clip(np.floor_divide(num, 1 << sh), 0, 3)


def _fp32_path(u, m, sh):
    x = (u.astype(np.float64) * float(m) + 2.0 ** (sh - 1)) / 2.0 ** sh  # exact
    y = x.astype(np.float32).astype(np.float64)                          # one rounding
    return np.minimum(np.where(y > 0, np.trunc(y), 0.0), 3.0).astype(np.int64)


def _cases(m, sh, rng):
    """u near every step of the 2-bit staircase (both sides of each
    threshold), at the ends of the range and at random."""
    us = [np.arange(-3000, 3001)]
    if m != 0:
        for k in range(1, 4):
            th = -(-((2 * k - 1) << (sh - 1)) // m)  # ceil, the step to code k for m > 0
            us.append(np.arange(th - 3000, th + 3001))
    us.append(np.array([-(1 << 24) + 1, (1 << 24) - 1]))
    us.append(rng.integers(-(1 << 24) + 1, 1 << 24, 20000))
    u = np.concatenate(us).astype(np.int64)
    return u[np.abs(u) < (1 << 24)]


MULTS = [1, 2, 3, 5, 7, 255, 1 << 14, (1 << 14) + 1, (1 << 15) - 1, 46341, (1 << 20) - 3, (1 << 23) + 1,
         (1 << 24) - 1, 0, -1, -((1 << 15) - 1)]


def test_fp32_requant_equals_definition_within_bounds():
    rng = np.random.default_rng(2208)
    for sh in range(1, 23):
        for m in MULTS + [int(v) for v in rng.integers(1, 1 << 24, 4)]:
            u = _cases(m, sh, rng)
            want = _definition(u, m, sh)
            got = _fp32_path(u, m, sh)
            bad = np.nonzero(got != want)[0]
            assert bad.size == 0, (sh, m, u[bad[:5]], got[bad[:5]], want[bad[:5]])


def test_fp32_requant_shift_bound_is_needed():
    """Past the bound a single fp32 rounding to nearest can cross a step: for
    large shifts some u rounds up onto the next code."""
    rng = np.random.default_rng(7)
    found = False
    for sh in (26, 27, 28):
        for m in [(1 << 24) - 1, (1 << 23) + 1] + [int(v) for v in rng.integers(1 << 20, 1 << 24, 6)]:
            u = _cases(m, sh, rng)
            if np.any(_fp32_path(u, m, sh) != _definition(u, m, sh)):
                found = True
    assert found


def test_round_down_requant_equals_definition_for_every_shift():
    """The tile kernels' other form: one fma rounding towards minus infinity.
    Integers are representable in fp32, so floor(RD(x)) = floor(x)."""
    rng = np.random.default_rng(11)
    for sh in list(range(1, 63)):
        for m in [1, 3, 46341, (1 << 24) - 1, int(rng.integers(1, 1 << 24))]:
            us = [0, 1, (1 << 24) - 1] + [int(v) for v in rng.integers(1, 1 << 24, 20)]
            for k in (1, 2, 3, 8, 15):  # the step to code k, both sides
                th = -(-((2 * k - 1) << (sh - 1)) // m)
                us += [v for v in (th - 1, th, th + 1) if 0 <= v < 1 << 24]
            for u in us:
                num = u * m + (1 << (sh - 1))
                drop = max(0, num.bit_length() - 24)
                assert min(((num >> drop) << drop) >> sh, 15) == min(num >> sh, 15), (sh, m, u)


def test_fp64_round_down_requant_equals_definition():
    """The wide builds: the same fma in fp64, over the whole parameter range
    (u = t + bias + shortcut below 2^32, M below 2^31, every shift)."""
    rng = np.random.default_rng(12)
    for sh in range(1, 63):
        for m in [1, (1 << 31) - 1, (1 << 30) + 1] + [int(v) for v in rng.integers(1, 1 << 31, 5)]:
            us = [0, 1, (1 << 32) - 1] + [int(v) for v in rng.integers(1, 1 << 32, 20)]
            for k in (1, 2, 3, 8, 15, 200, 255):
                th = -(-((2 * k - 1) << (sh - 1)) // m)
                us += [v for v in (th - 1, th, th + 1) if 0 <= v < 1 << 32]
            for u in us:
                num = u * m + (1 << (sh - 1))
                drop = max(0, num.bit_length() - 53)
                assert min(((num >> drop) << drop) >> sh, 255) == min(num >> sh, 255), (sh, m, u)


def test_fp4_conversion_requant_equals_definition():
    """The 2-bit form by the FP4 conversion, shifts up to 21: z = clamp(RN32(v / 4
    + 2^-24)) to [0, 1], v = u M 2^-sh, and the nibble RNE(4 z) with 4 taken to
    3."""
    rng = np.random.default_rng(13)
    for sh in range(1, 22):
        for m in MULTS + [int(v) for v in rng.integers(1, 1 << 24, 4)]:
            u = _cases(m, sh, rng)
            v = (u * m).astype(np.float64) / 2.0 ** sh + 2.0 ** -22  # exact
            z = np.clip((v / 4).astype(np.float32), np.float32(0), np.float32(1))
            got = np.minimum(np.rint(z.astype(np.float64) * 4), 3).astype(np.int64)
            want = _definition(u, m, sh)
            bad = np.nonzero(got != want)[0]
            assert bad.size == 0, (sh, m, u[bad[:5]], got[bad[:5]], want[bad[:5]])
