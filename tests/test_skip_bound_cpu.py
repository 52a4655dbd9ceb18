"""The skip rule of the walks, from their source's constants (no GPU).

Every RS_STEPS steps a wave asks whether any of its plain chains may reach 2^-skip before the next look:
whether max(|e^l|, |e^{l-1}|) >= 2^(-skip - RS_STEPS bits), bits being the staged bound of the next RS_STEPS
steps' growth: the largest over them of the b with |A'| + |nB'| + 1 < 2^b (grow_bits; segments of RS_STEPS values
of l from l0 on).  The lanes of the adjoint trail by up to 15 steps, so it takes the larger of the segment and
the one before.  A scaled chain, below 2^-900 then, is not asked.  Modelled here on the columns of
test_kernel_bounds, up to l = 16384."""
import os
import re

import numpy as np

from test_kernel_bounds import coefficients, columns, normalisation

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = open(os.path.join(ROOT, "paper_1002_1050_amd", "csrc", "tc_kernels.hip")).read()
SKEW = 15          # steps the last lane of the adjoint's rows of 16 trails


def constant(name):
    return int(re.search(r"constexpr int %s = (-?\d+);" % name, SRC).group(1))


RS, BITS, FOLD = constant("RS_STEPS"), constant("GROWTH_BITS_PER_STEP"), constant("FOLD_EXP")
SKIP = 100


def step_factors(mb, ms, lmax):
    """|A'| + |nB'| + 1 of the steps from l = l0 on: the most a step grows max(|e^l|, |e^{l-1}|), |x| <= 1."""
    l0 = max(abs(mb), ms)
    l = np.arange(l0, lmax, dtype=np.int64)
    if l.size == 0:
        return np.ones(0)
    F0, F1, _ = coefficients(l, mb, ms)
    _, alpha = normalisation(l, mb, ms)
    return alpha * F0 * (1.0 + np.abs(F1)) + 1.0


def grow_bits(v):
    """The kernel's expression on the high words of v: the b with v < 2^b <= 2 v."""
    return (v.view(np.uint64) >> np.uint64(52)).astype(np.int64) - 1022


def test_source_states_the_modelled_rule():
    assert re.search(r"grow_bits\(double A, double nB\)\s*\{\s*return \(__double2hiint\(fabs\(A\) \+ fabs\(nB\) \+ 1\.0\) >> 20\) - 1022;", SRC)
    assert "(1023 - skip_exp - bits * RS_STEPS) << 20" in SRC
    assert constant("NORM_SEG") == RS           # one bound per segment
    assert constant("ROW") - 1 == SKEW <= RS


def test_grow_bits_bounds_its_argument():
    v = np.concatenate([2.0 ** np.arange(0, 18), np.nextafter(2.0 ** np.arange(1, 18), 0.0), [1.5, 3.0, 65537.0]])
    b = grow_bits(v)
    assert np.all(v < 2.0 ** b) and np.all(2.0 ** b <= 2.0 * v)


def test_staged_bound_covers_every_look():
    lmax, worst = 16384, 0
    for mb, ms in columns(lmax):
        f = step_factors(mb, ms, lmax)
        if f.size == 0:
            continue
        f = np.concatenate([f, np.ones(-f.size % RS + RS)])       # the switched-off steps: A' = nB' = 0
        bits = grow_bits(f).reshape(-1, RS).max(axis=1)
        worst = max(worst, int(bits.max()))
        lg = np.concatenate([[0.0], np.cumsum(np.log2(f))])       # growth up to a step, in bits
        s = np.arange(bits.size - 1)
        assert np.all(lg[RS * s + RS] - lg[RS * s] <= RS * bits[s]), (mb, ms)          # forward
        both = np.maximum(bits[s], np.concatenate([[0], bits[s[:-1]]]))                 # adjoint
        for k in range(SKEW + 1):
            a = np.maximum(RS * s - k, 0)           # lane k: from offset a (its seed until it starts)
            e = RS * s + RS - k
            assert np.all(lg[e] - lg[a] <= RS * both), (mb, ms, k)
    assert worst <= BITS


def test_thresholds_are_exponents():
    assert 1023 - SKIP - RS * BITS >= 1             # a biased exponent of a normal double
    assert RS * BITS < 1023                         # a chain left scaled below 1 does not overflow
    assert FOLD + RS * BITS <= -SKIP                # nor reach the skip threshold before the next look
