"""The window kernel's evaluation forms of KS, written out here operation by
operation with every result rounded once (exact rationals), against the
oracle: the fused Laplacian, and the exact-product form for powers of two
c1 = 1/(2dx), c2 = 1/dx^2 (b kept as b/c2, the multiplications by c1 and c2
merged into the operations that take their products) over the range of
magnitudes the kernel allows it, [2^-400, 1e30] (paper, Section 6)."""
from fractions import Fraction as Q

import numpy as np
import pytest

from tests.conftest import same_bits


def rn(x):
    return float(x)          # Fraction -> nearest binary64, ties to even


def fma(a, b, c):
    return rn(Q(a) * Q(b) + Q(c))


def ks_step(u, dt, dx, exact, contracted):
    n = len(u)
    c1, c2, h = 1.0 / (2.0 * dx), 1.0 / (dx * dx), 0.5 * dt

    def half(a, base, coef):
        lap = lambda x, i: fma(-2.0, x[i], x[i - 1] + x[(i + 1) % n])      # noqa: E731
        b = [lap(a, i) for i in range(n)]
        if not exact:
            b = [x * c2 for x in b]
        out = []
        for i in range(n):
            d, l2 = a[(i + 1) % n] - a[i - 1], lap(b, i)
            if exact:
                t = fma(a[i], d * (c1 / c2), b[i]) if contracted else \
                    fma(a[i] * d, c1 / c2, b[i])
                x = fma(l2, c2, t)
                out.append(fma(-(coef * c2), x, base[i]) if contracted else
                           base[i] - (coef * c2) * x)
            else:
                t = fma(a[i], d * c1, b[i]) if contracted else a[i] * (d * c1) + b[i]
                f = -(t + l2 * c2)
                out.append(fma(coef, f, base[i]) if contracted else base[i] + coef * f)
        return out

    return half(half(u, u, h), u, dt)


def field(lo, hi, seed, n=14):
    """Magnitudes log-uniform in [2^lo, 2^hi), random signs."""
    g = np.random.default_rng(seed)
    return np.ldexp(g.uniform(1.0, 2.0, n), g.integers(lo, hi, n)) * g.choice([-1.0, 1.0], n)


@pytest.mark.parametrize("contracted", [False, True])
@pytest.mark.parametrize("dx,exact", [(0.5, True), (0.25, True), (1.0, True), (0.0625, True),
                                      (0.7, False), (0.5, False)])
@pytest.mark.parametrize("lo,hi", [(-400, -398), (-400, 99), (-3, 3), (60, 99), (-399, -340)])
def test_forms_give_the_canonical_bits(oracle_mod, lo, hi, dx, exact, contracted):
    oracle = oracle_mod.ks_fma if contracted else oracle_mod.ks
    for seed in range(6):
        u0 = field(lo, hi, seed)
        got = np.array(ks_step(list(map(float, u0)), 0.005, dx, exact, contracted))
        assert same_bits(got, oracle(u0, 1, 0.005, dx))

