"""The exact-product evaluation of heat (r = 2^-e): fma(r, lap, u) equals
u + r*lap bit for bit over h steps from a field whose nonzero magnitudes are
at least 2^(emin + e*h), emin the exponent of the smallest normal value
(no product underflows).  The oracle's contraction-on heat evaluates exactly
that form (u' = fma(r, fma(-2, u, s), u)); paper, Section 4."""
import numpy as np
import pytest

from tests.conftest import same_bits

EMIN = {np.float64: -1022, np.float32: -126}


def field(dtype, exponent, seed, n=400):
    """Random signs and significands, magnitudes in [2^exponent, 2^(exponent+3)),
    a tenth of the values zero."""
    g = np.random.default_rng(seed)
    m = np.ldexp(g.uniform(1.0, 2.0, n).astype(dtype), g.integers(exponent, exponent + 3, n))
    m = (m * g.choice([-1, 1], n)).astype(dtype)
    m[g.uniform(size=n) < 0.1] = 0
    return m


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("e", [1, 2, 3])
@pytest.mark.parametrize("h", [1, 7, 20])
def test_no_underflow_above_the_bound(oracle_mod, dtype, e, h):
    for seed in range(5):
        u0 = field(dtype, EMIN[dtype] + e * h, seed)
        r = 2.0 ** -e
        assert same_bits(oracle_mod.heat_fma(u0, h, r), oracle_mod.heat(u0, h, r))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_the_forms_differ_once_products_underflow(oracle_mod, dtype):
    """The bound is needed: among subnormal values the two forms differ."""
    u0 = field(dtype, EMIN[dtype] - 15, 7)
    assert not same_bits(oracle_mod.heat_fma(u0, 3, 0.25), oracle_mod.heat(u0, 3, 0.25))
