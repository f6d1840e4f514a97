"""Host-side values and choices of the launches (no GPU: the library assumes 256
compute units without one)."""

import ctypes
import decimal

import pytest

from paper_2607_15456_amd import lla


@pytest.fixture(scope="module")
def host():
    return ctypes.CDLL(lla.LIB_PATH)


@pytest.mark.parametrize("base", [1.5, 100.0, 1e4, 5e5, 1e6, 1e30, 1.7e308])
def test_rope_frequency(host, base):
    """Frequencies base^(-2 f / 128) within 2^-52: a position's angle is the
    position times the frequency, so their errors count from far positions on
    (2^31 positions of a query: 2^-21)."""
    fn = host.lla_internal_rope_frequency
    fn.restype, fn.argtypes = ctypes.c_double, [ctypes.c_double] * 2
    with decimal.localcontext() as ctx:
        ctx.prec = 50
        ln = decimal.Decimal(base).ln()
        for f in range(64):
            c = -2.0 * f / 128
            exact = (ln * decimal.Decimal(c)).exp()
            err = abs(decimal.Decimal(fn(base, c)) / exact - 1)
            assert err <= decimal.Decimal(2) ** -52, (f, float(err))
