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


FEW, STREAM, TOK32, GEMM1, GEMM2 = range(5)


def encode_route(host, B, M, H, K, r_k, r_v, pos0=0):
    """(kernel, heads per workgroup, token blocks, rounds) of a bf16 write."""
    out = [ctypes.c_int() for _ in range(3)]
    return (host.lla_internal_encode_route(B, M, H, K, r_k, r_v, pos0, *map(ctypes.byref, out)),
            *(o.value for o in out))


@pytest.mark.parametrize("B,M,pos0", [(1, 4096, 0), (2, 3001, 0), (3, 600, 0), (3, 600, 7), (5, 500, 3), (4, 8192, 1),
                                      (7, 300, 0), (64, 257, 5), (17, 513, 0)])
def test_gemm_token_blocks(host, B, M, pos0):
    """A GEMM write's token blocks go to the 8 XCDs in turn: cutting them per
    sequence may not add more than a sixteenth to the rounds of the flattened
    tokens."""
    route, _, blocks, _ = encode_route(host, B, M, 16, 512, 240, 400, pos0)
    assert route in (GEMM1, GEMM2)
    per = 128 if route == GEMM1 else 256
    flat = -(-B * M // per)
    rounds, least = -(-blocks // 8), -(-flat // 8)
    assert rounds <= least + least // 16
    if B == 1 and pos0 == 0:
        assert blocks == flat
