"""Host-side values and choices of the launches (no GPU: the library assumes 256
compute units without one)."""

import ctypes
import decimal

import pytest
import torch

from paper_2607_15456_amd import lla
from tests.helpers import FEW, GEMM1, GEMM2, STREAM, TOK32, encode_route


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


@pytest.mark.parametrize("B,M,pos0", [(1, 4096, 0), (2, 3001, 0), (3, 600, 0), (3, 600, 7), (5, 500, 3), (4, 8192, 1),
                                      (7, 300, 0), (64, 257, 5), (17, 513, 0)])
def test_gemm_token_blocks(host, B, M, pos0):
    """A GEMM write's token blocks go to the 8 XCDs in turn: cutting them per
    sequence may not add more than an eighth to the rounds of the flattened
    tokens."""
    route, _, blocks = encode_route(host, B, M, 16, 512, 240, 400, pos0)
    assert route in (GEMM1, GEMM2)
    per = 128 if route == GEMM1 else 256
    flat = -(-B * M // per)
    rounds, least = -(-blocks // 8), -(-flat // 8)
    assert rounds <= least + least // 8
    if B == 1 and pos0 == 0:
        assert blocks == flat


@pytest.mark.parametrize("B,M,H,K,r_k,r_v,route", [
    # few workgroups: the 32-token kernel (us, 32-token / GEMM)
    (1, 203, 4, 512, 96, 160, TOK32),      # 8.4 / 14.6
    (2, 98, 16, 512, 120, 200, TOK32),     # 22.3 / 24.0
    (1, 1259, 1, 320, 36, 60, TOK32),      # 5.9 / 9.6
    (5, 104, 4, 256, 18, 30, TOK32),       # 5.1 / 7.6
    (2, 111, 1, 128, 65, 33, TOK32),       # 4.3 / 12.6
    (32, 70, 2, 64, 1, 33, TOK32),         # 4.5 / 10.8
    # many: the GEMM
    (1, 300, 16, 512, 96, 160, GEMM1),     # 24.4 / 20.1
    (1, 3000, 16, 512, 36, 60, GEMM2),     # 75.7 / 26.4
    (1, 197, 16, 512, 288, 480, GEMM1),    # 43.6 / 31.2
    (1, 194, 16, 512, 192, 320, GEMM1),    # 30.3 / 25.7
    (3, 217, 16, 512, 18, 30, GEMM1),      # 13.1 / 8.5
    (2, 3001, 16, 512, 192, 320, GEMM2),
    (4, 8192, 16, 512, 288, 480, GEMM2),
    (1, 300, 1, 8192, 288, 480, GEMM1),    # an LLA-2D prompt
    (1, 238, 1, 8192, 288, 480, TOK32),    # 77.5 / 79.8
    (1, 2500, 16, 320, 288, 480, GEMM1),   # 6 rounds of 32 tokens per wavefront, 4 of 64
    # other kernels
    (1, 64, 16, 512, 96, 160, FEW),
    (2, 4096, 16, 512, 18, 30, STREAM),
    (1, 3000, 16, 96, 192, 320, TOK32),    # K not a multiple of 64
])
def test_encode_route(host, B, M, H, K, r_k, r_v, route):
    assert encode_route(host, B, M, H, K, r_k, r_v)[0] == route


@pytest.mark.parametrize("B,M,p0,streams", [
    # us per call at (96, 160), 16 heads, 1 / 2 / 4 / 8 streams
    (1, 300, 7000, 8),    # 211 / 150 / 118 / 85
    (1, 1024, 0, 4),      # 47 / 38 / 32 / 33
    (1, 2048, 0, 4),      # 76 / 60 / 55 / 64
    (1, 4096, 0, 2),      # 134 / 114 / 139 / 163
    (4, 300, 2000, 2),    # 104 / 87 / 97 / 101
    (2, 3191, 0, 1),      # 126 / 146 / 186 / 217, (104, 96)
    (4, 2048, 0, 1),      # 138 / 160 / 191 / 242
    (4, 550, 274, 1),     # 67 / 68 / 71 / 78, (240, 400)
    (1, 5486, 334, 1),    # 195 / 212 / 252 / 286
    (64, 4096, 0, 1),
])
def test_key_streams(host, B, M, p0, streams):
    assert host.lla_internal_key_streams(B, 16, M, p0) == streams


def test_key_streams_grid(host):
    """More than 65535 query blocks of the smaller sizes: a grid that fits."""
    for M in (2 ** 21 + 5, 2 ** 22, 2 ** 23 + 9):
        streams = host.lla_internal_key_streams(1, 1, M, 0)
        assert streams in (1, 2, 4, 8) and -(-M // (256 // streams)) <= 65535


@pytest.mark.parametrize("B,H,n_ctx,r_v,d_head,d_rope,workspace,matrix", [
    # us, scan / matrix
    (1, 16, 512, 160, 128, 0, 1, 1),      # 26 / 24
    (1, 16, 858, 160, 128, 0, 1, 0),      # 33 / 40
    (1, 4, 1573, 160, 128, 0, 1, 1),      # 54 / 32
    (1, 16, 2833, 160, 128, 0, 0, 0),     # 106 / 133
    (4, 16, 3928, 160, 128, 0, 1, 1),     # 97 / 60
    (1, 16, 8000, 160, 128, 0, 1, 0),
    (16, 16, 512, 160, 128, 0, 1, 0),
    (1, 16, 3756, 60, 128, 0, 0, 0),      # 21 / 61
    (2, 4, 3059, 60, 128, 0, 1, 1),       # 34 / 20
    (4, 2, 935, 64, 128, 0, 0, 0),        # 14 / 22
    (1, 2, 21, 64, 256, 0, 1, 0),         # 14 / 18
    (1, 16, 1, 60, 128, 64, 1, 0),        # 11.9 / 13.5
    (1, 16, 100, 30, 128, 0, 1, 0),
    (1, 8, 4, 130, 128, 0, 1, 0),         # 18 / 20
    (1, 1, 1978, 200, 128, 0, 1, 1),      # 94 / 40
    (1, 16, 1, 480, 128, 0, 1, 1),        # 101 / 33
    (8, 16, 2551, 480, 128, 0, 1, 1),     # 581 / 222
    (32, 32, 6, 320, 128, 64, 1, 0),      # 114 / 132
    (64, 16, 19, 480, 128, 0, 1, 1),      # 214 / 135
    (64, 16, 2048, 320, 128, 0, 1, 1),
])
def test_f32_decode(host, B, H, n_ctx, r_v, d_head, d_rope, workspace, matrix):
    assert host.lla_internal_f32_matrix_decode(B, H, n_ctx, r_v, d_head, d_rope, workspace) == matrix


def test_f32_decode_splits_without_head_width():
    """lla_decode_splits does not know d_head: no split count may depend on it.
    Where the choice of kernel does (below 16 pages) both take one slice."""
    for r_v in (33, 60, 88):
        for pages in range(1, 17):
            for units in (1, 16, 128):
                n = pages * 64
                wide = lla.lib().lla_internal_f32_matrix_decode(1, units, n, r_v, 256, 0, 1)
                narrow = lla.lib().lla_internal_f32_matrix_decode(1, units, n, r_v, 128, 0, 1)
                if wide != narrow:
                    assert pages < 16 and lla.decode_splits(torch.float32, 1, units, n, 30, r_v) == 1


@pytest.mark.parametrize("B,H,M,p0,r_v,d_head,d_rope,matrix", [
    # us, scan / matrix
    (1, 16, 500, 0, 160, 128, 0, 1),      # 305 / 38
    (32, 8, 431, 271, 16, 128, 0, 1),     # 844 / 200
    (1, 1, 350, 3729, 33, 128, 64, 0),    # 55 / 86
    (2, 2, 59, 3270, 8, 128, 0, 0),       # 14 / 42
    (1, 1, 40, 600, 160, 128, 0, 0),
    (1, 16, 64, 2000, 30, 128, 0, 1),     # 50 / 32
    (1, 16, 24, 2000, 30, 128, 0, 0),
    (8, 16, 4, 73, 200, 128, 0, 1),       # 48 / 20
    (1, 16, 16, 2000, 160, 128, 0, 1),    # 85 / 78
    (1, 2, 18, 10, 33, 256, 0, 0),        # 16 / 21
    (1, 4, 1, 8, 33, 128, 64, 0),         # 14 / 16
    (1, 1, 1, 8000, 320, 128, 0, 1),
])
def test_f32_prefill(host, B, H, M, p0, r_v, d_head, d_rope, matrix):
    assert host.lla_internal_f32_matrix_prefill(B, H, M, p0, r_v, d_head, d_rope) == matrix
