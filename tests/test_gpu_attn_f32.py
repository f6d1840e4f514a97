"""fp32 attention on the matrix instructions (prefill tiles of 16 queries,
decode over short contexts) against the float64 oracle, at the edges of its
tiles: query tiles, pages and groups of 8 pages, K batches, 16-row value tiles.
Latent slots past the context hold NaN throughout."""

import numpy as np
import pytest
import torch

import oracle
from paper_2607_15456_amd import lla, workloads as W
from tests.helpers import assert_close, f64, log
from tests.test_gpu_prefill import SMALL, _case, _oracle

pytestmark = pytest.mark.gpu

DEV, F32 = "cuda", torch.float32


def _heads(M, p0, r_v, d_head=128, d_rope=0):
    """The fewest of some head counts with which one sequence's M queries take the matrix kernel."""
    return next(h for h in (3, 12, 16, 28, 35, 66, 130, 400, 800)
                if lla.lib().lla_internal_f32_matrix_prefill(1, h, M, p0, r_v, d_head, d_rope))


@pytest.mark.parametrize("r_k,r_v", [(18, 30), (33, 17), (1, 1), (96, 160), (130, 129), (288, 480), (512, 512)])
@pytest.mark.parametrize("M,p0", [(16, 0), (17, 47), (15, 63), (33, 500), (1, 511), (40, 1030)])
def test_prefill_tiles(r_k, r_v, M, p0):
    if r_v <= 256 and M < 16 and p0 > 64:
        M += 32  # the same edges with queries enough for the matrix kernel
    if r_v <= 32:
        M = 256 + M
    wl = W.Workload("f32_tiles", 1, _heads(M, p0, r_v), 128, 4, 1, 0, ((r_k, r_v),), F32)
    log(f"prefill fp32 tiles r=({r_k},{r_v}) H={wl.H} M={M} p0={p0}")
    q, ck, cv, uk, uv, muk, muv, pk, pv = _case(wl, r_k, r_v, 1, M, p0, F32)
    out = lla.prefill_attn(q, pk, pv, uk, uv, p0=p0, mu_k=muk, mu_v=muv)
    assert_close(f64(out), _oracle(q, ck, cv, uk, uv, muk, muv, p0), F32, "prefill fp32")


def _two_per_unit(B, H, M):
    """More workgroups than compute units: below r_v = 256 two of them share one."""
    return B * H * ((M + 15) // 16) > torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("r_k,r_v", [(18, 30), (33, 17), (96, 160), (130, 129), (250, 256), (64, 128)])
@pytest.mark.parametrize("M,p0", [(300, 37), (511, 0)])
def test_prefill_many_tiles(r_k, r_v, M, p0):
    """The variant for more workgroups than compute units, with one and two value
    tiles per wavefront."""
    wl = W.Workload("f32_many", 1, 16, 128, 4, 1, 0, ((r_k, r_v),), F32)
    assert _two_per_unit(1, 16, M) and _heads(M, p0, r_v) <= 16
    log(f"prefill fp32 many tiles r=({r_k},{r_v}) M={M} p0={p0}")
    q, ck, cv, uk, uv, muk, muv, pk, pv = _case(wl, r_k, r_v, 1, M, p0, F32)
    out = lla.prefill_attn(q, pk, pv, uk, uv, p0=p0, mu_k=muk, mu_v=muv)
    assert_close(f64(out), _oracle(q, ck, cv, uk, uv, muk, muv, p0), F32, "prefill fp32")


@pytest.mark.parametrize("Hr", [1, 16])
@pytest.mark.parametrize("M", [100, 290])
def test_prefill_rotary(Hr, M):
    """The rotary rows, unwritten slots NaN, in both variants."""
    wl = W.Workload("f32_rotary", 1, 16, 128, 4, 1, 0, ((36, 60),), F32)
    r_k, r_v, dr, p0 = 36, 60, 40, 21
    N = p0 + M
    n_max = (N + 63) // 64 * 64 + 64
    assert _two_per_unit(1, 16, M) == (M == 290) and _heads(M, p0, r_v, d_rope=dr) <= 16
    q, ck, cv, uk, uv, muk, muv, pk, pv = _case(wl, r_k, r_v, 1, M, p0, F32, n_max=n_max)
    kr = W.rotary_keys(wl, dr, Hr, 0, B=1, N=N, device=DEV, dtype=F32)
    qr = W.rotary_queries(wl, dr, 0, 2, B=1, M=M, device=DEV, dtype=F32)
    rc = torch.full((1, Hr, n_max // 64, dr, 64), float("nan"), dtype=F32, device=DEV)
    lla.rope_write(kr, rc, pos0=0)
    log(f"prefill fp32 rotary Hr={Hr} M={M}")
    out = lla.prefill_attn(q, pk, pv, uk, uv, p0=p0, mu_k=muk, mu_v=muv, q_rope=lla.rope_rotate(qr, pos0=p0), r_cache=rc)
    ref = oracle.prefill_attn_rope_batched(f64(q), f64(qr), f64(ck), f64(cv), f64(kr).transpose(0, 2, 1, 3), f64(uk),
                                           f64(uv), f64(muk), f64(muv), p0=p0)
    assert_close(f64(out), ref, F32, "prefill fp32 rotary")


@pytest.mark.parametrize("d_head", [32, 96, 256])
@pytest.mark.parametrize("H", [28, 100])
def test_prefill_head_widths(H, d_head):
    wl = W.Workload("f32_width", 1, H, d_head, 4, 1, 0, ((36, 60),), F32)
    assert _heads(37, 70, 60, d_head) <= 28 and _two_per_unit(1, H, 37) == (H == 100)
    q, ck, cv, uk, uv, muk, muv, pk, pv = _case(wl, 36, 60, 1, 37, 70, F32)
    out = lla.prefill_attn(q, pk, pv, uk, uv, p0=70, mu_k=muk, mu_v=muv, out_dtype=F32)
    assert_close(f64(out), _oracle(q, ck, cv, uk, uv, muk, muv, 70), F32, f"d={d_head}")


@pytest.mark.parametrize("H", [12, 44])
@pytest.mark.parametrize("axis", ["k", "v"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("n_bad", [3, 63, 64, 70, 79])
def test_nonfinite_reaches_only_its_queries(H, axis, value, n_bad):
    """A non-finite latent at position n makes queries n .. non-finite (a value
    latent; a key latent at least where its score is not -inf) and leaves the
    queries before n as they are."""
    r_k, r_v, M = 36, 60, 90
    wl = W.Workload("f32_nonfinite", 1, H, 128, 4, 1, 0, ((r_k, r_v),), F32)
    assert lla.lib().lla_internal_f32_matrix_prefill(1, H, M, 0, r_v, 128, 0) and _two_per_unit(1, H, M) == (H == 44)
    q, ck, cv, uk, uv, muk, muv, pk, pv = _case(wl, r_k, r_v, 1, M, 0, F32)
    ref = _oracle(q, ck, cv, uk, uv, muk, muv, 0)
    cache = pk if axis == "k" else pv
    cache[0, 1, n_bad // 64, 5, n_bad % 64] = value
    out = f64(lla.prefill_attn(q, pk, pv, uk, uv, p0=0, mu_k=muk, mu_v=muv))
    assert_close(out[:, [0, 2]], ref[:, [0, 2]], F32, "the other heads")
    assert_close(out[:, 1, :n_bad], ref[:, 1, :n_bad], F32, f"queries before {n_bad}")
    hit = out[0, 1, n_bad:]
    if axis == "v" or np.isnan(value):
        assert not np.any(np.isfinite(hit)), "queries that attend it"
    else:
        # an infinite key: a score of +inf gives NaN, one of -inf weight 0
        kinds = np.isfinite(hit).all(-1) | np.isnan(hit).all(-1)
        assert kinds.all() and np.isnan(hit).any()


# with a workspace (split) or short the matrix kernel, with one, two or four value tiles per wavefront; else the scan
@pytest.mark.parametrize("r_k,r_v", [(48, 80), (96, 160), (192, 320), (300, 257)])
@pytest.mark.parametrize("N,lens", [(64, [64, 1]), (513, [513, 65]), (1500, [1500, 700]), (2048, [2048, 1985]),
                                    (4000, [3968, 64])])
@pytest.mark.parametrize("split", [False, True])
def test_decode_short_contexts(r_k, r_v, N, lens, split):
    wl = W.Workload("f32_decode", 1, 8, 128, 4, 2, N, ((r_k, r_v),), F32)
    q, ck, cv, uk, uv, muk, muv, pk, pv = _case(wl, r_k, r_v, 2, N, 0, F32)
    q = q[:, :, 0].contiguous()
    ws = lla.new_workspace(2, 8, r_v, N) if split else None
    log(f"decode fp32 r=({r_k},{r_v}) N={N} splits={lla.decode_splits(F32, 2, 8, N, r_k, r_v, with_workspace=split)} "
        f"matrix={lla.lib().lla_internal_f32_matrix_decode(2, 8, N, r_v, 128, 0, int(split))}")
    for cur in (lens, lens[::-1]):
        out = lla.decode_attn(q, pk, pv, uk, uv, n_ctx=N, ctx_len=torch.tensor(cur, dtype=torch.int32, device=DEV),
                              mu_k=muk, mu_v=muv, workspace=ws)
        ref = np.concatenate([oracle.decode_attn_batched(f64(q)[b:b + 1], f64(ck)[b:b + 1], f64(cv)[b:b + 1], f64(uk),
                                                         f64(uv), f64(muk), f64(muv), None, ctx_len=cur[b])
                              for b in range(2)])
        assert_close(f64(out), ref, F32, f"lens={cur}")
    bad = lla.decode_attn(q, pk, pv, uk, uv, n_ctx=N, ctx_len=torch.tensor([0, N + 1], dtype=torch.int32, device=DEV),
                          workspace=ws)
    assert bool(torch.isnan(bad).all())
    if split:
        assert int(ws[:4 * 2 * 8].view(torch.int32).abs().sum()) == 0
