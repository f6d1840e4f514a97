"""GPU parity of lla_encode (Eq. 2 cache write) against the float64 oracle,
called through the C ABI, plus an encode -> decode chain."""

import numpy as np
import pytest
import torch

import oracle
from paper_2607_15456_amd import lla, workloads as W
from tests.helpers import GEMM1, GEMM2, TOK32, assert_close, assert_units_close, encode_route, f64, f64_dev, log, round_bf16

pytestmark = pytest.mark.gpu

DEV = "cuda"
SENTINEL = 7.0


def _inputs(wl, r_k, r_v, B, M, means, dtype):
    xk = W.stacked_kv(wl, "k", 0, B=B, M=M, device=DEV, dtype=dtype)
    xv = W.stacked_kv(wl, "v", 0, B=B, M=M, device=DEV, dtype=dtype)
    wk = W.down_projection(wl, r_k, "k", 0, DEV, dtype)
    wv = W.down_projection(wl, r_v, "v", 0, DEV, dtype)
    muk = W.stacked_mean(wl, "k", 0, DEV, dtype) if means else None
    muv = W.stacked_mean(wl, "v", 0, DEV, dtype) if means else None
    return xk, xv, wk, wv, muk, muv


def _run(wl, r_k, r_v, B, M, pos0, n_max, means, dtype):
    xk, xv, wk, wv, muk, muv = _inputs(wl, r_k, r_v, B, M, means, dtype)
    ck = torch.full((B, wl.H, n_max // 64, r_k, 64), SENTINEL, dtype=dtype, device=DEV)
    cv = torch.full((B, wl.H, n_max // 64, r_v, 64), SENTINEL, dtype=dtype, device=DEV)
    lla.encode(xk, xv, wk, wv, ck, cv, T=wl.T, pos0=pos0, mu_k=muk, mu_v=muv)
    torch.cuda.synchronize()
    return (xk, xv, wk, wv, muk, muv), ck, cv


def _check(wl, inputs, ck, cv, pos0, M, dtype, what):
    xk, xv, wk, wv, muk, muv = inputs
    for x, w, mu, c, name in ((xk, wk, muk, ck, "K"), (xv, wv, muv, cv, "V")):
        ref = oracle.encode_batched(f64(x), None if mu is None else f64(mu), f64(w))
        got = f64(lla.from_paged(c))
        assert_close(got[:, :, pos0:pos0 + M], ref, dtype, f"{what} {name}")
        untouched = np.concatenate([got[:, :, :pos0].ravel(), got[:, :, pos0 + M:].ravel()])
        assert np.all(untouched == SENTINEL), f"{what} {name}: slots outside [pos0, pos0+M) changed"


def _check_rounded(inputs, ck, cv, pos0, M):
    """The stored value is the fp32 sum rounded to bf16: half an ulp is at most
    2^-8 of the value; the sums themselves (terms of variance 1/K, with the mean's
    subtracted) are good to 1e-3 by far.  For caches of so many values that some
    exceed 8, whose rounding alone is above a max-abs of 2e-2."""
    xk, xv, wk, wv, muk, muv = inputs
    for x, w, mu, c in ((xk, wk, muk, ck), (xv, wv, muv, cv)):
        ref = oracle.encode_batched(f64(x), None if mu is None else f64(mu), f64(w))
        got = f64(lla.from_paged(c))
        new = got[:, :, pos0:pos0 + M]
        assert np.all(np.abs(new - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-3)
        assert np.all(got[:, :, :pos0] == SENTINEL) and np.all(got[:, :, pos0 + M:] == SENTINEL)


def test_tiny_fp32_encode():
    wl = W.WORKLOADS["tiny_fp32"]
    r_k, r_v = wl.ranks[0]
    for means in (False, True):
        log(f"tiny_fp32 encode means={means}")
        inputs, ck, cv = _run(wl, r_k, r_v, wl.B, wl.N, 0, wl.N, means, torch.float32)
        _check(wl, inputs, ck, cv, 0, wl.N, torch.float32, f"means={means}")


SMALL = W.Workload("enc_small", 1, 3, 128, 4, 3, 0, ((18, 30),), torch.bfloat16)


@pytest.mark.parametrize("r_k,r_v", [(18, 30), (36, 60), (96, 160), (192, 320), (7, 9), (1, 512)])
@pytest.mark.parametrize("M,pos0", [(1, 0), (1, 63), (11, 5), (21, 40), (100, 37), (64, 64), (129, 0)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_encode_ragged(r_k, r_v, M, pos0, dtype):
    n_max = 256
    log(f"encode r=({r_k},{r_v}) M={M} pos0={pos0} {dtype}")
    inputs, ck, cv = _run(SMALL, r_k, r_v, 3, M, pos0, n_max, True, dtype)
    _check(SMALL, inputs, ck, cv, pos0, M, dtype, f"M={M} pos0={pos0}")


def test_other_head_widths():
    for d, T in ((64, 4), (96, 2), (256, 1)):
        wl = W.Workload(f"enc_d{d}", 1, 2, d, T, 2, 0, ((18, 30),), torch.bfloat16)
        log(f"encode d_head={d} T={T}")
        inputs, ck, cv = _run(wl, 18, 30, 2, 70, 5, 128, True, torch.bfloat16)
        _check(wl, inputs, ck, cv, 5, 70, torch.bfloat16, f"d={d}")


def test_decode_time_write_ouro14b_shape():
    """One new token per sequence at position 4096 (the decode step's cache write)."""
    wl = W.WORKLOADS["ouro14b_decode"]
    r_k, r_v = wl.ranks[0]
    inputs, ck, cv = _run(wl, r_k, r_v, wl.B, 1, 4096, 4160, False, torch.bfloat16)
    _check(wl, inputs, ck, cv, 4096, 1, torch.bfloat16, "M=1 at 4096")


@pytest.mark.slow
def test_full_prefill_write_encode():
    """Workload 5's cache write at full size: 4 x 8192 tokens, every latent
    checked (against the oracle's Eq. 2 rounded to bf16 like the cache)."""
    wl = W.WORKLOADS["prefill_write"]
    r_k, r_v = wl.ranks[0]
    log("prefill_write encode full size")
    xk, xv, wk, wv, _, _ = _inputs(wl, r_k, r_v, wl.B, wl.N, False, torch.bfloat16)
    ck = lla.alloc_cache(wl.B, wl.H, wl.N, r_k)
    cv = lla.alloc_cache(wl.B, wl.H, wl.N, r_v)
    lla.encode(xk, xv, wk, wv, ck, cv, T=wl.T, pos0=0)
    torch.cuda.synchronize()
    for x, w, c, name in ((xk, wk, ck, "K"), (xv, wv, cv, "V")):
        got = f64_dev(lla.from_paged(c))            # [B, H, M, r]
        w64 = f64(w)
        for b in range(wl.B):
            ref = oracle.encode_batched(f64_dev(x[b:b + 1]), None, w64)
            assert_units_close(got[b:b + 1], round_bf16(ref), f"{name} sequence {b}: every (h, token)")


def test_encode_then_decode_chain_fp32():
    """Workload 1: encode 512 tokens' loop-stacked K/V, then decode at every loop."""
    wl = W.WORKLOADS["tiny_fp32"]
    r_k, r_v = wl.ranks[0]
    inputs, ck, cv = _run(wl, r_k, r_v, wl.B, wl.N, 0, wl.N, True, torch.float32)
    xk, xv, wk, wv, muk, muv = inputs
    c_k = oracle.encode_batched(f64(xk), f64(muk), f64(wk))
    c_v = oracle.encode_batched(f64(xv), f64(muv), f64(wv))
    for loop in range(wl.T):
        q = W.queries(wl, 0, loop, device=DEV, dtype=torch.float32)
        uk, uv, _, _ = W.codec_loop(wl, r_k, r_v, 0, loop, DEV, torch.float32)
        sl = slice(loop * wl.d, (loop + 1) * wl.d)
        mk, mv = muk[:, sl].contiguous(), muv[:, sl].contiguous()
        out = lla.decode_attn(q, ck, cv, uk, uv, n_ctx=wl.N, mu_k=mk, mu_v=mv,
                              workspace=lla.new_workspace(wl.B, wl.H, r_v, wl.N))
        torch.cuda.synchronize()
        ref = oracle.decode_attn_batched(f64(q), c_k, c_v, f64(uk), f64(uv), f64(mk), f64(mv))
        assert_close(f64(out), ref, torch.float32, f"chain loop {loop}")


@pytest.mark.parametrize("r_k,r_v,T,d,B,M,pos0", [
    (18, 30, 4, 128, 3, 2900, 7),     # K = 512, 16-row tiles x 2, ragged last block
    (33, 64, 4, 128, 2, 4100, 0),     # four 16-row tiles per wave
    (5, 17, 2, 128, 1, 8200, 60),     # K = 256
])
def test_encode_many_tokens(r_k, r_v, T, d, B, M, pos0):
    """Prefill-sized writes (>= 8192 tokens): the resident-weight streaming path."""
    wl = W.Workload(f"enc_many_{T}_{d}", 1, 4, d, T, B, 0, ((r_k, r_v),), torch.bfloat16)
    n_max = ((pos0 + M + 63) // 64) * 64 + 64
    log(f"encode many tokens r=({r_k},{r_v}) K={T * d} B={B} M={M} pos0={pos0}")
    inputs, ck, cv = _run(wl, r_k, r_v, B, M, pos0, n_max, True, torch.bfloat16)
    _check(wl, inputs, ck, cv, pos0, M, torch.bfloat16, f"M={M}")


@pytest.mark.parametrize("r_k,r_v,T,d,H,B,M,pos0", [
    (33, 17, 1, 96, 3, 1, 8200, 60),   # K an odd multiple of 32
    (150, 40, 3, 32, 2, 3, 2800, 5),   # more than 8 row tiles: two chunks of them
])
def test_encode_many_tokens_32(r_k, r_v, T, d, H, B, M, pos0):
    """Writes of 8192 tokens and more on the 32-token kernel: a workgroup takes
    all heads of its tokens."""
    wl = W.Workload(f"enc_many32_{T}_{d}", 1, H, d, T, B, 0, ((r_k, r_v),), torch.bfloat16)
    n_max = ((pos0 + M + 63) // 64) * 64 + 64
    assert encode_route(lla.lib(), B, M, H, T * d, r_k, r_v, pos0, True)[0] == TOK32
    log(f"encode many tokens r=({r_k},{r_v}) K={T * d} H={H} B={B} M={M} pos0={pos0}")
    inputs, ck, cv = _run(wl, r_k, r_v, B, M, pos0, n_max, True, torch.bfloat16)
    _check(wl, inputs, ck, cv, pos0, M, torch.bfloat16, f"M={M}")


@pytest.mark.parametrize("r_k,r_v,T,d,B,M,pos0", [
    (96, 160, 4, 128, 2, 300, 5),      # the 4x tier, K = 512, ragged token block
    (288, 480, 4, 128, 1, 1000, 64),   # the 1.33x tier
    (120, 200, 4, 128, 3, 257, 0),     # row blocks of 96 with ragged ends
    (96, 160, 2, 128, 1, 513, 7),      # K = 256
    (200, 8, 4, 96, 2, 400, 0),        # K = 384, one rank above 64
])
@pytest.mark.parametrize("means", [False, True])
def test_encode_many_tokens_tier_ranks(r_k, r_v, T, d, B, M, pos0, means):
    """Prompt-sized writes at the paper's per-head rank tiers: the MFMA GEMM path."""
    wl = W.Workload(f"enc_tier_{T}_{d}", 1, 8, d, T, B, 0, ((r_k, r_v),), torch.bfloat16)
    assert encode_route(lla.lib(), B, M, wl.H, T * d, r_k, r_v, pos0, means)[0] in (GEMM1, GEMM2)
    n_max = ((pos0 + M + 63) // 64) * 64 + 64
    log(f"encode tier ranks r=({r_k},{r_v}) K={T * d} B={B} M={M} pos0={pos0} means={means}")
    inputs, ck, cv = _run(wl, r_k, r_v, B, M, pos0, n_max, means, torch.bfloat16)
    _check(wl, inputs, ck, cv, pos0, M, torch.bfloat16, f"M={M}")


@pytest.mark.parametrize("r_k,r_v,T,d,H,B,M,pos0,runs", [
    (96, 160, 1, 64, 15, 2, 11900, 5, 2),      # one chunk per head; the last run 1
    (288, 480, 2, 64, 16, 1, 12230, 3, 3),     # two chunks; the last run 1
    (288, 480, 2, 128, 15, 1, 10190, 3, 2),    # four; the last run 1
    (96, 160, 3, 64, 16, 1, 22100, 0, 2),      # three
    (288, 480, 4, 128, 16, 1, 1000, 64, 1),    # 32 tokens per wavefront: always one head
])
@pytest.mark.parametrize("means", [False, True])
def test_encode_gemm_head_runs(r_k, r_v, T, d, H, B, M, pos0, runs, means):
    """Prompt-sized per-head writes where a GEMM workgroup walks a run of heads,
    over odd and even chunk counts and including a last run shorter than the
    others; every latent is checked against the oracle."""
    route, heads, _ = encode_route(lla.lib(), B, M, H, T * d, r_k, r_v, pos0, means)
    assert (route, heads) == (GEMM2 if runs > 1 else GEMM1, runs), "case no longer takes the intended runs"
    wl = W.Workload(f"enc_runs_{T}_{d}_{H}", 1, H, d, T, B, 0, ((r_k, r_v),), torch.bfloat16)
    n_max = ((pos0 + M + 63) // 64) * 64 + 64
    log(f"encode head runs r=({r_k},{r_v}) K={T * d} H={H} B={B} M={M} pos0={pos0} runs={runs} means={means}")
    inputs, ck, cv = _run(wl, r_k, r_v, B, M, pos0, n_max, means, torch.bfloat16)
    _check_rounded(inputs, ck, cv, pos0, M)


@pytest.mark.parametrize("r_k,r_v,means", [(96, 160, False), (200, 8, True)])
def test_encode_gemm_ring_slots(r_k, r_v, means):
    """Prompt-sized chunks at ranks above 64 (the GEMM write) streamed into a
    sink + window ring cache whose positions wrap: every kept position's slot
    holds the oracle's latent of that token (later tokens overwrite earlier ones)."""
    sink, window, chunks = 4, 512, [300, 500, 260]  # at most `window` tokens per call
    wl = W.Workload("enc_ring_gemm", 1, 8, 128, 4, 2, 0, ((r_k, r_v),), torch.bfloat16)
    assert all(encode_route(lla.lib(), 2, m, 8, 512, r_k, r_v, 0, means)[0] in (GEMM1, GEMM2) for m in chunks)
    B, H, K = wl.B, wl.H, wl.T * wl.d
    n_max = ((sink + window + 63) // 64) * 64
    wk = W.down_projection(wl, r_k, "k", 0, DEV, torch.bfloat16)
    wv = W.down_projection(wl, r_v, "v", 0, DEV, torch.bfloat16)
    muk = W.stacked_mean(wl, "k", 0, DEV, torch.bfloat16) if means else None
    muv = W.stacked_mean(wl, "v", 0, DEV, torch.bfloat16) if means else None
    ck = lla.alloc_cache(B, H, n_max, r_k, device=DEV)
    cv = lla.alloc_cache(B, H, n_max, r_v, device=DEV)
    refs_k, refs_v, pos = [], [], 0
    for i, M in enumerate(chunks):
        xk = W.normal((B, M, H, K), ("enc_ring_gemm", "x_k", i), 1.0, torch.bfloat16, DEV)
        xv = W.normal((B, M, H, K), ("enc_ring_gemm", "x_v", i), 1.0, torch.bfloat16, DEV)
        log(f"ring GEMM write r=({r_k},{r_v}) chunk {i}: M={M} pos0={pos} means={means}")
        lla.encode(xk, xv, wk, wv, ck, cv, T=wl.T, pos0=pos, mu_k=muk, mu_v=muv, evict=(sink, window))
        refs_k.append(oracle.encode_batched(f64(xk), None if muk is None else f64(muk), f64(wk)))
        refs_v.append(oracle.encode_batched(f64(xv), None if muv is None else f64(muv), f64(wv)))
        pos += M
    torch.cuda.synchronize()
    keep = oracle.kept_positions(pos, sink, window)
    slots = [oracle.ring_slot(p, sink, window) for p in keep]
    assert sorted(slots) == list(range(sink + window)), "kept positions must fill every slot once"
    for refs, c, name in ((refs_k, ck, "K"), (refs_v, cv, "V")):
        ref = np.concatenate(refs, axis=2)[:, :, keep]          # [B, H, kept, r]
        got = f64(lla.from_paged(c))[:, :, slots]
        assert_close(got, ref, torch.bfloat16, f"ring GEMM write {name}")


@pytest.mark.parametrize("r_k,r_v", [(1, 33), (31, 32), (96, 160)])
@pytest.mark.parametrize("M,pos0,d_head", [(1, 63, 32), (11, 60, 96), (33, 5, 128)])
def test_fp32_tiles(r_k, r_v, M, pos0, d_head):
    """fp32 writes at the edges of their 32 x 32 tiles, K = 32 (two of the four
    wavefronts idle), 96 and 512."""
    wl = W.Workload("enc_f32", 1, 3, d_head, 4 if d_head == 128 else 1, 3, 0, ((18, 30),), torch.float32)
    log(f"encode fp32 r=({r_k},{r_v}) M={M} pos0={pos0} d={d_head}")
    inputs, ck, cv = _run(wl, r_k, r_v, 3, M, pos0, 192, True, torch.float32)
    _check(wl, inputs, ck, cv, pos0, M, torch.float32, "fp32 tiles")


@pytest.mark.parametrize("r_k,r_v", [(33, 65), (160, 97), (96, 320), (36, 60)])
@pytest.mark.parametrize("B,M,pos0,T,d_head", [(1, 192, 0, 4, 128), (3, 171, 5, 4, 128), (2, 601, 61, 2, 96),
                                               (40, 13, 7, 1, 64), (90, 3, 5, 1, 64), (2, 1997, 3, 4, 128)])
@pytest.mark.parametrize("means", [False, True])
def test_gemm_tiles(r_k, r_v, B, M, pos0, T, d_head, means):
    """The GEMM write at the edges of its blocks: row blocks of 3, 2 and 1
    tiles, token blocks cut per sequence (odd lengths and positions) and over
    short sequences, an odd number of K-chunks (K = 192), one chunk (K = 64),
    32 and 64 tokens per wavefront."""
    if max(r_k, r_v) <= 64 and B * M < 256:
        M = 257  # the fewest tokens that take the GEMM at these ranks
    want = GEMM2 if M == 1997 else GEMM1
    H = next(h for h in (3, 5, 9, 17, 33, 48, 65, 97, 129, 193)
             if encode_route(lla.lib(), B, M, h, T * d_head, r_k, r_v, pos0, means)[0] == want)
    wl = W.Workload("enc_gemm", 1, H, d_head, T, B, 0, ((18, 30),), torch.bfloat16)
    n_max = (pos0 + M + 63) // 64 * 64 + 64
    log(f"encode gemm r=({r_k},{r_v}) B={B} M={M} pos0={pos0} H={H} K={T * d_head} means={means}")
    inputs, ck, cv = _run(wl, r_k, r_v, B, M, pos0, n_max, means, torch.bfloat16)
    _check_rounded(inputs, ck, cv, pos0, M)


@pytest.mark.parametrize("pos0", [0, 203, 1001])
def test_gemm_ring(pos0):
    """The GEMM write into a sink + window budget: pieces that are 8 consecutive
    aligned slots, and those that cross the ring's end or the sink."""
    H = 6
    wl = W.Workload("enc_ring", 1, H, 128, 4, 2, 0, ((18, 30),), torch.bfloat16)
    B, M, r_k, r_v, sink, window = 2, 350, 96, 160, 4, 380
    assert encode_route(lla.lib(), B, M, H, 512, r_k, r_v)[0] in (GEMM1, GEMM2)
    xk, xv, wk, wv, muk, muv = _inputs(wl, r_k, r_v, B, M, True, torch.bfloat16)
    ck = torch.full((B, H, 6, r_k, 64), SENTINEL, dtype=torch.bfloat16, device=DEV)
    cv = torch.full((B, H, 6, r_v, 64), SENTINEL, dtype=torch.bfloat16, device=DEV)
    lla.encode(xk, xv, wk, wv, ck, cv, T=4, pos0=pos0, mu_k=muk, mu_v=muv, evict=(sink, window))
    p = np.arange(pos0, pos0 + M)
    slot = np.where(p < sink, p, sink + (p - sink) % window)
    for x, w, mu, c in ((xk, wk, muk, ck), (xv, wv, muv, cv)):
        got = f64(lla.from_paged(c))
        assert_close(got[:, :, slot], oracle.encode_batched(f64(x), f64(mu), f64(w)), torch.bfloat16, f"ring {pos0}")
        rest = np.setdiff1d(np.arange(384), slot)
        assert np.all(got[:, :, rest] == SENTINEL)


@pytest.mark.parametrize("B,M", [(2048, 65536), (1, 2 ** 27 + 64)])
def test_fp32_many_workgroups(B, M):
    """2^27 tokens at four 32-row blocks, 2^24 workgroups of 256 threads, more than
    a launch's x takes: whole sequences, and one.  17 GB of inputs (both axes read
    the same) and 35 of caches."""
    K, r = 32, 33
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("80 GB of free device memory")
    gen = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randn((B, M, 1, K), generator=gen, device=DEV)
    wk, wv = (torch.randn((1, r, K), generator=gen, device=DEV) / K ** 0.5 for _ in range(2))
    ck, cv = (torch.full((B, 1, M // 64, r, 64), SENTINEL, device=DEV) for _ in range(2))
    log(f"encode fp32 of {B} x {M} tokens")
    lla.encode(x, x, wk, wv, ck, cv, T=1, pos0=0)
    torch.cuda.synchronize()
    # the first tokens, both sides of the cut between the launches, the last ones
    cut = ((1 << 24) - 1) // 4 * 32
    span = min(M, 65536)
    for b in sorted({0, min(cut // M, B - 1), min(cut // M + 1, B - 1), B - 1}):
        for m in sorted({0, min(cut, M - span) // 64 * 64, max(0, min(cut - span // 2, M - span)) // 64 * 64, M - span}):
            for w, c in ((wk, ck), (wv, cv)):
                ref = x[b, m:m + span, 0].double() @ w[0].double().t()
                got = lla.from_paged(c[b:b + 1, :, m // 64:(m + span) // 64])[0, 0].double()
                assert float((got - ref).norm() / ref.norm()) <= 1e-6, (b, m)
