"""Cached calls without a key-range split: every tile they take against the oracle, and the
training forward's rows bit for bit over a whole history.  Each case states its tile, so that a
later threshold cannot move it to another kernel unnoticed."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2608_01127_amd as pkg
import synth
from helpers import assert_close, bits_equal, f64, to_f64, to_gpu

PLAN, GROUPS4, GROUPS2, ROWS128 = range(4)


def unsplit_tile(D, BH, Tq, Tk, training_rows):
    fn = pkg.load()["_ZN2mw19cached_unsplit_tileEiiiii"]  # mw::cached_unsplit_tile(int, int, int, int, int)
    fn.restype, fn.argtypes = ctypes.c_int, [ctypes.c_int] * 5
    return fn(D, BH, Tq, Tk, training_rows)


# D, B, H, chunk length, queued chunks, committed chunks, tile
HISTORY = [
    (64, 1, 2, 40, 1, 14, GROUPS4), (64, 1, 2, 40, 1, 4, PLAN), (64, 26, 20, 40, 1, 4, ROWS128),
    (64, 54, 20, 40, 1, 4, ROWS128), (64, 1, 2, 100, 2, 6, GROUPS4), (64, 1, 3, 90, 2, 2, GROUPS2),
    (64, 3, 20, 110, 2, 4, GROUPS2), (64, 10, 20, 100, 2, 4, PLAN), (64, 10, 20, 150, 2, 2, PLAN),
    (72, 1, 2, 33, 1, 20, GROUPS4), (72, 1, 2, 33, 1, 5, PLAN), (72, 15, 20, 60, 1, 3, ROWS128),
    (72, 1, 2, 100, 2, 6, GROUPS4), (72, 1, 3, 90, 2, 2, GROUPS2), (72, 3, 20, 110, 2, 4, GROUPS2),
    (72, 8, 16, 100, 2, 4, PLAN), (128, 1, 2, 200, 3, 6, GROUPS4), (128, 1, 2, 192, 3, 4, GROUPS2),
    (128, 3, 12, 192, 3, 2, GROUPS2), (128, 4, 15, 192, 3, 2, PLAN), (128, 7, 16, 192, 3, 2, PLAN)]


@pytest.mark.parametrize("D,B,H,L,nq,n_hist,tile", HISTORY)
def test_history_tiles(D, B, H, L, nq, n_hist, tile):
    assert unsplit_tile(D, B * H, nq * L, (n_hist + nq) * L, 1) == tile


@pytest.mark.gpu
@pytest.mark.parametrize("D,B,H,L,nq,n_hist,tile", HISTORY)
def test_unsplit_rows_are_training_rows(mw, D, B, H, L, nq, n_hist, tile):
    """At D = 64 and 72 for any number of queued rows, at D = 128 for more than 512."""
    import torch
    print(f"[case] history D={D} B={B} H={H} L={L} nq={nq} hist={n_hist}", flush=True)
    T = (n_hist + nq) * L
    g = torch.Generator(device="cuda").manual_seed(D + H + L + n_hist)
    q, k, v = (torch.randn(B, H, T, D, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    cache = mw.KVCache(n_hist, B, H, L, D)
    for c in range(n_hist):
        mw.mw_kvcache_append(cache, k[:, :, c * L:(c + 1) * L], v[:, :, c * L:(c + 1) * L])
    n0 = n_hist * L
    of, lf = mw.mw_block_causal_attn_fwd(q, k, v, L)
    for mode in (0, 1) if nq == 1 else (0,):
        o, lse = mw.mw_chunk_attn_cached(q[:, :, n0:], k[:, :, n0:], v[:, :, n0:], nq, L, cache, flags=mode,
                                         want_lse=True, split=False)
        assert bits_equal(o.contiguous(), of[:, :, n0:].contiguous())
        assert torch.equal(lse, lf[:, :, n0:].contiguous())


# D, B, H, L, window, queued chunks, their rows, sink, mode, tile, heads compared
ORACLE = [
    (72, 1, 3, 96, 2, 2, 90, 0, 0, GROUPS2, None), (72, 1, 3, 96, 2, 2, 90, 0, 1, GROUPS2, None),
    (64, 1, 3, 96, 2, 2, 90, 11, 0, GROUPS2, None), (64, 1, 40, 360, 2, 2, 100, 9, 1, PLAN, [(0, 0), (0, 39)]),
    (72, 1, 40, 360, 2, 2, 100, 9, 1, PLAN, [(0, 0), (0, 39)]), (64, 1, 40, 360, 2, 4, 100, 0, 1, PLAN, [(0, 17)]),
    (72, 1, 40, 360, 2, 4, 100, 0, 1, PLAN, [(0, 17)]), (64, 32, 25, 33, 3, 1, 20, 5, 0, ROWS128, [(0, 0), (31, 24)]),
    (72, 24, 25, 33, 3, 1, 64, 5, 1, ROWS128, [(0, 0), (23, 24)]), (64, 1, 2, 130, 5, 1, 20, 5, 0, GROUPS4, None),
    (72, 1, 2, 130, 5, 1, 64, 0, 0, GROUPS4, None), (128, 1, 2, 200, 2, 3, 181, 7, 0, GROUPS2, None)]


@pytest.mark.gpu
@pytest.mark.parametrize("D,B,H,L,window,nq,qlen,sink,mode,tile,heads", ORACLE)
def test_unsplit_tiles_vs_oracle(mw, D, B, H, L, window, nq, qlen, sink, mode, tile, heads):
    print(f"[case] unsplit D={D} B={B} H={H} L={L} w={window} nq={nq} ql={qlen} sink={sink} mode={mode}", flush=True)
    Tk = sink + window * L + nq * qlen
    assert unsplit_tile(D, B * H, nq * qlen, Tk, int(mode == 0 or nq == 1)) == tile
    check(mw, D, B, H, L, window, nq, qlen, sink, mode, heads, split=False)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 1])
def test_05b_streaming_step(mw, mode):
    """The 0.5B model's streaming step (batch 2, 16 heads of width 72, 8 chunks of 600 queued tokens
    over a 6-chunk window and a 300-token sink): its plan is unsplit, in 128-row tiles."""
    print(f"[case] 0.5B streaming step mode={mode}", flush=True)
    assert unsplit_tile(72, 32, 4800, 8700, int(mode == 0)) == PLAN
    check(mw, 72, 2, 16, 600, 6, 8, 600, 300, mode, [(0, 0), (1, 15)], split=True, plan=(1, 0))


def check(mw, D, B, H, L, window, nq, qlen, sink, mode, heads, split, plan=None):
    cache = mw.KVCache(window + 1, B, H, L, D)
    chunks = [tuple(synth.normal_bf16((B, H, L, D), 7100 + 2 * c + i) for i in range(2)) for c in range(window)]
    for kc, vc in chunks:
        mw.mw_kvcache_append(cache, to_gpu(kc), to_gpu(vc))
    kw = {}
    if sink:
        sk, sv = (synth.normal_bf16((B, H, sink, D), 7200 + i) for i in range(2))
        cache.set_sink(to_gpu(sk), to_gpu(sv))
        kw = dict(sink_k=f64(sk), sink_v=f64(sv))
    if plan is not None:
        assert mw.mw_chunk_attn_cached_plan(cache, nq, qlen, window, mode) == plan
    x = [synth.normal_bf16((B, H, nq * qlen, D), 7300 + i) for i in range(3)]
    o, lse = mw.mw_chunk_attn_cached(*(to_gpu(t) for t in x), nq, qlen, cache, flags=mode, want_lse=True, split=split)
    pairs = heads or [(b, h) for b in range(B) for h in range(H)]
    ro, rl = oracle.cached_chunk_attn(*(f64(t) for t in x), [f64(c[0]) for c in chunks], [f64(c[1]) for c in chunks],
                                      nq, qlen, mode=mode, heads=pairs, **kw)
    go, gl = to_f64(o), to_f64(lse)
    at = tuple(np.array(pairs).T)
    assert_close("o", go[at], ro[at])
    assert_close("lse", gl[at], rl[at], max_abs=2e-3, mean_abs=2e-4)
