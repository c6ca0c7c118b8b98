"""Training grids whose work order or tile configuration depends on the number of heads and
tiles: parity of every output with the fp64 oracle, so that a tile taken twice or not at all, or
a wrong edge, shows as garbage rows."""
import pytest

import oracle
import synth
from helpers import assert_close, f64, to_f64, to_gpu
from test_gpu_train import run_fwd_bwd, small_case

pytestmark = pytest.mark.gpu


def check(mw, B, H, T, D, L):
    print(f"[case] grid B={B} H={H} T={T} D={D} L={L}", flush=True)
    bits = small_case(B, H, T, D, L, seed=2000 + B * H + T + D)
    g = run_fwd_bwd(mw, bits, L)
    q, k, v, do = (f64(bits[n]) for n in ("q", "k", "v", "do"))
    o, lse = oracle.block_causal_attn_fwd(q, k, v, L)
    assert_close("o", to_f64(g["o"]), o)
    assert_close("lse", to_f64(g["lse"]), lse, max_abs=2e-3, mean_abs=2e-4)
    for n, ref in zip(("dq", "dk", "dv"), oracle.block_causal_attn_bwd(q, k, v, do, L)):
        assert_close(n, to_f64(g[n]), ref)


# Batch x heads with and without a multiple of eight heads, every remainder class (spread over 1, 2
# or 4 groups of XCDs), and tile counts that leave a partial last row of workgroup ids
@pytest.mark.parametrize("B,H,T,D,L", [(1, 1, 900, 128, 200), (1, 3, 500, 64, 100), (3, 5, 300, 72, 77),
                                       (2, 3, 650, 128, 130), (1, 10, 200, 64, 64), (1, 12, 300, 128, 100),
                                       (2, 10, 150, 72, 50), (1, 24, 140, 64, 30), (1, 9, 300, 64, 77),
                                       (1, 13, 150, 72, 50), (2, 7, 200, 128, 100)])
def test_work_order(mw, B, H, T, D, L):
    check(mw, B, H, T, D, L)


# Each tile configuration of the training forward at ragged sizes: 64-row tiles in four and in two
# key groups (a sequence shorter than a step, one past a tile, many key steps), D = 128's 128-row
# tiles, and the widest tiles (the larger grids: the other tests' training shapes)
@pytest.mark.parametrize("B,H,T,D,L", [(1, 1, 5, 128, 3), (1, 2, 511, 64, 90), (1, 2, 513, 64, 90), (1, 1, 577, 72, 577),
                                       (1, 3, 1537, 128, 257), (1, 2, 2049, 72, 300), (2, 1, 2113, 64, 1),
                                       (6, 16, 513, 128, 130), (13, 16, 330, 64, 65), (12, 16, 400, 72, 100),
                                       (11, 16, 300, 64, 70), (30, 16, 213, 64, 40), (54, 16, 290, 64, 70),
                                       (20, 16, 257, 72, 100)])
def test_forward_tiles(mw, B, H, T, D, L):
    check(mw, B, H, T, D, L)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("split", [True, False])
@pytest.mark.parametrize("B,H,D,L,S,window,nq,qlen,sink_len", [
    (1, 2, 64, 130, 4, 3, 1, 1, 0), (1, 3, 72, 96, 5, 4, 1, 33, 20), (2, 2, 64, 70, 4, 4, 2, 32, 9),
    (1, 2, 72, 300, 3, 3, 1, 64, 0), (1, 2, 64, 300, 4, 4, 1, 65, 33), (1, 2, 72, 300, 4, 4, 3, 100, 33),
    (1, 3, 64, 200, 4, 3, 3, 171, 0), (1, 2, 72, 600, 4, 4, 1, 600, 40), (1, 2, 128, 600, 4, 4, 1, 600, 40),
    (1, 2, 128, 200, 3, 2, 3, 181, 7)])
def test_cached_tiles(mw, mode, split, B, H, D, L, S, window, nq, qlen, sink_len):
    """Cached calls that take the few-row tiles at D = 64 and 72, the 128-row tiles, and (unsplit)
    the training forward's 64-row tiles; sinks, ragged rows, both visibility rules."""
    print(f"[case] cached tiles mode={mode} split={split} B={B} H={H} D={D} L={L} w={window} nq={nq} ql={qlen} "
          f"sink={sink_len}", flush=True)
    cache = mw.KVCache(S, B, H, L, D)
    chunks = [tuple(synth.normal_bf16((B, H, L, D), 6000 + 2 * c + i) for i in range(2)) for c in range(window)]
    for kc, vc in chunks:
        mw.mw_kvcache_append(cache, to_gpu(kc), to_gpu(vc))
    kw = {}
    if sink_len:
        sk, sv = (synth.normal_bf16((B, H, sink_len, D), 6100 + i) for i in range(2))
        cache.set_sink(to_gpu(sk), to_gpu(sv))
        kw = dict(sink_k=f64(sk), sink_v=f64(sv))
    x = [synth.normal_bf16((B, H, nq * qlen, D), 6200 + i) for i in range(3)]
    o, lse = mw.mw_chunk_attn_cached(*(to_gpu(t) for t in x), nq, qlen, cache, flags=mode, want_lse=True, split=split)
    ro, rl = oracle.cached_chunk_attn(*(f64(t) for t in x), [f64(c[0]) for c in chunks], [f64(c[1]) for c in chunks],
                                      nq, qlen, mode=mode, **kw)
    assert_close("o", to_f64(o), ro)
    assert_close("lse", to_f64(lse), rl, max_abs=2e-3, mean_abs=2e-4)
