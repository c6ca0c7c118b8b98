"""The key-range split of cached calls bound by streaming their window (host logic, no GPU): the
workgroups fill whole rounds of the CUs for head counts that do not divide them."""
import ctypes

import pytest

import paper_2608_01127_amd as mw
from test_abi_host import new_cache


@pytest.mark.parametrize("H,D,q_len,bm,per_cu", [(12, 128, 64, 64, 1), (24, 128, 64, 64, 1), (24, 128, 100, 128, 1),
                                                 (36, 128, 33, 64, 1), (40, 64, 64, 64, 1), (24, 72, 17, 64, 1),
                                                 (24, 72, 100, 128, 2), (20, 64, 128, 128, 2), (72, 128, 94, 128, 1)])
def test_streaming_splits_fill_rounds(H, D, q_len, bm, per_cu):
    lib = mw.load()
    c = new_cache(S=8, B=1, H=H, L=2640, D=D)
    c.head = 6
    ns, nw = ctypes.c_int(), ctypes.c_int()
    ws = lib.mw_chunk_attn_cached_workspace_size(ctypes.byref(c), 1, q_len, 6)
    assert lib.mw_chunk_attn_cached_plan(ctypes.byref(c), 1, q_len, 6, mw.MW_QUEUED_CAUSAL, ws, ctypes.byref(ns),
                                         ctypes.byref(nw)) == mw.MW_OK
    wgs, room = H * -(-q_len // bm) * ns.value, 256 * per_cu
    assert nw.value == 0 and wgs >= 0.75 * room * -(-wgs // room), (ns.value, wgs)
    assert ns.value * H * q_len * (D + 2) * 4 <= ws


@pytest.mark.parametrize("H,D,nq,q_len,L,window,sink,bm,bk", [
    (5, 128, 1, 155, 880, 24, 0, 128, 128), (20, 72, 2, 70, 880, 4, 300, 128, 64), (8, 128, 1, 129, 600, 8, 300, 128, 128),
    (4, 128, 8, 32, 1320, 4, 0, 128, 128), (16, 128, 1, 64, 2640, 6, 0, 64, 64), (5, 128, 1, 257, 600, 8, 300, 128, 128)])
def test_streaming_splits_fill_key_steps(H, D, nq, q_len, L, window, sink, bm, bk):
    """A range more, with as many workgroups on the busiest CU, would not shorten the longest range (in whole
    key steps, which a workgroup's time goes by) by a step in eight or more."""
    lib = mw.load()
    c = new_cache(S=window + 1, B=1, H=H, L=L, D=D)
    c.head = window
    c.sink_len = sink
    c.k_sink = c.v_sink = c.k_slots
    ns, nw = ctypes.c_int(), ctypes.c_int()
    ws = lib.mw_chunk_attn_cached_workspace_size(ctypes.byref(c), nq, q_len, window)
    assert lib.mw_chunk_attn_cached_plan(ctypes.byref(c), nq, q_len, window, mw.MW_QUEUED_CAUSAL, ws, ctypes.byref(ns),
                                         ctypes.byref(nw)) == mw.MW_OK
    steps = -(-(sink + window * L + nq * q_len) // bk)
    n_tiles = H * -(-nq * q_len // bm)
    longest = -(-steps // ns.value)
    for more in range(ns.value + 1, ns.value + 4):
        if -(-n_tiles * more // 256) == -(-n_tiles * ns.value // 256):
            assert -(-steps // more) > longest * 7 / 8, (ns.value, more, longest)


@pytest.mark.parametrize("mode", [mw.MW_QUEUED_CAUSAL, mw.MW_QUEUED_ISOLATED])
@pytest.mark.parametrize("D", [64, 72, 128])
def test_whole_tiles_only_where_an_unsplit_call_has_them(D, mode):
    """A whole tile of a split plan is what the unsplit call computes for its rows, bit for bit:
    no plan keeps one where the unsplit call splits its keys among wave groups."""
    unsplit_tile = mw.load()["_ZN2mw19cached_unsplit_tileEiiiii"]
    unsplit_tile.restype, unsplit_tile.argtypes = ctypes.c_int, [ctypes.c_int] * 5
    lib, seen = mw.load(), set()
    for H in (1, 3, 6, 8, 12, 16, 24):
        for window in (1, 2, 3):
            for nq, q_len in ((1, 900), (2, 700), (3, 500), (3, 1500), (5, 600), (8, 300)):
                c = new_cache(S=4, B=1, H=H, L=q_len, D=D)
                c.head = window
                ns, nw = ctypes.c_int(), ctypes.c_int()
                ws = lib.mw_chunk_attn_cached_workspace_size(ctypes.byref(c), nq, q_len, window)
                assert lib.mw_chunk_attn_cached_plan(ctypes.byref(c), nq, q_len, window, mode, ws, ctypes.byref(ns),
                                                     ctypes.byref(nw)) == mw.MW_OK
                own = unsplit_tile(D, H, nq * q_len, (window + nq) * q_len, int(mode == mw.MW_QUEUED_CAUSAL or nq == 1))
                seen.add((own, nw.value > 0))
                assert own == 0 or nw.value == 0, (H, window, nq, q_len, ns.value, nw.value)
    assert (1, False) in seen and (2, False) in seen
