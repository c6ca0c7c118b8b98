"""Training grids whose work order or tile configuration depends on the number of heads and
tiles: parity of every output with the fp64 oracle, so that a tile taken twice or not at all, or
a wrong edge, shows as garbage rows."""
import pytest

import oracle
from helpers import assert_close, f64, to_f64
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


# Batch x heads of every residue class of the work order (1, 2, 4 or 8 groups of XCDs), with tile
# counts that leave a partial last row of workgroup ids
@pytest.mark.parametrize("B,H,T,D,L", [(1, 1, 900, 128, 200), (1, 3, 500, 64, 100), (3, 5, 300, 72, 77),
                                       (2, 3, 650, 128, 130), (1, 10, 200, 64, 64), (1, 12, 300, 128, 100),
                                       (2, 10, 150, 72, 50), (1, 24, 140, 64, 30)])
def test_work_order(mw, B, H, T, D, L):
    check(mw, B, H, T, D, L)
