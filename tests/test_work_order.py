"""The training grids' work order (host side, no GPU): every tile once, heaviest tiles first, and
whole heads on one XCD (workgroup ids are dealt to the 8 XCDs round-robin)."""
import ctypes

import pytest

import paper_2608_01127_amd as mw


def order(BH, ntiles):
    fn = mw.load()["_ZN2mw18training_work_itemEiiRiS0_"]  # mw::training_work_item(int, int, int&, int&)
    fn.restype, fn.argtypes = None, [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    bh, rank = ctypes.c_int(), ctypes.c_int()
    items = []
    for bid in range(BH * ntiles):
        fn(bid, BH, ctypes.addressof(bh), ctypes.addressof(rank))
        items.append((bh.value, rank.value))
    return items


@pytest.mark.parametrize("BH", [1, 2, 3, 4, 6, 7, 8, 9, 10, 12, 13, 15, 16, 20, 24, 45, 63, 99])
@pytest.mark.parametrize("ntiles", [1, 2, 5, 13])
def test_work_order(BH, ntiles):
    items = order(BH, ntiles)
    assert sorted(items) == [(b, r) for b in range(BH) for r in range(ntiles)]  # every tile once
    assert [r for _, r in items] == [r for r in range(ntiles) for _ in range(BH)]  # heaviest first
    xcds = {}
    for bid, (bh, _) in enumerate(items):
        xcds.setdefault(bh, set()).add(bid % 8)
    lead = BH % 8
    for bh, x in xcds.items():
        assert len(x) <= (8 // min(lead & -lead, 8) if bh < lead else 1), (bh, x)
