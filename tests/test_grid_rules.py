"""Which configuration a training grid takes (host side, no GPU): the measured points on both sides
of each line, and that the GPU tests reach every configuration."""
import ctypes

import pytest

import paper_2608_01127_amd as mw
import test_gpu_grid_shapes as shapes

SPARSE, SMALL, MID, FULL, LARGE = range(5)
WIDE, PAIRS, WIDE3, QUADS = 0, 2, 3, 4


class Choice(ctypes.Structure):  # mw::FwdChoice
    _fields_ = [("bm", ctypes.c_int), ("bk", ctypes.c_int), ("wg_per_cu", ctypes.c_int),
                ("lone_rate", ctypes.c_double), ("part_rate", ctypes.c_double)]


# (head width, queued rows): rows and keys of the cached tile, and workgroups resident per CU
CHOICES = [(64, 64, 64, 64, 2), (64, 65, 128, 64, 4), (64, 257, 256, 64, 2), (72, 64, 64, 64, 1), (72, 65, 128, 64, 3),
           (72, 257, 128, 64, 3), (128, 64, 64, 64, 1), (128, 65, 128, 128, 1), (128, 513, 256, 64, 1)]


def check_choice(D, Tq, bm, bk, wgs):
    fn = mw.load()["_ZN2mw10fwd_choiceEii"]  # mw::fwd_choice(int, int)
    fn.restype, fn.argtypes = Choice, [ctypes.c_int] * 2
    c = fn(D, Tq)
    assert (c.bm, c.bk, c.wg_per_cu) == (bm, bk, wgs)


@pytest.mark.parametrize("D,Tq,bm,bk,wgs", CHOICES)
def test_residency_assumed_without_a_device(D, Tq, bm, bk, wgs):
    check_choice(D, Tq, bm, bk, wgs)


@pytest.mark.gpu
@pytest.mark.parametrize("D,Tq,bm,bk,wgs", CHOICES)
def test_residency_on_the_device(mw, D, Tq, bm, bk, wgs):
    """The runtime's occupancy of the built kernels is what is assumed where no device is present, so
    that plans and workspace sizes made there hold here."""
    check_choice(D, Tq, bm, bk, wgs)


def rule(symbol, *args):
    fn = mw.load()[symbol]  # loaded in the tests only: on a GPU, torch comes first
    fn.restype, fn.argtypes = ctypes.c_int, [ctypes.c_int] * len(args)
    return fn(*args)


def fwd_fill(D, BH, T):
    return rule("_ZN2mw17training_fwd_fillEiii", D, BH, T)  # mw::training_fwd_fill(int, int, int)


def bwd_grid(D, BH, T):
    return rule("_ZN2mw17training_bwd_gridEiii", D, BH, T)  # mw::training_bwd_grid(int, int, int)


@pytest.mark.parametrize("D,BH,T,fill", [
    (64, 16, 42240, LARGE), (64, 16, 19200, LARGE), (64, 7, 42240, LARGE), (64, 96, 4800, LARGE),
    (64, 24, 10560, FULL), (64, 8, 19200, FULL), (64, 4, 42240, FULL), (72, 16, 19200, FULL), (128, 16, 42240, FULL),
    (128, 16, 4800, MID), (72, 16, 3000, SMALL), (128, 144, 200, MID), (128, 96, 330, MID), (128, 64, 512, SMALL),
    (128, 36, 1000, SMALL), (128, 12, 2800, SMALL), (72, 112, 512, FULL), (72, 64, 1000, FULL), (72, 56, 1000, SMALL), (64, 4, 4000, SPARSE)])
def test_forward_lines(D, BH, T, fill):
    assert fwd_fill(D, BH, T) == fill


# (heads, tokens) where one configuration measured at least 4% ahead of the next
@pytest.mark.parametrize("D,BH,T,grid", [
    # short sequences in one round of 128-row tiles: two groups lose
    (64, 65, 512, WIDE), (64, 80, 330, WIDE), (72, 93, 330, WIDE), (72, 120, 200, WIDE), (128, 120, 200, WIDE),
    (128, 93, 330, WIDE), (128, 68, 512, WIDE), (64, 40, 512, PAIRS), (72, 40, 512, PAIRS), (128, 60, 512, PAIRS),
    (64, 12, 2400, PAIRS), (64, 32, 1000, PAIRS), (72, 24, 1500, WIDE), (128, 18, 2000, PAIRS), (72, 8, 4096, PAIRS),
    # four groups
    (64, 5, 4096, PAIRS), (72, 5, 4096, PAIRS), (64, 4, 5000, PAIRS), (64, 12, 1024, PAIRS), (128, 12, 1024, PAIRS),
    (64, 1, 24000, QUADS), (128, 1, 24000, QUADS), (64, 4, 2500, QUADS), (64, 8, 1000, QUADS), (128, 4, 4096, QUADS), (128, 2, 12000, QUADS),
    (64, 1, 30000, PAIRS), (128, 2, 16000, PAIRS), (64, 2, 256, PAIRS), (128, 1, 400, PAIRS), (72, 8, 512, PAIRS),
    # three waves per SIMD
    (64, 8, 7200, WIDE), (64, 1, 60000, WIDE), (64, 12, 5120, WIDE), (64, 4, 18000, WIDE), (64, 6, 13000, WIDE3),
    (64, 24, 2500, WIDE3), (64, 48, 1280, WIDE3), (64, 24, 10560, WIDE3)])
def test_backward_lines(D, BH, T, grid):
    assert bwd_grid(D, BH, T) == grid


def gpu_shapes():
    for fn in (shapes.test_work_order, shapes.test_forward_tiles):
        for B, H, T, D, _ in fn.pytestmark[0].args[1]:
            yield D, B * H, T


def test_gpu_shapes_reach_every_configuration():
    reached = {(D, bwd_grid(D, BH, T)) for D, BH, T in gpu_shapes()}
    assert reached == {(D, g) for D in (64, 72, 128) for g in (WIDE, PAIRS, QUADS)} | {(64, WIDE3)}
    reached = {(D, fwd_fill(D, BH, T)) for D, BH, T in gpu_shapes()}
    # (FULL at D = 128: the training shapes of test_gpu_train)
    assert reached == {(D, f) for D in (64, 72, 128) for f in (SPARSE, SMALL)} | {(64, FULL), (64, LARGE), (72, FULL),
                                                                               (128, MID)}
