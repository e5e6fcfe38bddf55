"""Workspace sizes that callers depend on (no GPU: sizes only)."""
import ctypes

import pytest

from paper_2006_14794_amd import _lib
from paper_2006_14794_amd._lib import SkPaths

FAKE = 0x10000


def need(op, nx, lx, ny, ly, d, lam, flags=0):
    X, Y = SkPaths(FAKE, None, nx, lx, d), SkPaths(FAKE * 2, None, ny, ly, d)
    return _lib.load().sigkernel_workspace_bytes(op, ctypes.byref(X), ctypes.byref(Y), lam, flags)


# Many pairs with short y paths: the x-side parts are one per task, so tasks of
# single pairs would take tens of times the space of runs.  Bound: the plan with runs
# of up to 64 pairs, a quarter of it more and 64 MB.
@pytest.mark.parametrize("lam,d,nx,ny,lx,ly,bytes_", [
    (0, 3, 557, 1841, 1504, 2, 819419904), (2, 13, 630, 316, 2102, 2, 6752291072),
    (2, 2, 2377, 2484, 656, 12, 14332197376), (0, 5, 300, 300, 400, 8, 276540160),
    (1, 4, 64, 1000, 100, 10, 229324800), (1, 5, 256, 256, 200, 20, 840188160)])
def test_gradient_of_many_short_y_paths(lam, d, nx, ny, lx, ly, bytes_):
    """bytes_: the recomputing kernel's plan, runs of up to 64 pairs per task."""
    got = need(_lib.SK_OP_GRAM_BACKWARD, nx, lx, ny, ly, d, lam)
    assert got <= 1.25 * bytes_ + (64 << 20)


# x paths within one wave's rows: the Gram needs its increments and their padding,
# not the layout of the persistent pair kernel (pairs of long paths, in bands)
@pytest.mark.parametrize("lam,d,nx,ny,lx,ly", [(1, 6, 100, 100, 300, 300), (5, 1, 129, 129, 33, 94),
                                               (4, 2, 12, 81, 100, 2700), (0, 8, 128, 128, 256, 256)])
def test_gram_of_one_wave_paths(lam, d, nx, ny, lx, ly):
    rep = 1 << max(lam - 3, 0)
    rows = (nx * (lx - 1) + ny * (ly - 1)) * rep + 4 * 128
    assert need(_lib.SK_OP_GRAM, nx, lx, ny, ly, d, lam) <= rows * ((d + 3) // 4 * 4) * 4 + 4096


# Wide batches (above 16 channels): a run's columns stay within a grid's second
# dimension (65535 tiles of 128), so a wave's slots are at most those of one such run.
@pytest.mark.parametrize("nx,ny,ly", [(16384, 64, 1 << 18), (40000, 60, 1 << 19)])
def test_wide_gram_of_long_streams(nx, ny, ly):
    inc = (nx + ny * (ly - 1) + 4 * 128) * 20 * 4
    slots = (128 * 65535 + 64 + 8) * 64 * 4
    assert need(_lib.SK_OP_GRAM, nx, 2, ny, ly, 17, 0) <= inc + slots + (1 << 20)
