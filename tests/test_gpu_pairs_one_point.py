"""Pairs of equal lengths with one-point paths on both sides or on one: every value is
the boundary value 1, from fewer and from more pairs than wave slots, whatever the
workspace holds before the call (no batch has increments whose launch could clear the
pair queue's head by the way), and nothing is written outside the output."""
import ctypes

import pytest
import torch

import paper_2006_14794_amd as sk
from paper_2006_14794_amd import _lib
from paper_2006_14794_amd._lib import SkPaths

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


@pytest.mark.parametrize("byte", [0x00, 0x7F, 0xFF])
@pytest.mark.parametrize("n", [1, 3, 4097, 9000])
@pytest.mark.parametrize("lx,ly", [(1, 1), (1, 6), (6, 1)])
def test_every_value_is_one(lx, ly, n, byte):
    lib = _lib.load()
    for d in (3, 4):  # both increment kernels
        x = torch.ones(n, lx, d, device="cuda")
        y = torch.ones(n, ly, d, device="cuda")
        X, Y = SkPaths(x.data_ptr(), None, n, lx, d), SkPaths(y.data_ptr(), None, n, ly, d)
        need = lib.sigkernel_workspace_bytes(_lib.SK_OP_PAIR, ctypes.byref(X), ctypes.byref(Y), 1,
                                             0)
        ws = torch.full((need,), byte, dtype=torch.uint8, device="cuda")
        guard = 4096
        out = torch.full((n + 2 * guard,), 7.0, device="cuda")
        st = lib.sigkernel_pair(ctypes.byref(X), ctypes.byref(Y), 1, 0,
                                out.data_ptr() + 4 * guard, ws.data_ptr(), need,
                                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == _lib.SK_OK, sk.status_string(st)
        assert torch.all(out[guard:guard + n] == 1.0)
        assert torch.all(out[:guard] == 7.0) and torch.all(out[guard + n:] == 7.0)
