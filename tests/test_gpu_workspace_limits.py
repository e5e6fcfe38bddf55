"""Calls whose pair workspace has a choice of layouts: the Gram without a caller
workspace takes a problem whenever one of them fits its 64 MiB, a pair call takes a
workspace that holds any of them, and the values are those of the call with all the
space it asks for, bit for bit (the layouts order the same fine cells differently)."""
import ctypes

import pytest
import torch

import paper_2006_14794_amd as sk
import workloads
from paper_2006_14794_amd import _lib, tuning
from paper_2006_14794_amd._lib import SkPaths

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def batch(seed, n, length, d):
    return torch.from_numpy(workloads.random_paths(seed, n, length, d, std=0.7)).cuda()


def desc(t):
    return SkPaths(t.data_ptr(), None, t.shape[0], t.shape[1], t.shape[2])


def stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


# x paths in one wave's rows, and taller ones (several bands); all of them fit 64 MiB
# with bands of the largest height
@pytest.mark.parametrize("nx,ny,lx,ly,d,lam", [(2, 227, 290, 2974, 5, 0), (3, 78, 443, 455, 2, 3),
                                               (43, 1, 1860, 430, 1, 3), (1, 1, 2345, 2345, 1, 5),
                                               (1, 23, 1970, 24, 12, 5), (6, 61, 107, 3543, 12, 3)])
def test_gram_without_a_caller_workspace(nx, ny, lx, ly, d, lam):
    X, Y = batch(lx, nx, lx, d), batch(ly + 1, ny, ly, d)
    K = torch.full((nx, ny), float("nan"), device="cuda")
    st = _lib.load().sigkernel_gram_noalloc(ctypes.byref(desc(X)), ctypes.byref(desc(Y)), lam, 0,
                                            K.data_ptr(), stream())
    assert st == _lib.SK_OK, sk.status_string(st)
    assert torch.equal(K, sk.sigkernel_gram(X, Y, lam))


@pytest.mark.parametrize("n,lx,ly,d,lam,mib", [(78, 1815, 2373, 11, 1, 44), (27, 52, 3463, 2, 4, 16),
                                               (64, 275, 85, 12, 5, 42)])
def test_pairs_in_a_small_workspace(n, lx, ly, d, lam, mib):
    X, Y = batch(lx, n, lx, d), batch(ly + 1, n, ly, d)
    ref = sk.sigkernel_pair(X, Y, lam)
    lib = _lib.load()
    full = lib.sigkernel_workspace_bytes(_lib.SK_OP_PAIR, ctypes.byref(desc(X)),
                                         ctypes.byref(desc(Y)), lam, 0)
    assert full > mib << 20
    ws = torch.empty(mib << 20, dtype=torch.uint8, device="cuda")
    out = torch.full((n,), float("nan"), device="cuda")
    for byte in (0x00, 0xFF):
        ws.fill_(byte)
        st = lib.sigkernel_pair(ctypes.byref(desc(X)), ctypes.byref(desc(Y)), lam, 0,
                                out.data_ptr(), ws.data_ptr(), ws.numel(), stream())
        assert st == _lib.SK_OK, sk.status_string(st)
        assert torch.equal(out, ref)
    # one wave per pair by tuning: no bands, the same values
    try:
        tuning.tune_set(tuning.tune_key("pair", X, Y, lam), {"pair_bands": 1})
        assert torch.equal(sk.sigkernel_pair(X, Y, lam), ref)
    finally:
        tuning.tune_clear()
    st = lib.sigkernel_pair(ctypes.byref(desc(X)), ctypes.byref(desc(Y)), lam, 0, out.data_ptr(),
                            ws.data_ptr(), 4096, stream())
    assert st == _lib.SK_ERR_WORKSPACE
