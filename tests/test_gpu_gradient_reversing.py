"""Gradients on both sides of every choice of the reversing gradient kernel
(rows per lane, pairs per wave, bands, segments, runs) and of its hand-back to
the recomputing kernel, against the FP64 oracle's discrete adjoint (bar:
conftest.grad_close, 1e-5 of max|g| and 1e-4 relative above 1e-3 max|g|)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
import workloads
from conftest import grad_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def cuda(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32).cuda()


def check(X, Y, lam, name, seed=0):
    dK = np.random.default_rng(seed).normal(size=(len(X), len(Y))).astype(np.float32)
    gx, gy = sk.sigkernel_gram_backward(cuda(X), cuda(Y), cuda(dK), lam)
    rx, ry = oracle.gram_backward(X.astype(np.float64), Y.astype(np.float64),
                                  dK.astype(np.float64), lam)
    grad_close(gx.cpu().numpy(), rx, f"dX {name}")
    grad_close(gy.cpu().numpy(), ry, f"dY {name}")
    gx1, gy1 = sk.sigkernel_gram_backward(cuda(X), cuda(Y), cuda(dK), lam, need_y=False)
    assert gy1 is None
    grad_close(gx1.cpu().numpy(), rx, f"dX alone {name}")


# fine rows at the edges of 16, 32 and 64 lanes of 4 and 8 rows, and of two bands
EDGES = [(0, 65, 5), (0, 66, 40), (0, 129, 33), (0, 130, 34), (0, 257, 20), (0, 514, 70),
         (1, 33, 24), (1, 34, 25), (1, 65, 26), (1, 66, 9), (1, 129, 50), (1, 130, 49),
         (1, 257, 98), (1, 258, 20), (2, 17, 17), (2, 18, 16), (2, 33, 40), (2, 129, 18),
         (2, 130, 64), (3, 9, 9), (3, 10, 30), (3, 33, 8), (3, 34, 65)]


@pytest.mark.parametrize("d", [1, 4, 7])
@pytest.mark.parametrize("lam,lx,ly", EDGES)
def test_edges_of_groups_bands_and_segments(lam, lx, ly, d):
    X = workloads.random_paths(1000 + lx, 2, lx, d, std=0.7)
    Y = workloads.random_paths(2000 + ly, 5, ly, d, std=0.7)
    check(X, Y, lam, f"lam{lam} {lx}x{ly} d{d}")


@pytest.mark.parametrize("no_diag", [False, True])
@pytest.mark.parametrize("lam,lx", [(0, 20), (1, 33), (1, 60), (2, 17), (3, 9)])
def test_symmetric_groups(lam, lx, no_diag):
    # packed waves around the diagonal: groups above, on and below it
    X = workloads.random_paths(3000 + lx, 7, lx, 3, std=0.7)
    dK = np.random.default_rng(lx).normal(size=(7, 7)).astype(np.float32)
    gx, _ = sk.sigkernel_gram_backward(cuda(X), None, cuda(dK), lam, symmetric=True,
                                       no_diag=no_diag)
    w = dK.astype(np.float64)
    if no_diag:
        np.fill_diagonal(w, 0.0)
    rx, ry = oracle.gram_backward(X.astype(np.float64), X.astype(np.float64), w, lam)
    grad_close(gx.cpu().numpy(), rx + ry, f"dX symmetric lam{lam} {lx} no_diag={no_diag}")


@pytest.mark.parametrize("lam,lx,ly", [(0, 30, 30), (0, 300, 40), (1, 20, 20), (1, 50, 80),
                                       (1, 300, 200), (2, 40, 40), (3, 12, 30)])
def test_huge_kernels_are_handed_back(lam, lx, ly):
    # nearly parallel straight paths, <x_T - x_0, y_T - y_0> about 700: kernels
    # near exp(2 sqrt(700)) / 13, about 1e21, on which rebuilding the forward
    # nodes backwards loses every digit (rounding grows like the square of the
    # kernel between two checkpoints), one ordinary pair among them
    rng = np.random.default_rng(lx)
    def line(n, scale):
        p = np.linspace(0.0, scale, n)[:, None] * np.array([[1.0, 0.5]])
        return p + 0.05 * rng.normal(size=(n, 2))
    X = np.stack([line(lx, 25.0), line(lx, 1.0)]).astype(np.float32)
    Y = np.stack([line(ly, 25.0), line(ly, 1.0), line(ly, 22.0)]).astype(np.float32)
    check(X, Y, lam, f"huge lam{lam} {lx}x{ly}")
