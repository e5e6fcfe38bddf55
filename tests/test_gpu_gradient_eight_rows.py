"""Gradients with eight rows per lane and one wave per SIMD (more increments per
lane than two waves leave room for): one band and two, pairs side by side in a
wave, both sides of the choice between four and eight rows, against the FP64
oracle's discrete adjoint (bar: conftest.grad_close, 1e-5 of max|g| and 1e-4
relative above 1e-3 max|g|)."""
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


@pytest.mark.parametrize("lam,lx,ly,d", [
    (0, 129, 40, 3), (0, 257, 33, 3), (0, 513, 40, 3), (0, 514, 30, 3),
    (1, 65, 26, 5), (1, 129, 50, 6), (1, 257, 98, 5), (1, 258, 30, 6), (1, 400, 60, 5),
    (2, 33, 40, 7), (2, 65, 30, 8), (2, 129, 20, 10), (2, 130, 64, 12), (2, 140, 20, 12)])
def test_eight_rows(lam, lx, ly, d):
    X = workloads.random_paths(4000 + lx, 2, lx, d, std=0.7)
    Y = workloads.random_paths(5000 + ly, 5, ly, d, std=0.7)
    dK = np.random.default_rng(lx).normal(size=(2, 5)).astype(np.float32)
    gx, gy = sk.sigkernel_gram_backward(cuda(X), cuda(Y), cuda(dK), lam)
    rx, ry = oracle.gram_backward(X.astype(np.float64), Y.astype(np.float64),
                                  dK.astype(np.float64), lam)
    grad_close(gx.cpu().numpy(), rx, "dX")
    grad_close(gy.cpu().numpy(), ry, "dY")
    gx1, _ = sk.sigkernel_gram_backward(cuda(X), cuda(Y), cuda(dK), lam, need_y=False)
    grad_close(gx1.cpu().numpy(), rx, "dX alone")
