"""A y path with a NaN or an infinity makes the gradients of its own pairs NaN and no
other pair's, whichever pairs share a wave: pairs side by side, runs of the reversing
kernel, runs of the recomputing kernel (short y paths, and tasks handed back).  The
other y paths' gradients are compared with the FP64 oracle's without that path (bar:
conftest.grad_close, 1e-5 of max|g| and 1e-4 relative above 1e-3 max|g|)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
import workloads
from conftest import grad_close
from paper_2006_14794_amd import tuning

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("at", [0, 20, -1])  # first, inner and last point
@pytest.mark.parametrize("lam,lx,ly,d,run", [(0, 30, 40, 3, 0), (1, 17, 31, 9, 0), (2, 17, 31, 4, 0),
                                             (1, 100, 40, 3, 0), (1, 300, 40, 3, 0),
                                             (0, 200, 40, 2, 4), (1, 129, 40, 3, 4),
                                             (1, 300, 40, 3, 5), (1, 30, 22, 3, 5),
                                             (3, 33, 40, 2, 3)])
def test_nonfinite_y_path(lam, lx, ly, d, run, at, value):
    bad = 2
    X = workloads.random_paths(31 + lx, 4, lx, d, std=0.7)
    Y = workloads.random_paths(32 + ly, 6, ly, d, std=0.7)
    keep = [b for b in range(len(Y)) if b != bad]
    dK = np.random.default_rng(lx).normal(size=(len(X), len(Y))).astype(np.float32)
    _, ry = oracle.gram_backward(X.astype(np.float64), Y[keep].astype(np.float64),
                                 dK[:, keep].astype(np.float64), lam)
    Y[bad, at, 0] = value
    Xc, Yc, Dc = (torch.from_numpy(a).cuda() for a in (X, Y, dK))
    try:
        if run:
            tuning.tune_set(tuning.tune_key("gram_backward", Xc, Yc, lam), {"run": run})
        gx, gy = sk.sigkernel_gram_backward(Xc, Yc, Dc, lam)
    finally:
        tuning.tune_clear()
    gy = gy.cpu().numpy()
    assert np.isnan(gx.cpu().numpy()).any(axis=(1, 2)).all()
    assert np.isnan(gy[bad]).any()
    grad_close(gy[keep], ry, f"dY lam{lam} {lx}x{ly} d{d} run {run} at {at}")
