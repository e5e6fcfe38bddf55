"""Gradients of runs of pairs that one wave sweeps back to back, with a pair of a
large kernel (near 1e7 and 1e12) in second, middle and last place of a run: the
rebuilt forward nodes of every pair of a run have to be checked, not those of its
first alone.  Segments per checkpoint 1, 2 and 4, one and two bands, runs set by
tuning and by the built-in rule; against the FP64 oracle's discrete adjoint (bar:
conftest.grad_close, 1e-5 of max|g| and 1e-4 relative above 1e-3 max|g|)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
from conftest import grad_close
from paper_2006_14794_amd import tuning

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def cuda(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32).cuda()


def lines(rng, n, length, large, scale):
    """n nearly straight paths of R^2; those listed in `large` scaled by `scale`."""
    s = np.ones(n)
    s[list(large)] = scale
    t = np.linspace(0.0, 1.0, length)[None, :, None] * np.array([1.0, 0.5])
    return (s[:, None, None] * t + 0.05 * rng.normal(size=(n, length, 2))).astype(np.float32)


def check(X, Y, lam, name, run=0):
    dK = np.random.default_rng(5).normal(size=(len(X), len(Y))).astype(np.float32)
    Xc, Yc, Dc = cuda(X), cuda(Y), cuda(dK)
    try:
        if run:
            tuning.tune_set(tuning.tune_key("gram_backward", Xc, Yc, lam), {"run": run})
        gx, gy = sk.sigkernel_gram_backward(Xc, Yc, Dc, lam)
        gx1, _ = sk.sigkernel_gram_backward(Xc, Yc, Dc, lam, need_y=False)
    finally:
        tuning.tune_clear()
    rx, ry = oracle.gram_backward(X.astype(np.float64), Y.astype(np.float64),
                                  dK.astype(np.float64), lam)
    grad_close(gx.cpu().numpy(), rx, f"dX {name}")
    grad_close(gy.cpu().numpy(), ry, f"dY {name}")
    grad_close(gx1.cpu().numpy(), rx, f"dX alone {name}")


# scale of the large paths: <x_T - x_0, y_T - y_0> = 1.25 scale^2, so kernels of
# about I0(2 sqrt(1.25) scale)
@pytest.mark.parametrize("scale", [8.4, 13.6])
@pytest.mark.parametrize("place", ["second", "middle", "last"])
@pytest.mark.parametrize("lam,lx,ly,run", [(0, 200, 40, 5), (0, 200, 40, 15), (0, 200, 40, 30),
                                           (1, 129, 40, 4), (1, 129, 40, 10), (1, 129, 40, 20),
                                           (1, 300, 40, 20), (1, 129, 80, 12), (2, 65, 30, 8),
                                           (2, 65, 30, 20), (3, 33, 12, 4), (3, 33, 12, 24)])
def test_large_kernel_inside_a_run(lam, lx, ly, run, place, scale):
    rng = np.random.default_rng(lx + run)
    b = {"second": 1, "middle": run // 2, "last": run - 1}[place]
    X = lines(rng, 3, lx, [1], scale)
    Y = lines(rng, run + 3, ly, [b], scale)
    check(X, Y, lam, f"lam{lam} {lx}x{ly} run {run} {place} {scale}", run)


@pytest.mark.parametrize("lam,lx,ly", [(0, 200, 40), (1, 129, 40)])
def test_built_in_runs(lam, lx, ly):
    # 6144 pairs: runs of three
    rng = np.random.default_rng(lx)
    X = lines(rng, 64, lx, [3], 8.4)
    Y = lines(rng, 96, ly, [1, 5, 40, 94], 8.4)
    check(X, Y, lam, f"built-in runs lam{lam} {lx}x{ly}")


@pytest.mark.parametrize("scale", [8.4, 20.0])
@pytest.mark.parametrize("lam,n,lx,ly", [(0, 30, 60, 60), (1, 12, 129, 40), (1, 70, 129, 40),
                                         (1, 8, 300, 200)])
def test_values_of_handed_back_tasks(lam, n, lx, ly, scale):
    # the MMD's blocks take their values from the gradient's forward pass, which a
    # handed-back task leaves where it meets the large nodes
    rng = np.random.default_rng(lx + n)
    X, Y = lines(rng, n, lx, [1, n - 1], scale), lines(rng, n + 2, ly, [2], scale)
    val, _ = sk.sigkernel_mmd2(cuda(X), cuda(Y), lam, grad=True)
    X, Y = X.astype(np.float64), Y.astype(np.float64)
    Kxx, Kyy, Kxy = oracle.gram(X, X, lam), oracle.gram(Y, Y, lam), oracle.gram(X, Y, lam)
    np.fill_diagonal(Kxx, 0.0)
    np.fill_diagonal(Kyy, 0.0)
    # the values are float32: 6e-8 of each term
    size = np.abs(Kxx).sum() / (n * (n - 1)) + np.abs(Kyy).sum() / ((n + 2) * (n + 1)) \
        + 2.0 * np.abs(Kxy).mean()
    assert abs(float(val) - oracle.mmd2_unbiased(Kxx, Kyy, Kxy)) <= 2e-7 * size
