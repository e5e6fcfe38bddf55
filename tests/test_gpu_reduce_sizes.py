"""Reduced measures at the edges of the kernels' sizes (one wave, one workgroup
with K in registers, K read from memory) against the FP64 oracle.  Each
iteration sums n products in double, so iterates agree to n eps times their
scale: 1e-10 (as tests/test_gpu_reduce.py)."""
import numpy as np
import pytest
import torch

import paper_2006_14794_amd as sk
from oracle import reduced_measure as rm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def spd(seed, n, cond=8.0):
    rng = np.random.default_rng(seed)
    Q, _ = np.linalg.qr(rng.normal(size=(n, n)))
    return ((Q * np.geomspace(1.0, cond, n)) @ Q.T).astype(np.float32)


SIZES = [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256,
         257, 263, 400]


@pytest.mark.parametrize("n", SIZES)
def test_iterates_losses_and_step(n):
    # K is not symmetric: a swapped index shows
    K = spd(60 + n, n) + 0.01 * np.random.default_rng(n).normal(size=(n, n)).astype(np.float32)
    K64 = K.astype(np.float64)
    rng = np.random.default_rng(900 + n)
    alpha = rng.uniform(0.5, 1.5, size=n).astype(np.float32)
    alpha /= np.float32(n)
    lam = 0.3 / n
    for iters in (0, 1, 60):
        beta, loss, used = sk.reduced_measure(torch.from_numpy(K).cuda(), lam, iters,
                                              alpha=torch.from_numpy(alpha).cuda())
        a64, step = alpha.astype(np.float64), used.item()
        b, ref_loss = a64.copy(), []
        for it in range(iters + 1):
            d = b - a64
            g = K64 @ d
            ref_loss.append(d @ g + lam * np.abs(b).sum())
            if it < iters:
                z = b - 2.0 * step * g
                b = np.sign(z) * np.maximum(np.abs(z) - step * lam, 0.0)
        assert np.abs(beta.cpu().numpy() - b).max() <= 1e-10
        assert np.abs(loss.cpu().numpy() - ref_loss).max() <= 1e-10 * np.abs(ref_loss).max()
    v = 1.0 + 1e-3 * (np.arange(n) % 7)
    for _ in range(200):
        w = K64 @ v
        rho = np.sqrt(w @ w)
        v = w / rho
    assert abs(step - 1.0 / (2.1 * rho)) <= 1e-12 * step


@pytest.mark.parametrize("n", [5, 32, 40, 64, 100, 150, 250, 300])
def test_support_search(n):
    K = spd(70 + n, n)
    K64 = K.astype(np.float64)
    alpha = np.random.default_rng(n).permutation(np.linspace(0.2, 1.8, n)).astype(np.float32) / n
    support = max(1, n // 4)
    beta, lam, used = sk.reduced_measure_support(torch.from_numpy(K).cuda(), support, 400, 30,
                                                 alpha=torch.from_numpy(alpha).cuda())
    b, lam = beta.cpu().numpy(), lam.item()
    assert np.count_nonzero(b) == support
    # the weights minimise eq. (min_lasso) at the penalty found (KKT)
    g = rm.gradient(K64, alpha.astype(np.float64), b)
    nz = b != 0
    assert np.abs(g[nz] + lam * np.sign(b[nz])).max() <= 1e-8
    assert np.all(np.abs(g[~nz]) <= lam + 1e-8)


@pytest.mark.parametrize("n", [20, 50, 100, 220, 300])
def test_nan_entries_threshold_to_zero(n):
    # a NaN in K makes every gradient of its row NaN, and a NaN thresholds to 0
    K = spd(80 + n, n)
    K[n // 2, 3] = np.nan
    beta, _, _ = sk.reduced_measure(torch.from_numpy(K).cuda(), 1e-3, 3, step=0.01)
    b = beta.cpu().numpy()
    assert b[n // 2] == 0.0 and np.isfinite(b).all()
