"""Forward Gram sweeps at the edges of their rows per lane and of the packing
of several runs into one wave, against the FP64 oracle.  Error metric and
tolerance as in test_gpu_parity.py: |k_gpu - k_ref| / max(1, |k_ref|) <= 1e-6."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
import workloads
from paper_2006_14794_amd import RaggedPaths

pytestmark = pytest.mark.gpu
TOL = 1e-6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def cuda(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32).cuda()


def worst(got, ref):
    got = got.cpu().numpy().astype(np.float64)
    return float((np.abs(got - ref) / np.maximum(1.0, np.abs(ref))).max())


# coarse rows at the last and first of a height: 16 lanes of 1 .. 16 rows, 64
# lanes of 2 .. 32
ROWS = {0: (1, 16, 17, 33, 48, 49, 65, 81, 97, 129, 160, 161, 193, 257, 320, 385, 641),
        1: (1, 8, 9, 16, 17, 48, 49, 64, 65, 96, 97, 129, 193, 257, 384, 513),
        2: (1, 5, 8, 9, 16, 17, 32, 33, 48, 64, 65, 192, 257, 385),
        3: (1, 2, 3, 8, 9, 16, 17, 32, 33, 64, 65, 129, 193)}


@pytest.mark.parametrize("lam,m", [(l, m) for l in ROWS for m in ROWS[l]])
def test_rows_per_lane_edges(lam, m):
    d = 1 + (m + lam) % 6
    X = workloads.random_paths(10 * m + lam, 3, m + 1, d)
    Y = workloads.random_paths(20 * m + lam, 7, 24 + m % 5, d)
    for scheme, ref in (("explicit", oracle.gram), ("implicit", None)):
        got = sk.sigkernel_gram(cuda(X), cuda(Y), lam, scheme=scheme)
        if ref is None:
            r = oracle.pairs_implicit([x.astype(np.float64) for x in X for _ in Y],
                                      [y.astype(np.float64) for _ in X for y in Y], lam)
            r = np.asarray(r).reshape(3, 7)
        else:
            r = ref(X.astype(np.float64), Y.astype(np.float64), lam)
        assert worst(got, r) <= TOL, scheme


@pytest.mark.parametrize("no_diag", [False, True])
@pytest.mark.parametrize("n", [1, 2, 5, 33])
@pytest.mark.parametrize("lam,m", [(0, 20), (1, 44), (2, 12)])
def test_packed_symmetric(lam, m, n, no_diag):
    X = workloads.random_paths(31 * n + m, n, m + 1, 3)
    got = sk.sigkernel_gram(cuda(X), None, lam, symmetric=True, no_diag=no_diag)
    ref = oracle.gram(X.astype(np.float64), X.astype(np.float64), lam)
    if no_diag:
        np.fill_diagonal(ref, 0.0)
    assert worst(got, ref) <= TOL
    assert torch.equal(got, got.T)


def test_packed_ragged_and_broken_paths():
    # lengths 1 .. 30 in one packed launch: pairs without cells, uneven widths
    # side by side in a wave, and one path with a NaN point, which stays in its pairs
    lx, ly = [1, 30, 7, 2, 19], [3, 30, 1, 12, 25, 9, 2]
    xs = [workloads.random_paths(700 + i, 1, L, 4)[0] for i, L in enumerate(lx)]
    ys = [workloads.random_paths(800 + i, 1, L, 4)[0] for i, L in enumerate(ly)]
    ys[4][11, 2] = np.nan
    X, Y = RaggedPaths.from_list(xs, "cuda"), RaggedPaths.from_list(ys, "cuda")
    got = sk.sigkernel_gram(X, Y, 1).cpu().numpy()
    for i, x in enumerate(xs):
        for j, y in enumerate(ys):
            if j == 4 and lx[i] > 1:
                assert np.isnan(got[i, j])
                continue
            ref = 1.0 if min(lx[i], ly[j]) == 1 else oracle.solve(x.astype(np.float64),
                                                                  y.astype(np.float64), 1)
            assert abs(got[i, j] - ref) <= TOL * max(1.0, abs(ref)), (i, j)
