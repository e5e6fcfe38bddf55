"""Lifted sweeps at the edges of their rows per lane, of the packing of several
runs into one wave and of the near-node distances, against the FP64 oracle.  Error
metric and tolerance as in test_gpu_lifted.py: all in double on both sides, so that
only the float32 rounding of the output (6e-8) separates them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
import workloads
from paper_2006_14794_amd import RaggedPaths

pytestmark = pytest.mark.gpu
TOL = 2e-7


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def cuda(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32).cuda()


def f64(a):
    return np.asarray(a, dtype=np.float64)


def worst(got, ref):
    got = got.cpu().numpy().astype(np.float64)
    return float((np.abs(got - ref) / np.maximum(1.0, np.abs(ref))).max())


# coarse rows at the last and first of a height: 16 lanes of 1 .. 16 rows, 64 lanes
ROWS = {0: (1, 16, 17, 48, 49, 65, 97, 129, 161, 257, 385),
        1: (1, 8, 9, 16, 17, 49, 64, 65, 97, 129, 193, 257),
        2: (1, 4, 5, 16, 17, 33, 48, 64, 65, 129),
        3: (1, 2, 3, 8, 9, 17, 33, 65, 97)}


@pytest.mark.parametrize("lam,m", [(l, m) for l in ROWS for m in ROWS[l]])
def test_rows_per_lane_edges(lam, m):
    d = 1 + (m + lam) % 5
    X = workloads.random_paths(10 * m + lam, 3, m + 1, d, std=1.0)
    Y = workloads.random_paths(20 * m + lam, 7, 24 + m % 5, d, std=1.0)
    for scheme in ("explicit", "implicit"):
        got = sk.sigkernel_gram_lifted(cuda(X), cuda(Y), lam, sigma=0.8, scheme=scheme)
        ref = oracle.lifted_rbf_gram(f64(X), f64(Y), lam, 0.8, scheme)
        assert worst(got, ref) <= TOL, scheme


# jumps |e| between the nodes of one lane on both sides of the near-node rule
# |e|^2 log2(e) / (2 sigma^2) <= 16 (|e| = 4.71 sigma), and far beyond it
@pytest.mark.parametrize("jump", [0.0, 1.0, 4.6, 4.8, 100.0, 1e6])
@pytest.mark.parametrize("lam,m,d", [(0, 60, 1), (1, 250, 9), (0, 150, 4), (1, 120, 8)])
def test_jumps_between_nodes(lam, m, d, jump):
    sigma = 1.5
    X = workloads.random_paths(900 + m, 4, m + 1, d, std=1.0)
    Y = workloads.random_paths(950 + m, 5, 41, d, std=1.0)
    X[1, m // 3:, 0] += jump * sigma
    X[2, m // 2, d - 1] -= jump * sigma
    Y[3, 20:, 0] += jump * sigma
    got = sk.sigkernel_gram_lifted(cuda(X), cuda(Y), lam, sigma=sigma)
    ref = oracle.lifted_rbf_gram(f64(X.astype(np.float32)), f64(Y.astype(np.float32)), lam, sigma)
    assert worst(got, ref) <= TOL


@pytest.mark.parametrize("sigma", [1e-30, 1e-3, 1e30])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3e38])
def test_points_far_away(bad, sigma):
    # an infinite point is infinitely far from every finite one (its kernel values
    # are 0), a NaN stays in its pairs
    X = workloads.random_paths(970, 4, 40, 3, std=1.0)
    Y = workloads.random_paths(980, 5, 40, 3, std=1.0)
    X[1, 11, 1] = bad
    Y[2, 20, 2] = bad
    got = sk.sigkernel_gram_lifted(cuda(X), cuda(Y), 1, sigma=sigma).cpu().numpy()
    with np.errstate(all="ignore"):
        ref = oracle.lifted_rbf_gram(f64(X.astype(np.float32)), f64(Y.astype(np.float32)), 1, sigma)
    hit = np.isnan(ref)
    assert np.array_equal(np.isnan(got), hit)
    assert (np.abs(got - ref) / np.maximum(1.0, np.abs(ref)))[~hit].max() <= TOL


@pytest.mark.parametrize("no_diag", [False, True])
@pytest.mark.parametrize("n", [1, 2, 5, 33])
@pytest.mark.parametrize("lam,m", [(0, 20), (1, 44), (2, 12)])
def test_packed_symmetric(lam, m, n, no_diag):
    X = workloads.random_paths(31 * n + m, n, m + 1, 3, std=1.0)
    got = sk.sigkernel_gram_lifted(cuda(X), None, lam, sigma=0.9, symmetric=True, no_diag=no_diag)
    ref = oracle.lifted_rbf_gram(f64(X), f64(X), lam, 0.9)
    if no_diag:
        np.fill_diagonal(ref, 0.0)
    assert worst(got, ref) <= TOL
    assert torch.equal(got, got.T)


def test_packed_ragged():
    # lengths 1 .. 30 in one packed launch: pairs without cells, uneven widths
    lx, ly = [1, 30, 7, 2, 19], [3, 30, 1, 12, 25, 9, 2]
    xs = [workloads.random_paths(700 + i, 1, L, 4, std=1.0)[0] for i, L in enumerate(lx)]
    ys = [workloads.random_paths(800 + i, 1, L, 4, std=1.0)[0] for i, L in enumerate(ly)]
    X, Y = RaggedPaths.from_list(xs, "cuda"), RaggedPaths.from_list(ys, "cuda")
    got = sk.sigkernel_gram_lifted(X, Y, 1, sigma=0.7).cpu().numpy()
    for i, x in enumerate(xs):
        for j, y in enumerate(ys):
            ref = oracle.lifted_rbf_pairs(f64(x)[None], f64(y)[None], 1, 0.7)[0]
            assert abs(got[i, j] - ref) <= TOL * max(1.0, abs(ref)), (i, j)
