"""Coefficient tiles of wide batches (coef.hip) at their edges: channels around
the register groups, rows around the 32-row tiles and the strips' alignment,
column streams whose 128-column tiles hold several runs or cut pairs, symmetric
Grams, every input precision; against the FP64 oracle with the bound of
test_gpu_wide.py (float32 sums of d products)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
import workloads
from paper_2006_14794_amd import RaggedPaths

pytestmark = pytest.mark.gpu


def tol(d):
    return 1e-6 * max(1.0, (d / 16.0) ** 0.5)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def f64(a):
    return np.asarray(a, dtype=np.float64)


def worst(got, ref):
    return float((np.abs(f64(got) - ref) / np.maximum(1.0, np.abs(ref))).max())


# (order, x points, y points, y paths, channels)
CASES = [(0, 2, 2, 5, 17), (0, 34, 40, 7, 20), (0, 100, 130, 3, 31), (0, 257, 20, 9, 32),
         (0, 300, 65, 4, 33), (1, 18, 6, 60, 40), (1, 49, 33, 11, 63), (1, 98, 129, 3, 64),
         (1, 130, 128, 2, 65), (1, 194, 7, 40, 24), (2, 10, 12, 30, 128), (2, 66, 50, 5, 129),
         (2, 129, 64, 3, 48), (3, 3, 30, 9, 20), (3, 17, 90, 4, 36), (3, 70, 40, 3, 72)]


@pytest.mark.parametrize("lam,lx,ly,ny,d", CASES)
def test_gram(lam, lx, ly, ny, d):
    X = workloads.random_paths(7000 + lx, 4, lx, d)
    Y = workloads.random_paths(7100 + ly, ny, ly, d)
    ref = oracle.gram(f64(X), f64(Y), lam)
    assert worst(sk.sigkernel_gram(cuda(X), cuda(Y), lam).cpu().numpy(), ref) <= tol(d)
    got = sk.sigkernel_gram(cuda(X), cuda(Y), lam, scheme="implicit").cpu().numpy()
    imp = oracle.pairs_implicit([f64(x) for x in X for _ in Y], [f64(y) for _ in X for y in Y], lam)
    assert worst(got, np.asarray(imp).reshape(4, ny)) <= tol(d)


@pytest.mark.parametrize("no_diag", [False, True])
@pytest.mark.parametrize("n,lx,lam,d", [(1, 20, 1, 18), (2, 40, 0, 33), (23, 12, 1, 70),
                                        (40, 60, 1, 20)])
def test_symmetric(n, lx, lam, d, no_diag):
    X = workloads.random_paths(7200 + n, n, lx, d)
    ref = oracle.gram(f64(X), f64(X), lam)
    if no_diag:
        np.fill_diagonal(ref, 0.0)
    got = sk.sigkernel_gram(cuda(X), None, lam, symmetric=True, no_diag=no_diag).cpu().numpy()
    assert np.array_equal(got, got.T)
    assert worst(got, ref) <= tol(d)


@pytest.mark.parametrize("precision", ["bf16", "f16"])
@pytest.mark.parametrize("d", [17, 24, 40, 72])
def test_sixteen_bit_increments(precision, d):
    X = workloads.random_paths(7300 + d, 3, 40, d)
    Y = workloads.random_paths(7400 + d, 6, 50, d)
    dt = torch.bfloat16 if precision == "bf16" else torch.float16

    def rounded(P):  # paths whose exact increments are the rounded float32 ones
        inc = torch.from_numpy(np.diff(P, axis=1)).to(dt).double().numpy()
        return np.concatenate([np.zeros_like(inc[:, :1]), np.cumsum(inc, axis=1)], axis=1)

    ref = oracle.gram(rounded(X), rounded(Y), 1)
    got = sk.sigkernel_gram(cuda(X), cuda(Y), 1, gram_precision=precision).cpu().numpy()
    assert worst(got, ref) <= tol(d)


def test_ragged_rows_and_columns():
    lx, ly = [1, 31, 64, 2, 97], [45, 1, 140, 7, 33, 2]
    xs = [workloads.random_paths(7500 + i, 1, L, 21)[0] for i, L in enumerate(lx)]
    ys = [workloads.random_paths(7600 + i, 1, L, 21)[0] for i, L in enumerate(ly)]
    X, Y = RaggedPaths.from_list(xs, "cuda"), RaggedPaths.from_list(ys, "cuda")
    for a, b, A, B in ((X, Y, xs, ys), (X, cuda(np.stack([ys[0]] * 3)), xs, [ys[0]] * 3),
                       (cuda(np.stack([xs[1]] * 2)), Y, [xs[1]] * 2, ys)):
        got = sk.sigkernel_gram(a, b, 1).cpu().numpy()
        for i, x in enumerate(A):
            for j, y in enumerate(B):
                ref = 1.0 if min(len(x), len(y)) == 1 else oracle.solve(f64(x), f64(y), 1)
                assert abs(got[i, j] - ref) <= tol(21) * max(1.0, abs(ref)), (i, j)
