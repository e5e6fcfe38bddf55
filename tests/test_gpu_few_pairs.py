"""Grams of so few pairs that every wave has a SIMD to itself, with x paths of at most
64 fine rows: one row per lane, rows on 16 lanes and heights between, explicit,
implicit and lifted, uniform and ragged, against the FP64 oracle.  Error metric and
tolerances as in test_gpu_parity.py (1e-6 of max(1, |k|)) and test_gpu_lifted.py (2e-7)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
import workloads
from paper_2006_14794_amd import RaggedPaths

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def worst(got, ref):
    got = got.cpu().numpy().astype(np.float64)
    return float((np.abs(got - ref) / np.maximum(1.0, np.abs(ref))).max())


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("nx,ny", [(1, 1), (3, 2)])
@pytest.mark.parametrize("lam,m", [(0, 1), (0, 41), (0, 63), (0, 64), (0, 65), (1, 7), (1, 31),
                                   (1, 32), (1, 33), (2, 15), (2, 16), (2, 17), (3, 5), (3, 8),
                                   (3, 9)])
def test_short_x_paths_alone(lam, m, nx, ny, ragged):
    d = 1 + (m + lam) % 5
    xs = list(workloads.random_paths(100 + m, nx, m + 1, d, std=0.7))
    ys = list(workloads.random_paths(200 + m, ny, 150, d, std=0.7))
    if ragged:
        xs = [x[:m + 1 - i] if m > i else x for i, x in enumerate(xs)]
        ys = [y[:150 - 60 * i] for i, y in enumerate(ys)]
        X, Y = RaggedPaths.from_list(xs, "cuda"), RaggedPaths.from_list(ys, "cuda")
    else:
        X, Y = (torch.from_numpy(np.stack(p)).cuda() for p in (xs, ys))
    x64, y64 = ([p.astype(np.float64) for p in q] for q in (xs, ys))
    pairs = [(x, y) for x in x64 for y in y64]
    ref = np.array([oracle.solve(x, y, lam) for x, y in pairs]).reshape(nx, ny)
    assert worst(sk.sigkernel_gram(X, Y, lam), ref) <= 1e-6
    ref = np.array([oracle.solve_implicit(x, y, lam) for x, y in pairs]).reshape(nx, ny)
    assert worst(sk.sigkernel_gram(X, Y, lam, scheme="implicit"), ref) <= 1e-6
    ref = np.array([oracle.solve_lifted(x, y, lam, kernel=oracle.rbf(0.8))
                    for x, y in pairs]).reshape(nx, ny)
    assert worst(sk.sigkernel_gram_lifted(X, Y, lam, sigma=0.8), ref) <= 2e-7
