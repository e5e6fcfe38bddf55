"""Few pairs of equal lengths on both sides of the choice between one wave per
pair and pipelined bands at a kernel order below the dyadic order, against the
FP64 oracle (|k_gpu - k_ref| / max(1, |k_ref|) <= 1e-6) and, bit for bit,
against the same pairs inside a batch large enough to be swept otherwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2006_14794_amd as sk
import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sk.load()


def cuda(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32).cuda()


# rows of one band, of several, one row past a band; 15 to 17, 63 to 65 columns
# past a chunk of 16; every order, orders above 3
CASES = [(1, 66, 66, 1, 0), (2, 130, 145, 2, 0), (1, 258, 272, 3, 0), (3, 601, 640, 5, 0),
         (2, 513, 528, 4, 1), (1, 514, 577, 16, 1), (5, 300, 1025, 2, 1), (1, 257, 321, 7, 2),
         (4, 258, 400, 9, 2), (1, 400, 401, 3, 3), (2, 129, 130, 2, 4), (1, 200, 215, 12, 4),
         (1, 65, 97, 2, 6)]


@pytest.mark.parametrize("n,lx,ly,d,lam", CASES)
def test_against_oracle_and_large_batch(n, lx, ly, d, lam):
    X = workloads.random_paths(5000 + lx, n, lx, d, std=1.0)
    Y = workloads.random_paths(6000 + ly, n, ly, d, std=1.0)
    got = sk.sigkernel_pair(cuda(X), cuda(Y), lam)
    ref = np.asarray(oracle.pairs([x.astype(np.float64) for x in X],
                                  [y.astype(np.float64) for y in Y], lam))
    g = got.cpu().numpy().astype(np.float64)
    assert (np.abs(g - ref) / np.maximum(1.0, np.abs(ref))).max() <= TOL
    # swapped arguments: the shorter path goes on the rows either way
    assert torch.equal(got, sk.sigkernel_pair(cuda(Y), cuda(X), lam))
    if lam <= 3:
        reps = 2100 // n + 1
        many = sk.sigkernel_pair(cuda(np.tile(X, (reps, 1, 1))), cuda(np.tile(Y, (reps, 1, 1))), lam)
        assert torch.equal(many, got.repeat(reps))


@pytest.mark.parametrize("lam", [0, 2, 4])
def test_implicit_and_broken_pairs(lam):
    X = workloads.random_paths(71, 3, 300, 3, std=1.0)
    Y = workloads.random_paths(72, 3, 420, 3, std=1.0)
    ref = np.asarray(oracle.pairs_implicit([x.astype(np.float64) for x in X],
                                           [y.astype(np.float64) for y in Y], lam))
    Y[1, 200, 1] = np.nan
    got = sk.sigkernel_pair(cuda(X), cuda(Y), lam, scheme="implicit").cpu().numpy()
    assert np.isnan(got[1])
    for k in (0, 2):
        assert abs(got[k] - ref[k]) <= TOL * max(1.0, abs(ref[k]))
