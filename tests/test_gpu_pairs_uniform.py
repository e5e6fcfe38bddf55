"""Pairs of equal lengths, which run without the plan kernel: fewer and more pairs
than wave slots (the first pair of a wave is its slot's, the others come from the
queue), each class of rows per lane, one-point paths, and repeated calls on one
workspace, eager and captured.  Error metric and tolerance as in test_gpu_parity.py:
|k_gpu - k_ref| / max(1, |k_ref|) <= 1e-6."""
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


@pytest.mark.parametrize("n,lx,ly,lam", [(1, 2, 2, 0), (3, 1, 5, 0), (2, 7, 1, 2), (5, 65, 66, 0),
                                         (5, 66, 65, 1), (7, 129, 40, 0), (6, 130, 131, 0),
                                         (4097, 5, 9, 0), (9000, 6, 4, 1)])
def test_equal_lengths(n, lx, ly, lam):
    X = workloads.random_paths(n + lx, n, lx, 3)
    Y = workloads.random_paths(n + ly + 1, n, ly, 3)
    Xc, Yc = cuda(X), cuda(Y)
    got = sk.sigkernel_pair(Xc, Yc, lam)
    ref = np.asarray(oracle.pairs([x.astype(np.float64) for x in X],
                                  [y.astype(np.float64) for y in Y], lam))
    err = np.abs(got.cpu().numpy() - ref) / np.maximum(1.0, np.abs(ref))
    assert err.max() <= TOL
    for _ in range(2):
        assert torch.equal(sk.sigkernel_pair(Xc, Yc, lam), got)


def test_captured_replays():
    X, Y = cuda(workloads.random_paths(61, 5000, 12, 2)), cuda(workloads.random_paths(62, 5000, 9, 2))
    ref = sk.sigkernel_pair(X, Y, 1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = sk.sigkernel_pair(X, Y, 1)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        assert torch.equal(sk.sigkernel_pair(X, Y, 1), ref)
