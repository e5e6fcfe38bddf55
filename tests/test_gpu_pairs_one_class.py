"""Ragged pairs on both sides of the rule that runs all of them in one launch (at
most 1024 pairs, 2048 where a step holds few cells): one launch and two give the
same values bit for bit, and those of the FP64 oracle.  Error metric and tolerance
as in test_gpu_parity.py: |k_gpu - k_ref| / max(1, |k_ref|) <= 1e-6."""
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


def batch(seed, n, hi):
    rng = np.random.default_rng(seed)
    return [workloads.random_paths(seed + i, 1, int(rng.integers(1, hi + 1)), 2)[0] for i in range(n)]


@pytest.mark.parametrize("lam,hi,n", [(0, 30, 3), (0, 100, 2048), (0, 100, 2049), (2, 40, 1024),
                                      (2, 40, 2049), (3, 120, 1024), (3, 120, 1025)])
def test_launches_agree(lam, hi, n):
    base = 60  # distinct pairs, repeated; the last pairs of the batch are short ones
    xs, ys = batch(17 + lam, base, hi), batch(900 + lam, base, hi)
    # a path without cells and one that needs the most rows, in every batch
    xs[0], xs[1], ys[1] = xs[0][:1], workloads.random_paths(5, 1, hi, 2)[0], workloads.random_paths(6, 1, hi, 2)[0]
    pick = [i % base for i in range(n)]
    X = RaggedPaths.from_list([xs[i] for i in pick], "cuda")
    Y = RaggedPaths.from_list([ys[i] for i in pick], "cuda")
    got = sk.sigkernel_pair(X, Y, lam).cpu().numpy()
    few = min(n, base)
    ref = np.asarray(oracle.pairs([x.astype(np.float64) for x in xs[:few]],
                                  [y.astype(np.float64) for y in ys[:few]], lam))
    err = np.abs(got[:few] - ref) / np.maximum(1.0, np.abs(ref))
    assert err.max() <= TOL
    assert all(got[i] == got[pick[i]] for i in range(n))
    # the same pairs among more than any single launch takes
    m = 2100
    more = [i % base for i in range(m)]
    two = sk.sigkernel_pair(RaggedPaths.from_list([xs[i] for i in more], "cuda"),
                            RaggedPaths.from_list([ys[i] for i in more], "cuda"), lam).cpu().numpy()
    assert np.array_equal(two[:few], got[:few])
