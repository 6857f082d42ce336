"""The tile kernel where its loads are clamped: fewer rows than a tile or one
row into the next, fewer frames than waves, frame counts at both ends of a
class, in every storage type and contraction; against the oracle, relative to
the norm of the window."""
import numpy as np
import pytest

import paper_2506_10257_amd as rp
from oracle import rpca
from tests.gpu_helpers import device, to_dev, to_host

pytestmark = pytest.mark.gpu


def _window(m, n):
    r = np.random.default_rng(1000 * m + n)
    X = np.outer(r.standard_normal(m), 1.0 + 0.1 * r.standard_normal(n)) + 0.01 * r.standard_normal((m, n))
    X[r.random((m, n)) < 0.03] += 2.0
    return X


def _errors(X, dtype, k, **kw):
    ref = rpca(X.astype(dtype).astype(np.float64), tol=0.0, maxit=k)
    r = rp.solve(to_dev(X, dtype), tol=0.0, maxit=k, **kw)
    assert r.iterations == k
    s = np.linalg.norm(X)
    return max(np.linalg.norm(to_host(r.L) - ref.L), np.linalg.norm(to_host(r.S) - ref.S)) / s


@pytest.mark.parametrize("m,n", [(1, 2), (63, 3), (64, 16), (65, 17), (130, 32), (191, 33), (64, 48), (257, 49),
                                 (129, 97), (65, 144)])
def test_bf16x6_edges(m, n):
    device()
    assert _errors(_window(m, n), np.float32, 8, gram_mode=rp.RPCA_GRAM_BF16X6) <= 1e-4


@pytest.mark.parametrize("m,n", [(1, 65), (63, 80), (65, 81), (129, 112), (64, 113), (191, 144)])
def test_fp32_edges(m, n):
    device()
    assert _errors(_window(m, n), np.float32, 8) <= 1e-4


@pytest.mark.parametrize("m,n", [(1, 33), (63, 48), (65, 49), (129, 64), (64, 65), (191, 96), (130, 97), (65, 128)])
def test_fp64_edges(m, n):
    device()
    assert _errors(_window(m, n), np.float64, 8) <= 1e-10
