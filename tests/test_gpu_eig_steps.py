"""The eigensolver's simultaneous steps and the first-order projector, at the
spectra where they can go wrong: clusters on both sides of the threshold,
clusters that the threshold cuts, repeated and zero singular values, and frame
counts at the edges of the 16-frame blocks of the matrix products.  The oracle
runs the same iterations with a full SVD."""
import numpy as np
import pytest

from oracle import rel_fro, rpca

from .gpu_helpers import gpu_solve, to_host

pytestmark = pytest.mark.gpu


def _spectrum(m, n, s, seed):
    """m x n with singular values s (n of them), plus 2% large outliers."""
    r = np.random.default_rng(seed)
    Q, _ = np.linalg.qr(r.standard_normal((m, n)))
    W, _ = np.linalg.qr(r.standard_normal((n, n)))
    X = (Q * s) @ W.T
    hit = r.random((m, n)) < 0.02
    X[hit] += 3.0 * np.sqrt(np.mean(X * X)) * r.standard_normal(int(hit.sum()))
    return X


def _cases(n):
    tau = 1.0
    near = tau * (1.0 + 1e-6 * np.arange(n))
    lo_hi = np.where(np.arange(n) % 2 == 0, 3.0, 0.5)           # two clusters, one dropped
    cut = tau * (1.0 + 1e-3 * (np.arange(n) - n / 2) / n)       # the threshold cuts a tight cluster
    zero = np.where(np.arange(n) < max(1, n // 3), 5.0, 0.0)    # rank deficient
    return {"near": near, "lo_hi": lo_hi, "cut": cut, "graded": 10.0 ** np.linspace(3, -1, n),
            "zero": zero, "equal": np.full(n, 2.0)}


@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64])
@pytest.mark.parametrize("kind", ["near", "lo_hi", "cut", "graded", "zero", "equal"])
def test_spectra_fp64(n, kind):
    X = _spectrum(401, n, _cases(n)[kind], 7 * n + 1)
    for k in (1, 2, 3, 9, 30):
        ref = rpca(X, mu=1.0, tol=0.0, maxit=k)
        L, S, it, rc, _ = gpu_solve(X, np.float64, mu=1.0, tol=0.0, maxit=k)
        assert it == k
        # the FP64 bar, relative to the window: L or S alone may be near zero
        scale = np.linalg.norm(X)
        for got, want in ((L, ref.L), (S, ref.S)):
            assert np.linalg.norm(to_host(got) - want) <= 1e-10 * scale, (kind, n, k)


@pytest.mark.parametrize("n", [3, 20, 40, 64])
@pytest.mark.parametrize("kind", ["near", "cut", "graded", "zero"])
def test_spectra_fp32(n, kind):
    X = _spectrum(300, n, _cases(n)[kind], 5 * n + 2)
    ref = rpca(X, mu=1.0, tol=0.0, maxit=12)
    L, S, it, rc, _ = gpu_solve(X, np.float32, mu=1.0, tol=0.0, maxit=12)
    scale = np.linalg.norm(X)
    for got, want in ((L, ref.L), (S, ref.S)):
        assert np.linalg.norm(to_host(got) - want) <= 1e-4 * scale, (kind, n)


def test_long_run_stays_orthogonal():
    """300 iterations of warm starts: the projector does not drift."""
    r = np.random.default_rng(3)
    X = _spectrum(600, 20, 10.0 ** np.linspace(2, 0, 20), 11) + 0.05 * r.standard_normal((600, 20))
    ref = rpca(X, tol=0.0, maxit=300)
    L, S, it, rc, _ = gpu_solve(X, np.float64, tol=0.0, maxit=300)
    assert rel_fro(to_host(L), ref.L) <= 1e-10 and rel_fro(to_host(S), ref.S) <= 1e-10
