"""FP64 inputs far from one.  Those whose Gram overflows (sums of squares above 1.8e308): the
solve says RPCA_ERR_NONFINITE, by every eigensolver and entry point, instead of
dropping the infinite eigenvalues; all others give what the same input near one
gives."""
import numpy as np
import pytest

import paper_2506_10257_amd as rp

from .gpu_helpers import device

pytestmark = pytest.mark.gpu

NONFINITE = r"\(-4\)"


def _window(n, m=3000):
    import torch
    g = torch.Generator(device=device()).manual_seed(n)
    a = 1.0 + 0.3 * torch.randn((1, m), generator=g, device="cuda", dtype=torch.float64).abs()
    return (a + 0.1 * torch.randn((n, m), generator=g, device="cuda", dtype=torch.float64)).reshape(n, 1, m)


@pytest.mark.parametrize("n", [1, 10, 20, 32, 33, 64, 65, 100, 113, 128])
def test_an_overflowing_gram_is_an_error(n):
    X = _window(n)
    for big in (1e155, 1e160, 1e200):
        Y = X.clone()
        Y[n // 2, 0, 7] = big
        with pytest.raises(RuntimeError, match=NONFINITE):
            rp.solve(Y, tol=1e-6, maxit=20)
        with pytest.raises(RuntimeError, match=NONFINITE):
            rp.solve_many([Y, Y.clone()], tol=1e-6, maxit=20)
    for name in ("S0", "Y0"):
        Z = X * 0.0
        Z[n // 2, 0, 3] = 1e300
        with pytest.raises(RuntimeError, match=NONFINITE):
            rp.solve(X, tol=1e-6, maxit=20, **{name: Z})


@pytest.mark.parametrize("scale", [2.0**-340, 2.0**-260, 2.0**255, 2.0**330, 2.0**495])
@pytest.mark.parametrize("n", [1, 10, 20, 32, 33, 64, 65, 100, 113, 128])
def test_powers_of_two_change_no_bit(n, scale):
    """X and its multiple by a power of two: the same iterates, scaled, as long as
    the sums of squares themselves stay in range."""
    import torch
    X = _window(n)
    X[n // 2, 0, ::7] += 3.0
    want = rp.solve(X, tol=0.0, maxit=8)
    for got in (rp.solve(X * scale, tol=0.0, maxit=8), rp.solve_many([X * scale, X * scale], tol=0.0, maxit=8)[1]):
        assert got.iterations == 8
        assert torch.equal(got.L, want.L * scale) and torch.equal(got.S, want.S * scale)
