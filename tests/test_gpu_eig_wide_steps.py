"""The simultaneous steps above 64 frames, at the spectra where they can go
wrong and at frame counts around the 16-frame blocks, against the oracle's full
SVD; and with every number of workgroups per solve that the dispatch chooses
(one solve alone gets a full team, 7 and 40 solves in a batch smaller ones, down
to one workgroup): the same bits."""
import numpy as np
import pytest

from oracle import rpca

from .gpu_helpers import device, gpu_solve, to_dev, to_host
from .test_gpu_eig_steps import _cases, _spectrum

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 80, 81, 97, 112, 113, 128])
@pytest.mark.parametrize("kind", ["near", "lo_hi", "cut", "graded", "zero", "equal"])
def test_wide_spectra_fp64(n, kind):
    X = _spectrum(301, n, _cases(n)[kind], 3 * n + 1)
    for k in (1, 2, 4, 15):
        ref = rpca(X, mu=1.0, tol=0.0, maxit=k)
        L, S, it, rc, _ = gpu_solve(X, np.float64, mu=1.0, tol=0.0, maxit=k)
        assert it == k
        scale = np.linalg.norm(X)
        for got, want in ((L, ref.L), (S, ref.S)):
            assert np.linalg.norm(to_host(got) - want) <= 1e-10 * scale, (kind, n, k)


@pytest.mark.parametrize("n", [129, 137, 144])
@pytest.mark.parametrize("kind", ["near", "cut", "graded", "zero"])
def test_wide_spectra_fp32(n, kind):
    X = _spectrum(300, n, _cases(n)[kind], 5 * n + 2)
    ref = rpca(X, mu=1.0, tol=0.0, maxit=12)
    L, S, it, rc, _ = gpu_solve(X, np.float32, mu=1.0, tol=0.0, maxit=12)
    scale = np.linalg.norm(X)
    for got, want in ((L, ref.L), (S, ref.S)):
        assert np.linalg.norm(to_host(got) - want) <= 1e-4 * scale, (kind, n)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("count", [7, 40])
def test_team_sizes_give_the_same_bits(count, dtype):
    import torch
    import paper_2506_10257_amd as rp
    device()
    sizes = [65, 96, 112, 127] if dtype == np.float64 else [65, 96, 112, 144]
    Ms = [to_dev(_spectrum(200 + 3 * i, sizes[i % 4], 10.0 ** np.linspace(2, -1, sizes[i % 4]), i), dtype)
          for i in range(count)]
    together = rp.solve_many(Ms, tol=0.0, maxit=14)
    for i in range(min(count, 8)):
        alone = rp.solve(Ms[i], tol=0.0, maxit=14)
        assert torch.equal(alone.L, together[i].L) and torch.equal(alone.S, together[i].S), (i, sizes[i % 4])
