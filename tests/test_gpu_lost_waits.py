"""Waits inside a launch that give up (rpca_inject_wait(0): nearly every wait
ends at once, and every kernel still ends normally): the results are right."""
from contextlib import contextmanager

import numpy as np
import pytest

from oracle import rpca
from paper_2506_10257_amd import _lib

from .gpu_helpers import device, gpu_solve, to_host
from .test_gpu_eig_steps import _spectrum

pytestmark = pytest.mark.gpu


@contextmanager
def no_waiting():
    lib = _lib.load()
    assert lib.rpca_inject_wait(0.0) == 0
    try:
        yield
    finally:
        lib.rpca_inject_wait(-1.0)


@pytest.mark.parametrize("n,dtype", [(80, np.float64), (128, np.float64), (112, np.float32), (132, np.float32), (144, np.float32)])
def test_a_lost_team_leaves_the_oracles_iterates(n, dtype):
    device()
    X = _spectrum(300, n, 10.0 ** np.linspace(2, -1, n), n)
    ref = rpca(X, mu=1.0, tol=0.0, maxit=12)
    with no_waiting():
        L, S, it, rc, _ = gpu_solve(X, dtype, mu=1.0, tol=0.0, maxit=12)
        assert _lib.load().rpca_last_run() & _lib.RPCA_RUN_TEAM_LOST
    assert it == 12
    bar = (1e-10 if dtype == np.float64 else 1e-4) * np.linalg.norm(X)  # as for waits that hold
    for got, want in ((L, ref.L), (S, ref.S)):
        assert np.linalg.norm(to_host(got) - want) <= bar, n
