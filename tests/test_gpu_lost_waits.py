"""Waits inside a launch that give up (rpca_inject_wait(0): nearly every wait
ends at once, and every kernel still ends normally): the results are those of
waits that hold, bit for bit, through every entry point."""
from contextlib import contextmanager

import numpy as np
import pytest

import paper_2506_10257_amd as rp
from oracle import rpca
from paper_2506_10257_amd import _lib

from .gpu_helpers import device, gpu_solve, to_dev, to_host
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


def _window(n, dtype, m=300):
    return to_dev(_spectrum(m, n, 10.0 ** np.linspace(2, -1, n), n), dtype)


def _same(a, b):
    import torch
    assert (a.iterations, a.status, a.residual) == (b.iterations, b.status, b.residual)
    for k in "LSY":
        if getattr(a, k) is not None:
            assert torch.equal(getattr(a, k), getattr(b, k)), k


@pytest.mark.parametrize("n,dtype", [(65, np.float32), (132, np.float32), (100, np.float64)])
def test_a_lost_team_changes_no_bit(n, dtype):
    device()
    M = _window(n, dtype)
    want = rp.solve(M, tol=1e-7, maxit=40, return_Y=True)
    with no_waiting():
        _same(rp.solve(M, tol=1e-7, maxit=40, return_Y=True), want)
        assert _lib.load().rpca_last_run() == _lib.RPCA_RUN_TEAM_LOST
    want2 = rp.solve(M, tol=0.0, maxit=9, S0=want.S, Y0=want.Y, return_Y=True)
    assert _lib.load().rpca_last_run() == 0
    with no_waiting():
        _same(rp.solve(M, tol=0.0, maxit=9, S0=want.S, Y0=want.Y, return_Y=True), want2)


def test_lost_teams_in_a_batch_a_server_and_without_allocation():
    import torch
    device()
    ns = [100, 20, 132, 65, 40]
    Ms = [_window(n, np.float32, 200 + 7 * n) for n in ns]
    want = [rp.solve(M, tol=0.0, maxit=15) for M in Ms]
    srv = rp.Server(dtype=rp.RPCA_F32, hbm_budget=1 << 30, max_active=8, quantum=4)
    with no_waiting():
        for got, ref in zip(rp.solve_many(Ms, tol=0.0, maxit=15), want):
            _same(got, ref)
        assert _lib.load().rpca_last_run() & _lib.RPCA_RUN_TEAM_LOST
        for i, M in enumerate(Ms):
            srv.submit(M, i, tol=0.0, maxit=15)
        done = {}
        for _ in range(40):
            done.update((c.tag, c) for c in srv.step())
        assert sorted(done) == list(range(len(Ms)))
        for i, ref in enumerate(want):
            assert (done[i].iterations, done[i].status) == (ref.iterations, ref.status)
            assert torch.equal(done[i].L, ref.L) and torch.equal(done[i].S, ref.S), ns[i]
        for M, ref in zip(Ms, want):
            L, S = torch.empty_like(M), torch.empty_like(M)
            rc, it = rp.rpca_solve_noalloc(M, M.shape[0], M.shape[1], rp.RPCA_F32, -1.0, -1.0, 0.0, 15, L, S)
            assert (rc, it) == (ref.status, ref.iterations)
            assert torch.equal(L, ref.L) and torch.equal(S, ref.S)


@pytest.mark.parametrize("m,n,dtype", [(4096, 10, np.float32), (16384, 20, np.float64), (262144, 20, np.float32)])
def test_a_lost_whole_solve_runs_again(m, n, dtype):
    """The whole-solve kernel (up to 32 frames) and its launched replacement."""
    device()
    g = np.random.default_rng(n)
    M = to_dev(g.standard_normal((m, 1)) @ g.standard_normal((1, n)) + 0.1 * g.standard_normal((m, n)), dtype)
    want = rp.solve(M, tol=0.0, maxit=12, return_Y=True)
    assert _lib.load().rpca_last_run() == _lib.RPCA_RUN_WHOLE
    with no_waiting():
        _same(rp.solve(M, tol=0.0, maxit=12, return_Y=True), want)
        assert _lib.load().rpca_last_run() == _lib.RPCA_RUN_WHOLE_LOST
