"""Single solves beside other calls: a large one runs whole only while no other
call is under way, a small one beside anything; the bits are the same."""
import numpy as np
import pytest

import paper_2506_10257_amd as rp
from paper_2506_10257_amd import _lib

from .gpu_helpers import device, to_dev

pytestmark = pytest.mark.gpu


def _window(m, n):
    g = np.random.default_rng(m + n)
    return to_dev(g.standard_normal((m, 1)) @ g.standard_normal((1, n)) + 0.1 * g.standard_normal((m, n)), np.float32)


def _ran():
    return _lib.load().rpca_last_run()


def test_whole_solves_beside_a_server():
    import torch
    device()
    large, small = _window(262144, 20), _window(4096, 10)
    alone = [rp.solve(M, tol=0.0, maxit=9) for M in (large, small)]
    assert _ran() == _lib.RPCA_RUN_WHOLE
    srv = rp.Server(dtype=rp.RPCA_F32, hbm_budget=1 << 30, max_active=2, quantum=2)
    srv.submit(_window(5000, 40), 1, tol=0.0, maxit=6)
    runs = []
    while srv.pending()[0]:
        srv.step()
        ran = []
        for M, ref in zip((large, small), alone):
            got = rp.solve(M, tol=0.0, maxit=9)
            ran.append(_ran())
            assert torch.equal(got.L, ref.L) and torch.equal(got.S, ref.S)
        runs.append((srv.pending()[0] > 0, ran))
    assert len(runs) >= 3
    for active, ran in runs:  # by launches while the server has an active request
        assert ran == [0 if active else _lib.RPCA_RUN_WHOLE, _lib.RPCA_RUN_WHOLE]
    assert runs[0][0] and not runs[-1][0]


def test_a_server_whose_set_up_failed_holds_nobody_back():
    device()
    large = _window(262144, 20)
    srv = rp.Server(dtype=rp.RPCA_F32, hbm_budget=1 << 30, max_active=2, quantum=2)
    assert srv.inject_failure(rp.RPCA_ERR_DEVICE) == rp.RPCA_OK
    srv.submit(_window(5000, 40), 1, tol=0.0, maxit=6)
    with pytest.raises(RuntimeError):  # a device error: every later step fails too
        for _ in range(3):
            srv.step()
    rp.solve(large, tol=0.0, maxit=3)
    assert _ran() == _lib.RPCA_RUN_WHOLE


def test_more_than_a_thousand_iterations_go_by_launches():
    import torch
    device()
    M = _window(4096, 10)
    a = rp.solve(M, tol=1e-3, maxit=1000)
    assert _ran() == _lib.RPCA_RUN_WHOLE
    b = rp.solve(M, tol=1e-3, maxit=1001)
    assert _ran() == 0
    assert a.iterations == b.iterations < 1000 and torch.equal(a.L, b.L) and torch.equal(a.S, b.S)
