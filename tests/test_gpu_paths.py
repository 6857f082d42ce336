"""That the paths which other tests mean to compare did run: the whole-solve kernel
at the sizes of test_gpu_resident, every workgroup size of the launched eigensolver,
teams of one workgroup above 64 frames, and the sweeps that take over where the
steps do not converge (also those that accumulate their rotations as an FP32
increment: FP32, 113 to 136 frames)."""
import numpy as np
import pytest

import paper_2506_10257_amd as rp
from oracle import rpca
from paper_2506_10257_amd import _lib
from synth import batch_window

from .gpu_helpers import device, gpu_solve, to_dev, to_host
from .test_gpu_eig_steps import _cases, _spectrum
from .test_gpu_resident import F32, F64, _window

pytestmark = pytest.mark.gpu


def _ran():
    return _lib.load().rpca_last_run()


@pytest.mark.parametrize("dtype_name,sizes", [("float32", F32), ("float64", F64)])
def test_the_whole_solve_kernel_runs(dtype_name, sizes):
    import torch
    for m, n in sizes:
        rp.solve(_window(m, n, getattr(torch, dtype_name), m + n), tol=0.0, maxit=2)
        # FP64 from 512 tiles on: two tiles per partial, by launches
        whole = dtype_name == "float32" or m <= 130816
        assert _ran() == (_lib.RPCA_RUN_WHOLE if whole else 0), (m, n)


@pytest.mark.parametrize("n,cls", [(12, 16), (20, 32), (32, 32), (40, 64)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_eig_threads_bitwise_by_launches(n, cls, dtype):
    """Two problems at once are always launched; the workgroup size of their
    eigensolver changes no bit, and they agree with the whole-solve kernel."""
    import torch
    device()
    M = to_dev(batch_window(64, 64, n, 3100 + n).X(), dtype)
    dt = rp.RPCA_F64 if dtype == np.float64 else rp.RPCA_F32
    K = rp.RPCA_KNOB_EIG_THREADS
    old = rp.rpca_tune_get(K, dt, cls)
    want = rp.solve(M, tol=1e-6, maxit=60)
    sizes = 0
    try:
        for nt in (256, 512, 1024):
            if rp.rpca_tune_set(K, dt, cls, nt) != rp.RPCA_OK:
                continue
            sizes += 1
            for r in rp.solve_many([M, M.clone()], tol=1e-6, maxit=60):
                assert r.iterations == want.iterations, nt
                assert torch.equal(r.L, want.L) and torch.equal(r.S, want.S), nt
            assert _ran() == 0
    finally:
        rp.rpca_tune_set(K, dt, cls, old)
    assert sizes >= 2


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_teams_of_one_give_the_same_bits(dtype):
    """With kernel timing on a batch runs on one stream; 24 windows above 64 frames
    leave each one workgroup (42 // 24).  65 to 144 frames: odd and even numbers of
    16-frame blocks."""
    import torch
    device()
    sizes = [65, 80, 96, 112, 127, 128] if dtype == np.float64 else [65, 80, 96, 112, 132, 144]
    Ms = [to_dev(_spectrum(170 + 3 * i, sizes[i % 6], 10.0 ** np.linspace(2, -1, sizes[i % 6]), i), dtype)
          for i in range(24)]
    rp.rpca_profile_enable(True)
    try:
        together = rp.solve_many(Ms, tol=0.0, maxit=14)
    finally:
        rp.rpca_profile_enable(False)
        rp.rpca_profile_read(True)
    for i in range(0, 24, 3 if dtype == np.float32 else 5):
        alone = rp.solve(Ms[i], tol=0.0, maxit=14)
        assert torch.equal(alone.L, together[i].L) and torch.equal(alone.S, together[i].S), (i, sizes[i % 6])


@pytest.mark.parametrize("n,dtype", [(66, np.float32), (113, np.float32), (132, np.float32), (136, np.float32),
                                     (140, np.float32), (100, np.float64), (120, np.float64)])
@pytest.mark.parametrize("kind", ["near", "cut", "zero"])
def test_sweeps_after_steps_that_do_not_converge(n, dtype, kind):
    X = _spectrum(300, n, _cases(n)[kind], n)
    bar = (1e-10 if dtype == np.float64 else 1e-4) * np.linalg.norm(X)
    swept = 0
    for k in (2, 3):
        ref = rpca(X, mu=1.0, tol=0.0, maxit=k)
        L, S, it, rc, _ = gpu_solve(X, dtype, mu=1.0, tol=0.0, maxit=k)
        swept += 1 if _ran() & _lib.RPCA_RUN_SWEEPS else 0
        assert it == k
        for got, want in ((L, ref.L), (S, ref.S)):
            assert np.linalg.norm(to_host(got) - want) <= bar, (n, k)
    assert swept > 0
