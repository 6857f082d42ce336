"""The whole-solve kernel (one launch, rows in registers) against the launched
path, bitwise: the kernel-timing mode always takes the launched path.  Row
counts at the edges of the tiles per workgroup (1, 2, 4), of the reduction
groups (32 tiles) and of the grid; frame counts at the edges of the register
classes; starts, stops and special inputs."""
import threading

import numpy as np
import pytest

import paper_2506_10257_amd as rp

from .gpu_helpers import device

pytestmark = pytest.mark.gpu


def _window(m, n, dtype, seed):
    """(n, 1, m) stack: rank-one background, sparse spots, noise."""
    import torch
    g = torch.Generator(device=device()).manual_seed(seed)
    a = 1.0 + 0.3 * torch.randn((1, m), generator=g, device="cuda", dtype=torch.float64).abs()
    c = 1.0 + 0.05 * torch.sin(torch.arange(n, device="cuda", dtype=torch.float64))[:, None]
    hit = torch.rand((n, m), generator=g, device="cuda", dtype=torch.float64) < 0.03
    X = c * a + 2.0 * hit + 0.1 * torch.randn((n, m), generator=g, device="cuda", dtype=torch.float64)
    return X.to(dtype).reshape(n, 1, m).contiguous()


def _both(M, **kw):
    got = rp.solve(M, return_Y=True, **kw)
    rp.rpca_profile_enable(True)
    try:
        want = rp.solve(M, return_Y=True, **kw)
    finally:
        rp.rpca_profile_enable(False)
        rp.rpca_profile_read(True)
    return got, want


def _same(got, want):
    import torch
    assert (got.iterations, got.status, got.residual) == (want.iterations, want.status, want.residual)
    for k in "LSY":
        assert torch.equal(getattr(got, k), getattr(want, k)), k


F32 = [(1, 3), (255, 1), (256, 2), (257, 10), (513, 11), (8191, 16), (8193, 17), (65535, 20), (65536, 20),
       (65537, 20), (66000, 21), (70001, 32), (131072, 32), (131073, 10), (131073, 16), (200001, 20),
       (262144, 20), (262144, 9)]
F64 = [(1, 2), (300, 5), (256, 10), (8200, 11), (65536, 17), (65537, 20), (130816, 16), (130817, 20)]


@pytest.mark.parametrize("m,n", F32)
def test_f32_bitwise_launched(m, n):
    import torch
    M = _window(m, n, torch.float32, 31 * m + n)
    _same(*_both(M, tol=0.0, maxit=7))


@pytest.mark.parametrize("m,n", F64)
def test_f64_bitwise_launched(m, n):
    import torch
    M = _window(m, n, torch.float64, 17 * m + n)
    _same(*_both(M, tol=0.0, maxit=7))


@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
def test_stops_starts_and_special_inputs(dtype_name):
    import torch
    dt = getattr(torch, dtype_name)
    M = _window(5000, 12, dt, 5)
    _same(*_both(M, tol=1e-4, maxit=400))                   # stopped by the tolerance
    _same(*_both(M, tol=1e-4, maxit=1))                     # by the cap
    first = rp.solve(M, tol=0.0, maxit=20, return_Y=True)
    _same(*_both(M, tol=1e-5, maxit=400, S0=first.S, Y0=first.Y))
    _same(*_both(M, tol=0.0, maxit=3, S0=first.S))
    _same(*_both(M, tol=0.0, maxit=3, Y0=first.Y))
    Z = torch.zeros_like(M)
    got, want = _both(Z, tol=1e-6, maxit=5)
    _same(got, want)
    assert got.iterations == 0 and not bool(got.L.any())
    bad = M.clone()
    bad[3, 0, 17] = float("nan")
    with pytest.raises(RuntimeError):
        rp.solve(bad, tol=1e-6, maxit=5)
    # offsets that are not multiples of 16 bytes
    flat = torch.empty(12 * 4999 + 1, dtype=dt, device="cuda")
    V = flat[1:].view(12, 1, 4999)
    V.copy_(M[:, :, :4999])
    _same(*_both(V, tol=0.0, maxit=5))


def test_calls_at_once():
    """Two threads: one takes the whole-solve kernel, the other the launched
    path (or the kernel later); the results are the same."""
    import torch
    Ms = [_window(20000 + 77 * i, 20, torch.float32, 100 + i) for i in range(2)]
    alone = [rp.solve(M, tol=0.0, maxit=60) for M in Ms]
    out = [[], []]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(8):
                out[i].append(rp.solve(Ms[i], tol=0.0, maxit=60))

    torch.cuda.synchronize()
    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        for r in out[i]:
            assert torch.equal(r.L, alone[i].L) and torch.equal(r.S, alone[i].S)
