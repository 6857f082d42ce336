"""rpca_solve_noalloc just below its limit with more than 64 frames: the
matrices of the eigensolver's steps have room beside the 192 MiB."""
import numpy as np
import pytest

import paper_2506_10257_amd as rp
from paper_2506_10257_amd import _lib
from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,steps", [(100, 12 * 112 * 112 * 8), (140, 12 * 144 * 144 * 8)])
def test_wide_window_at_the_limit(n, steps):
    import torch
    device()
    lib = _lib.load()
    limit = _lib.RPCA_NOALLOC_MAX_BYTES
    m = 64 * (limit // (64 * 16 * n))  # four iterate buffers of FP32 alone fill the array
    while lib.rpca_footprint_bytes(m, n, _lib.RPCA_F32) - steps + 8192 > limit:
        m -= 64
    assert lib.rpca_footprint_bytes(m, n, _lib.RPCA_F32) > limit
    g = torch.Generator(device="cuda").manual_seed(n)
    M = torch.randn(n, m, generator=g, device="cuda").t()
    L = torch.empty(n, m, device="cuda").t()
    S = torch.empty(n, m, device="cuda").t()
    rc, it = rp.rpca_solve_noalloc(M, m, n, _lib.RPCA_F32, -1.0, -1.0, 0.0, 3, L, S)
    ref = rp.solve(M, tol=0.0, maxit=3)
    assert it == 3 and rc == ref.status
    assert torch.equal(L, ref.L) and torch.equal(S, ref.S)
