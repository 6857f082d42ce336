"""The split-BF16 modes round the two halves of a Gram's diagonal blocks
differently; the eigensolver takes the upper one, so that the same call gives the
same bits every time, alone and in a batch."""
import numpy as np
import pytest

import paper_2506_10257_amd as rp

from .gpu_helpers import device, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 20, 32, 40, 48, 64, 100])
@pytest.mark.parametrize("mode", [rp.RPCA_GRAM_BF16X3, rp.RPCA_GRAM_BF16X6])
def test_the_same_bits_every_time(n, mode):
    import torch
    device()
    g = np.random.default_rng(n)
    m = 20000
    M = to_dev(np.abs(1 + 0.3 * g.standard_normal((m, 1))) + 0.1 * g.standard_normal((m, n)), np.float32)
    first = rp.solve(M, tol=0.0, maxit=12, gram_mode=mode)
    others = [rp.solve(M, tol=0.0, maxit=12, gram_mode=mode) for _ in range(5)]
    others += rp.solve_many([M, M.clone()], tol=0.0, maxit=12, gram_mode=mode)
    for r in others:
        assert torch.equal(r.L, first.L) and torch.equal(r.S, first.S)
