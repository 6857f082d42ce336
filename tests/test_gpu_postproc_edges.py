"""Post-processing kernels at the sizes where a pack, a read-ahead run or a group
of frames is cut: odd lengths, views that start off a 16-byte boundary, frame
counts around the group size, more kept frames than one copy launch takes.
Values against NumPy in FP64; counts and copies exact."""
import ctypes

import numpy as np
import pytest

from tests.gpu_helpers import device

pytestmark = pytest.mark.gpu


def _view(torch, a, dtype, shift):
    """a (m x n) on the device as frames of a buffer that starts `shift` entries
    past its allocation, and the values the device holds, in FP64."""
    m, n = a.shape
    buf = torch.empty(m * n + shift, dtype=getattr(torch, np.dtype(dtype).name), device="cuda")
    v = buf[shift:].view(n, m).t()
    v.copy_(torch.from_numpy(a.astype(dtype)).cuda())
    return v, a.astype(dtype).astype(np.float64)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,shift", [(1, 2, 0), (3, 7, 1), (4, 8, 0), (255, 9, 0), (256, 16, 3),
                                       (769, 17, 0), (1028, 25, 0), (1029, 24, 2), (70001, 33, 1),
                                       (16384, 67, 0)])
def test_reductions_at_edges(m, n, shift, dtype):
    import torch
    import paper_2506_10257_amd.postproc as pp
    device()
    rng = np.random.default_rng(m * 31 + n)
    A, a = _view(torch, rng.standard_normal((m, n)), dtype, shift)
    B, b = _view(torch, rng.standard_normal((m, n)), dtype, shift // 2)  # A and B aligned alike or not
    mask = rng.random((m, n)) < 0.3
    mask[0, 0] = True
    mb = torch.empty(m * n + shift, dtype=torch.uint8, device="cuda")
    M = mb[shift:].view(n, m).t()
    M.copy_(torch.from_numpy(mask.astype(np.uint8)).cuda())

    # FP64 sums of N entries in another order: N eps of the summed magnitudes
    eps = m * n * np.finfo(np.float64).eps + 1e-14
    assert abs(pp.rmse(A, B) - np.sqrt(np.mean((a - b) ** 2))) <= eps * np.sqrt(np.mean((a - b) ** 2))
    assert abs(pp.masked_mean(A, M) - a[mask].mean()) <= eps * np.abs(a[mask]).mean()
    _, counts = pp.dice(A, 0.1, B, -0.2)
    x, y = a >= 0.1, b >= -0.2
    assert counts == (int((x & y).sum()), int(x.sum()), int(y.sum()))
    if m > 2:
        rho = pp.frame_correlation(A)
        ref = np.array([np.corrcoef(a[:, t], a[:, t + 1])[0, 1] for t in range(n - 1)])
        assert np.max(np.abs(rho - ref)) <= 1e-12
    for W in (1, min(n, 8), min(n, 32)):
        out = pp.moving_average(A, W).cpu().numpy().astype(np.float64)
        ref = np.stack([a[:, t:t + W].mean(1) for t in range(n - W + 1)], 1)
        assert np.max(np.abs(out - ref)) <= (1e-12 if dtype == np.float64 else 1e-6) * np.abs(a).max()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,shift", [(1, 5, 0), (5, 30, 1), (2048, 9, 0), (2052, 11, 0), (8195, 3, 0), (4, 700, 0)])
def test_frame_copies_at_edges(m, n, shift, dtype):
    import torch
    from paper_2506_10257_amd import _dtype_code, _lib
    device()
    rng = np.random.default_rng(m + n)
    X, _ = _view(torch, rng.standard_normal((m, n)), dtype, shift)
    buf = torch.zeros(m * n + 8, dtype=X.dtype, device="cuda")
    lib = _lib.load()
    for keep in (np.ones(n, np.int32), (rng.random(n) < 0.8).astype(np.int32)):
        kept = np.flatnonzero(keep)
        buf.fill_(-7.0)
        got = lib.rpca_frame_select(X.data_ptr(), m, n, _dtype_code(X),
                                    keep.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), buf.data_ptr(),
                                    torch.cuda.current_stream().cuda_stream)
        assert got == len(kept)
        want = X.t()[torch.from_numpy(kept).cuda()].reshape(-1)
        assert torch.equal(buf[:want.numel()], want)
        assert bool((buf[want.numel():] == -7.0).all())
