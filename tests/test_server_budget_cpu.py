"""What a request counts against a server's budget: the eigensolver's own matrices
above 64 frames (at most 2 MB per request) do not count, so a budget that was
measured in requests of a size holds as many of them whatever the eigensolver."""
import pytest

import paper_2506_10257_amd as rp
from paper_2506_10257_amd.server import Server, request_bytes

from .test_server_cpu import _prob

# M, L, S, the iterate buffers, partials, P, V, the sweeps' scratch, state, tables
COUNTED = [(4096, 64, rp.RPCA_F32, 7687168), (4096, 100, rp.RPCA_F32, 12605184),
           (262144, 132, rp.RPCA_F32, 991815936), (1000, 65, rp.RPCA_F64, 3979712),
           (96133, 97, rp.RPCA_F64, 538672248)]


@pytest.mark.parametrize("m,n,dtype,size", COUNTED)
def test_request_bytes(m, n, dtype, size):
    assert request_bytes(m, n, dtype) == size
    if n > 64:
        assert size < rp.rpca_footprint_bytes(m, n, dtype) + 3 * m * n * (4 if dtype == rp.RPCA_F32 else 8) <= size + (2 << 20)


def test_an_exact_budget_admits_its_requests():
    srv = Server(rp.RPCA_F32, hbm_budget=3 * 12605184, max_active=8, quantum=4, simulate=True)
    for i in range(3):
        assert srv.submit_raw(_prob(4096, 100, 8, (1 + i) << 36), i) == 0
    srv.step()
    assert srv.pending()[1:3] == (0, 3)
    srv.close()
