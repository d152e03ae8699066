"""lf_points with the point buffer as its own queries: the points are written
before they are queried, as with two calls."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1903_03837_amd as lp
    lp.library()
    return lp


# the whole buffer, its tail, and queries that start in it and end past it
@pytest.mark.parametrize("n,first,past", [(1, 0, 0), (257, 0, 0), (65535, 0, 0), (65535, 30001, 0), (5000, 4990, 300)])
@pytest.mark.parametrize("K", [1, 5, 9])
def test_points_queried_in_place(lp, n, first, past, K):
    K = min(K, n)
    nq = n - first + past
    buf = torch.zeros((first + nq, 3), device="cuda")
    buf[:, 2] = -1.0
    want_q = buf.clone()
    want_q[:n] = lp.points(n)[0]
    _, want_idx, want_w = lp.points(n, want_q[first:], K, want_xyz=False)
    idx = torch.full((nq, K), -7, dtype=torch.int32, device="cuda")
    w = torch.full((nq, K), -7.0, device="cuda")
    torch.cuda.synchronize()
    r = lp.library().lf_points(n, C.c_void_p(buf.data_ptr()), C.c_void_p(buf.data_ptr() + 12 * first), nq, K,
                               C.c_void_p(idx.data_ptr()), C.c_void_p(w.data_ptr()), None)
    torch.cuda.synchronize()
    assert r == 0
    assert torch.equal(buf, want_q) and torch.equal(idx, want_idx) and torch.equal(w, want_w)
    assert torch.equal(idx[:n - first, 0].cpu(), torch.arange(first, n, dtype=torch.int32))
