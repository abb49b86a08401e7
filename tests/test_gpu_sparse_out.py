"""Sparse preparation into arrays that start on a 16-byte boundary (entries stored in
pairs) and 8 bytes past one (one by one): the same columns and values to the last bit,
and nothing written before or behind them, for rows of few and of many entries."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1912_01491_amd import workloads as wl  # noqa: E402


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


def dcsr(A):
    return tuple(torch.from_numpy(x).cuda() for x in wl.to_csr(A))


@pytest.mark.parametrize("rocked", [False, True])
@pytest.mark.parametrize("N", [2, 3, 33, 130])
@pytest.mark.parametrize("dc,dv", [(2, 2), (3, 2), (2, 3), (3, 3)])
def test_alignment_of_the_arrays(lb, N, rocked, dc, dv):
    print("[gpu] sparse out N=%d rocked=%d offsets %d %d" % (N, rocked, dc, dv), flush=True)
    if rocked:
        H, _, rates, Ls = wl.rocked_dimer_model(N)
    else:
        H, rates, Ls = wl.dimer_model(N)
    M = N * N - 1
    H, Ls = dcsr(H), [dcsr(L) for L in Ls]
    with lb.Context(0) as ctx:
        rp, col, val, K = lb.lindblad_prepare_sparse(ctx, N, H, rates, Ls)
        n = len(col)
        c = torch.full((n + 6,), -7, dtype=torch.int64, device="cuda")
        v = torch.full((n + 6,), -7.0, dtype=torch.float64, device="cuda")
        r, k = torch.empty_like(rp), torch.empty_like(K)
        P = len(Ls)
        rc = lb.load().lindblad_prepare_sparse_fill(
            ctx.handle, N, ctypes.byref(lb._csr_struct(*H)), P, (ctypes.c_double * max(P, 1))(*[float(x) for x in rates]),
            (lb._CSR * max(P, 1))(*[lb._csr_struct(*L) for L in Ls]), n, ctypes.c_void_p(r.data_ptr()),
            ctypes.c_void_p(c.data_ptr() + 8 * dc), ctypes.c_void_p(v.data_ptr() + 8 * dv), ctypes.c_void_p(k.data_ptr()))
        torch.cuda.synchronize()
    assert rc == 0
    assert torch.equal(r, rp) and torch.equal(c[dc:dc + n], col) and torch.equal(v[dv:dv + n], val)
    assert torch.equal(k, K)
    for x, d in ((c, dc), (v, dv)):
        assert (x[:d] == -7).all() and (x[d + n:] == -7).all()
