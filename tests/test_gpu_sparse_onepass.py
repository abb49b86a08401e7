"""Sparse preparation in one call against its two phases: the same rows, columns
and values to the last bit, from no jump operator to two, twice on one context (the
second time without growing its workspace); a refused allocation and a null result
end the call with an error, an exception in the allocation reaches the caller, and
the context works afterwards."""
import ctypes

import numpy as np
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


def band(N, offsets, g):
    A = np.zeros((N, N), complex)
    for o in offsets:
        A += np.diag(wl.ginibre(g, 1, N - abs(o))[0], o)
    return A


def arguments(lb, N, P):
    g = wl.rng(N + P)
    H = dcsr(wl.hermitize(band(N, (-1, 0, 1) if N > 2 else (0,), g)))
    Ls = [dcsr(band(N, (1 - p,), g)) for p in range(P)]
    return H, [0.3, 0.2][:P], Ls


def two_phases(lb, ctx, N, H, rates, Ls):
    lib = lb.load()
    M = N * N - 1
    P = len(Ls)
    Hs = lb._csr_struct(*H)
    Lc = (lb._CSR * max(P, 1))(*[lb._csr_struct(*l) for l in Ls])
    r = (ctypes.c_double * max(P, 1))(*rates)
    nnz = ctypes.c_int64()
    assert lib.lindblad_prepare_sparse_count(ctx.handle, N, ctypes.byref(Hs), P, r, Lc, ctypes.byref(nnz)) == 0
    out = [torch.empty(M + 1, dtype=torch.int64, device="cuda"),
           torch.empty(max(nnz.value, 1), dtype=torch.int64, device="cuda"),
           torch.empty(max(nnz.value, 1), dtype=torch.float64, device="cuda"),
           torch.empty(M, dtype=torch.float64, device="cuda")]
    p = [ctypes.c_void_p(t.data_ptr()) for t in out]
    assert lib.lindblad_prepare_sparse_fill(ctx.handle, N, ctypes.byref(Hs), P, r, Lc, nnz.value + 1, *p) == -1
    assert lib.lindblad_prepare_sparse_fill(ctx.handle, N, ctypes.byref(Hs), P, r, Lc, nnz.value, *p) == 0
    return out[0], out[1][:nnz.value], out[2][:nnz.value], out[3]


@pytest.mark.parametrize("N,P", [(2, 0), (2, 1), (3, 2), (40, 0), (65, 1), (130, 2)])
def test_one_call_equals_two_phases(lb, N, P):
    H, rates, Ls = arguments(lb, N, P)
    print("[gpu] sparse one call N=%d P=%d" % (N, P), flush=True)
    with lb.Context(0) as ctx:
        for _ in range(2):
            one = lb.lindblad_prepare_sparse(ctx, N, H, rates, Ls)
            two = two_phases(lb, ctx, N, H, rates, Ls)
            torch.cuda.synchronize()
            for a, b in zip(one, two):
                assert a.shape == b.shape and torch.equal(a, b)


def test_allocation_refused(lb, monkeypatch):
    N = 40
    H, rates, Ls = arguments(lb, N, 1)
    print("[gpu] sparse one call, allocation refused", flush=True)
    with lb.Context(0) as ctx:
        want = lb.lindblad_prepare_sparse(ctx, N, H, rates, Ls)
        lib = lb.load()
        Hs, Lc = lb._csr_struct(*H), (lb._CSR * 1)(lb._csr_struct(*Ls[0]))
        r, nnz = (ctypes.c_double * 1)(*rates), ctypes.c_int64()
        for ret, code in ((1, -3), (0, -1)):  # refused; accepted with null pointers
            cb = lb._SPARSE_ALLOC(lambda user, n, out: ret)
            assert lib.lindblad_prepare_sparse(ctx.handle, N, ctypes.byref(Hs), 1, r, Lc, cb, None,
                                               ctypes.byref(nnz)) == code
        with monkeypatch.context() as m:
            m.setattr(torch, "empty", lambda *a, **k: (_ for _ in ()).throw(MemoryError("none left")))
            with pytest.raises(MemoryError, match="none left"):
                lb.lindblad_prepare_sparse(ctx, N, H, rates, Ls)
        got = lb.lindblad_prepare_sparse(ctx, N, H, rates, Ls)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want, got))
