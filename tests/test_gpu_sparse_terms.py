"""Pair rows whose entries are kept as terms (more than 24 of them) against the oracle
(normwise 1e-10, the bar of the sparse path): several jump operators, complex ones,
some at rate zero or without an entry between them, lists of the largest width that
the bound of 64 entries allows, and rows around multiples of 64."""
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


def model(kind, N):
    g = wl.rng(N)
    H = wl.hermitize(band(N, (-1, 0, 1), g))
    if kind == "many":  # 4*3 + 2*10: ten operators of one entry per row
        return H, [0.1 * (p + 1) for p in range(10)], [band(N, (p % 3 - 1,), g) for p in range(10)]
    if kind == "gaps":  # operators that add nothing before, between and after those that do
        Z = np.zeros((N, N), complex)
        return H, [0.3, 0.0, 0.2, 0.1, 0.5], [Z, band(N, (1,), g), band(N, (-1, 1), g), Z, band(N, (-1, 0), g)]
    if kind == "wide":  # one operator of four entries per row: G has 7 diagonals, 4*7 + 2*16
        return np.zeros((N, N), complex), [0.4], [band(N, (-1, 0, 1, 2), g)]
    return wl.hermitize(band(N, (-7, -5, -3, -1, 0, 1, 3, 5, 7), g)), [], []  # 4*9 entries of A alone


@pytest.mark.parametrize("kind", ["many", "gaps", "wide", "none"])
@pytest.mark.parametrize("N", [12, 23, 65])
def test_terms(lb, oracle, kind, N):
    print("[gpu] sparse terms %s N=%d" % (kind, N), flush=True)
    H, rates, Ls = model(kind, N)
    M = N * N - 1
    with lb.Context(0) as ctx:
        rp, col, val, K = [x.cpu().numpy() for x in lb.lindblad_prepare_sparse(ctx, N, dcsr(H), rates,
                                                                               [dcsr(L) for L in Ls])]
    use = [(r, L) for r, L in zip(rates, Ls) if r] or [(0.0, np.zeros((N, N), complex))]
    Qo, Ko = oracle.prepare_factored(H, [r for r, _ in use], [L for _, L in use], np.arange(M))[:2]
    Q = np.zeros((M, M))
    for s in range(M):
        assert np.all(np.diff(col[rp[s]:rp[s + 1]]) > 0)
        Q[s, col[rp[s]:rp[s + 1]]] = val[rp[s]:rp[s + 1]]
    assert np.abs(Q - Qo).max() <= 1e-10 * np.abs(Qo).max()
    assert np.abs(K - Ko).max() <= 1e-10 * max(np.abs(Ko).max(), 1e-3)
