"""The diagonals' lists of the sparse preparation where their space is reserved from the
operators' widths and where their number is read back first (a jump operator with a
full column makes the widths' bound useless): N on both sides, twice on one context,
sampled rows and K against the oracle (normwise 1e-10, the bar of the sparse path)."""
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


@pytest.mark.parametrize("N,full", [(2, True), (3, True), (60, True), (399, True), (405, True), (405, False)])
def test_lists(lb, oracle, N, full):
    print("[gpu] sparse lists N=%d full=%d" % (N, full), flush=True)
    g = wl.rng(N)
    A = np.diag(wl.ginibre(g, 1, N)[0]) + np.diag(wl.ginibre(g, 1, N - 1)[0], 1)
    H = wl.hermitize(A)
    L = np.zeros((N, N), complex)
    if full:
        L[:, N // 2] = wl.ginibre(g, 1, N)[0]
    else:
        L += np.diag(wl.ginibre(g, 1, N - 1)[0], -1)
    M, P = N * N - 1, N * (N - 1) // 2
    rows = np.unique(np.concatenate([[0, P - 1, P, 2 * P - 1, 2 * P, M - 1], g.integers(0, M, 8)]))
    Qo, Ko = oracle.prepare_factored(H, [0.2], [L], rows)
    with lb.Context(0) as ctx:
        for _ in range(2):
            rp, col, val, K = [x.cpu().numpy() for x in lb.lindblad_prepare_sparse(ctx, N, dcsr(H), [0.2], [dcsr(L)])]
            Q = np.zeros((len(rows), M))
            for i, s in enumerate(rows):
                Q[i, col[rp[s]:rp[s + 1]]] = val[rp[s]:rp[s + 1]]
            assert np.abs(Q - Qo).max() <= 1e-10 * np.abs(Qo).max()
            assert np.abs(K[rows] - Ko).max() <= 1e-10 * max(np.abs(Ko).max(), 1e-3)
