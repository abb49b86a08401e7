"""Dense preparation against the oracle where its launches change: the smallest
sizes, the edges of the 16 x 16 tiles and of the chunks of eight diagonal
positions, the last size whose assembly is one launch (80) and the first beyond,
with the leading dimension equal to M, one more, and the default.

Tolerance: with g = max|gamma|, h = max|H| every C value is at most 36 g (a
diagonal generator's weights sum to less than 6 in modulus), every partial sum of
at most N of them plus the Hamiltonian's at most S = 40 N g + 2 h, and an element is
the end of a chain of at most 2 N + 20 operations: (2 N + 20) u S with u = 2^-53,
twice for the two sides and twice for the complex products."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("N", [2, 3, 7, 8, 9, 16, 17, 18, 19, 33, 34, 64, 65, 79, 80, 81, 82, 97])
def test_prepare_dense_at_its_edges(lb, oracle, N):
    M = N * N - 1
    P = N * (N - 1) // 2
    g = np.random.default_rng(N)
    A = g.standard_normal((N, N)) + 1j * g.standard_normal((N, N))
    H = (A + A.conj().T) / 2
    W = g.standard_normal((M, 24)) + 1j * g.standard_normal((M, 24))
    gamma = W @ W.conj().T
    gamma = (gamma + gamma.conj().T) / (2 * N)
    rows = np.arange(M)
    if N > 34:
        rows = np.unique(np.concatenate([[0, 1, N - 2, N - 1, P - 1, P, P + 1, 2 * P - 1, 2 * P, M - 2, M - 1],
                                         g.integers(0, 2 * P, 150), g.integers(2 * P, M, 30)]))
    Qo, Ko = oracle.prepare_dense(H, gamma, rows=rows)
    tol = 4 * (2 * N + 20) * 2.0 ** -53 * (40 * N * np.abs(gamma).max() + 2 * np.abs(H).max())
    Hd, Gd = torch.from_numpy(H).cuda(), torch.from_numpy(gamma).cuda()
    for ldq in (M, M + 1, lb.default_ldq(M)):
        print("[gpu] prepare dense N=%d ldq=%d" % (N, ldq), flush=True)
        with lb.Context(0) as ctx:
            Q = torch.full((M, ldq), float("nan"), dtype=torch.float64, device="cuda")
            K = torch.full((M,), float("nan"), dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            lb.lindblad_prepare(ctx, Hd, Gd, ldq=ldq, Q=Q, K=K)
            torch.cuda.synchronize()
            assert not torch.isnan(Q).any() and not Q[:, M:].any()
            assert np.abs(Q[torch.from_numpy(rows).cuda(), :M].cpu().numpy() - Qo).max() <= tol
            assert np.abs(K.cpu().numpy() - Ko).max() <= tol
