"""The slice layout's entries with consecutive columns (one column kept per 64
rows) against the oracle: bands of 1 to 32 entries (every chunk remainder), mixed
with entries at scattered columns, a ragged last slice, one to five states, and a
banded drive matrix.

Tolerance: with u = 2^-53 a stage's row sum of w terms is off by at most (w + 2) u
||Q||_inf max|x|, enters v with weight h, and a step's combination adds at most
8 u max|v|; n steps grow an error by at most exp(n h ||Q||_inf). Twice that, one
for each side."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


def band(M, w, scattered, seed):
    """Rows of w entries: columns from max(0, r - w//2) on (consecutive from row to
    row), the last `scattered` of them at columns without a pattern."""
    g = np.random.default_rng(seed)
    D = np.zeros((M, M))
    for r in range(M):
        c0 = min(max(0, r - w // 2), M - w)
        cols = set(range(c0, c0 + w - scattered))
        while len(cols) < w:
            cols.add(int(g.integers(0, M)))
        D[r, sorted(cols)] = g.standard_normal(w) / w
    return D


def csr(D):
    rp = np.zeros(D.shape[0] + 1, np.int64)
    rp[1:] = np.cumsum((D != 0).sum(1))
    r, c = np.nonzero(D)
    return [torch.from_numpy(x).cuda() for x in (rp, c.astype(np.int64), D[r, c])]


def tol(Q, h, n, w, top):
    qn = np.abs(Q).sum(1).max()
    return 2 * np.exp(n * h * qn) * n * 2.0 ** -53 * (h * (w + 2) * qn + 8) * top


@pytest.mark.parametrize("w", [1, 2, 5, 8, 9, 10, 17, 18, 19, 27, 28, 31, 32])
@pytest.mark.parametrize("scattered,B", [(0, 1), (1, 1), (0, 5)])
def test_bands(lb, oracle, w, scattered, B):
    M, n, h = 3 * 64 + 5, 13, 0.05
    Q = band(M, w, min(scattered, w - 1), 100 + w)
    g = np.random.default_rng(w)
    K, V = g.standard_normal(M) * 0.1, g.standard_normal((B, M))
    print("[gpu] sparse band w=%d scattered=%d B=%d" % (w, scattered, B), flush=True)
    with lb.Context(0) as ctx:
        Vd = torch.from_numpy(V).cuda()
        lb.lindblad_propagate_csr(ctx, *csr(Q), torch.from_numpy(K).cuda(), Vd, h, n)
        ctx.sync()
    ref = oracle.rk4_dense(Q, K, V, h, n)
    assert np.abs(Vd.cpu().numpy() - ref).max() <= tol(Q, h, n, w, max(np.abs(V).max(), np.abs(ref).max()))


@pytest.mark.parametrize("w0,w1", [(18, 1), (7, 9), (4, 40)])
def test_banded_drive(lb, oracle, w0, w1):
    M, n, h = 4 * 64 + 1, 20, 0.01
    Q0, Q1 = band(M, w0, 0, 7), band(M, w1, 0, 8)
    g = np.random.default_rng(9)
    K, V = g.standard_normal(M) * 0.1, g.standard_normal((1, M))
    E, A, T = -1.0, -1.5, 0.2
    print("[gpu] sparse banded drive w0=%d w1=%d" % (w0, w1), flush=True)
    with lb.Context(0) as ctx:
        Vd = torch.from_numpy(V).cuda()
        lb.lindblad_propagate_csr_drive(ctx, csr(Q0), csr(Q1), torch.from_numpy(K).cuda(), Vd, h, n, 0.0, E, A, T)
        ctx.sync()
    ref = oracle.rk4_drive(Q0, Q1, K, V, h, n, 0.0, E, A, T)
    Qa = np.abs(Q0) + 2.5 * np.abs(Q1)
    assert np.abs(Vd.cpu().numpy() - ref).max() <= tol(Qa, h, n, w0 + w1, max(np.abs(V).max(), np.abs(ref).max()))
