"""Sparse preparation at the edges of its kernels, against the oracle (normwise
1e-10, the bar of the sparse path): the sort sizes of the pair rows (up to 16,
24, 40 and 64 entries of L^+(F_s)), lists longer than a wavefront and N around
multiples of 64, jump operators with one full column, zero rates, no jump
operators, and CSR input whose columns are unsorted, repeated or out of range."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1912_01491_amd import workloads as wl  # noqa: E402

RTOL = 1e-10


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


def model(kind, N, seed):
    g = wl.rng(seed)
    if kind == "n16":  # tridiagonal H, one jump of one entry per row: 4*3 + 2 entries
        return wl.hermitize(band(N, (-1, 0, 1), g)), [0.3], [band(N, (-1,), g)]
    if kind == "n24":  # pentadiagonal H: 4*5 + 2
        return wl.hermitize(band(N, (-2, -1, 0, 1, 2), g)), [0.3], [band(N, (1,), g)]
    if kind == "n40":  # 4*5 + 2*9
        return wl.hermitize(band(N, (-1, 0, 1), g)), [0.3], [band(N, (-1, 0, 1), g)]
    if kind == "n64":  # 4*5 + 2*9 + 2*9: more than 64 KB of LDS a block
        return wl.hermitize(band(N, (-1, 0, 1), g)), [0.3, 0.2], [band(N, (0, 1, 2), g), band(N, (-1, 0, 1), g)]
    if kind == "column":  # L^+ L is dense in one row and column of A only where x = N//2
        L = np.zeros((N, N), complex)
        L[:, N // 2] = wl.ginibre(g, 1, N)[0]
        return wl.hermitize(band(N, (-1, 0, 1), g)), [0.3], [L]
    if kind == "rates":  # a jump at rate zero next to a traced one
        return np.zeros((N, N), complex), [0.0, 0.4], [band(N, (1,), g), band(N, (0, -1), g)]
    return wl.hermitize(band(N, (-1, 0, 1), g)), [], []


def compare(lb, oracle, H, rates, Ls, csr):
    N = H.shape[0]
    M = N * N - 1
    with lb.Context(0) as ctx:
        rp, col, val, K = [x.cpu().numpy() for x in lb.lindblad_prepare_sparse(ctx, N, csr(H), rates,
                                                                               [csr(L) for L in Ls])]
    rows = np.arange(M) if N <= 16 else np.unique(np.concatenate(
        [np.arange(3), np.linspace(0, M - 1, 97).astype(int), np.arange(M - N + 1, M)]))
    zero = np.zeros((N, N), complex)  # the oracle wants at least one jump operator
    Qo, Ko = oracle.prepare_factored(H, np.array(rates or [0.0]), Ls or [zero], rows)
    Qg = np.zeros_like(Qo)
    for t, r in enumerate(rows):
        c = col[rp[r]:rp[r + 1]]
        assert np.all(np.diff(c) > 0)
        Qg[t, c] = val[rp[r]:rp[r + 1]]
    assert np.all(val != 0.0) and rp[M] == len(val)
    assert np.abs(Qg - Qo).max() <= RTOL * np.abs(Qo).max()
    assert np.abs(K[rows] - Ko).max() <= RTOL * max(np.abs(Ko).max(), np.abs(Qo).max())


@pytest.mark.parametrize("kind", ["n16", "n24", "n40", "n64", "column", "rates", "none"])
@pytest.mark.parametrize("N", [4, 11, 65])
def test_paths(lb, oracle, kind, N):
    if kind == "column" and N > 11:
        pytest.skip("4 N + 2 entries per row exceed the sparse path's limit")
    print("[gpu] sparse paths %s N=%d" % (kind, N), flush=True)
    compare(lb, oracle, *model(kind, N, 7 + N), dcsr)


@pytest.mark.parametrize("N", [64, 129])
def test_dimer_around_wavefronts(lb, oracle, N):
    print("[gpu] sparse paths dimer N=%d" % N, flush=True)
    compare(lb, oracle, *wl.dimer_model(N), dcsr)


def test_unsorted_repeated_columns(lb, oracle):
    """Rows reversed, one entry split into two equal halves, columns -1 and N ignored."""
    N = 12
    H, rates, Ls = model("n24", N, 3)

    def messy(A):
        rp, c, v = wl.to_csr(A)
        rows, cols, vals = [0], [], []
        for i in range(N):
            cc, vv = list(c[rp[i]:rp[i + 1]][::-1]), list(v[rp[i]:rp[i + 1]][::-1])
            if cc:
                vv[0] *= 0.5
                cc, vv = cc + [cc[0], -1, N], vv + [vv[0], 7.0, 8.0]
            cols += cc
            vals += vv
            rows.append(len(cols))
        return (torch.tensor(rows).cuda(), torch.tensor(cols).cuda(),
                torch.tensor(np.array(vals, np.complex128)).cuda())

    print("[gpu] sparse paths messy CSR", flush=True)
    compare(lb, oracle, H, rates, Ls, messy)
