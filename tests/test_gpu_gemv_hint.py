"""One state of a system that fits the last-level cache against two of them in one
batch that together do not (the rows are then read with the nontemporal hint): the
same bits, at 5104 and 5120 rows (rows of whole 128-byte lines) and with unaligned
rows, where the hint is never used."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("M,ldq", [(5120, 5120), (5104, 5120), (5120, 5121)])
def test_batch_beyond_the_cache_equals_single(lb, M, ldq):
    print("[gpu] gemv hint M=%d ldq=%d" % (M, ldq), flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + ldq)
    Q, K, V = [], [], []
    for _ in range(2):
        q = torch.zeros(M, ldq, dtype=torch.float64, device="cuda")
        q[:, :M] = torch.randn(M, M, dtype=torch.float64, device="cuda", generator=g) * (0.5 / M ** 0.5)
        Q.append(q)
        K.append(torch.randn(M, dtype=torch.float64, device="cuda", generator=g) / M)
        V.append(torch.randn(1, M, dtype=torch.float64, device="cuda", generator=g))
    one, two = [v.clone() for v in V], [v.clone() for v in V]
    torch.cuda.synchronize()
    with lb.Context(0) as ctx:
        lb.lindblad_propagate_batched(ctx, Q, K, two, 0.01, 3)
        for r in range(2):
            lb.lindblad_propagate(ctx, Q[r], K[r], one[r], 0.01, 3)
        torch.cuda.synchronize()
    assert torch.isfinite(two[0]).all() and not torch.equal(two[0], V[0])
    assert all(torch.equal(a, b) for a, b in zip(one, two))
