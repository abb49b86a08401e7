"""One long-row state alone (two rows a wave from M = 9000 on, one before) against the
same system four times in one launch (four rows a wave): the same bits."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("M,ldq", [(8999, 9024), (9000, 9024), (9001, 9002), (9024, 9024)])
def test_rows_per_wave(lb, M, ldq):
    print("[gpu] gemv rows M=%d ldq=%d" % (M, ldq), flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    Q = torch.zeros(M, ldq, dtype=torch.float64, device="cuda")
    Q[:, :M] = torch.randn(M, M, dtype=torch.float64, device="cuda", generator=g) * (0.5 / M ** 0.5)
    K = torch.randn(M, dtype=torch.float64, device="cuda", generator=g) / M
    V = torch.randn(1, M, dtype=torch.float64, device="cuda", generator=g)
    one, four = V.clone(), [V.clone() for _ in range(4)]
    torch.cuda.synchronize()
    with lb.Context(0) as ctx:
        lb.lindblad_propagate(ctx, Q, K, one, 0.01, 2)
        lb.lindblad_propagate_batched(ctx, [Q] * 4, [K] * 4, four, 0.01, 2)
        torch.cuda.synchronize()
    assert torch.isfinite(one).all() and not torch.equal(one, V)
    assert all(torch.equal(one, f) for f in four)
