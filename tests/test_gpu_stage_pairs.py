"""The stage combination in row pairs, where M is odd (the last row has no partner) and
even, where the state tiles are full and padded, in FP64 and FP32 and for systems in
one launch: two batches of the same states in another order and another padding give
the same bits, every state agrees with the oracle, and nothing leaks from the padding
(buffers that held NaN before).

Tolerance: FP64 as a chain of sums, u = 2^-53: a stage's row sum is off by at most
(M + 2) u ||Q||_inf max|x|, n steps grow it by at most exp(n h ||Q||_inf), twice for
the two sides. FP32: u = 2^-24 for the products and sums within a slab."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("M", [288, 289, 303, 304, 305, 1025])
@pytest.mark.parametrize("B", [2, 15, 16, 17, 33, 64])
@pytest.mark.parametrize("fp32", [False, True])
def test_row_pairs(lb, oracle, M, B, fp32):
    print("[gpu] stage pairs M=%d B=%d fp32=%d" % (M, B, fp32), flush=True)
    steps, dt = 2, 0.02
    g = np.random.default_rng(M + B)
    Q = g.standard_normal((M, M)) * (0.5 / M ** 0.5) - np.eye(M)
    K = g.standard_normal(M) / M
    V = g.standard_normal((B, M))
    if fp32:
        Q = Q.astype(np.float32).astype(np.float64)
    want = oracle.rk4_dense(Q, K, V, dt, steps)
    ldq = lb.default_ldq(M)
    Qd = torch.zeros(M, ldq, dtype=torch.float64, device="cuda")
    Qd[:, :M] = torch.from_numpy(Q)
    Kd = torch.from_numpy(K).cuda()
    junk = torch.full((1 << 22,), float("nan"), dtype=torch.float64, device="cuda")
    del junk
    torch.cuda.empty_cache()
    with lb.Context(0) as ctx:
        Q32 = lb.lindblad_q_to_f32(ctx, Qd) if fp32 else None
        prec = lb.FP32 if fp32 else lb.FP64
        a = torch.from_numpy(V).cuda()
        b = torch.from_numpy(V[::-1].copy()).cuda()
        torch.cuda.synchronize()
        lb.lindblad_propagate(ctx, Qd, Kd, a, dt, steps, prec, Q32)
        lb.lindblad_propagate(ctx, Qd, Kd, b, dt, steps, prec, Q32)
        torch.cuda.synchronize()
    assert torch.equal(a, b.flip(0))
    norm = np.abs(Q).sum(1).max()
    u = 2.0 ** (-24 if fp32 else -53)
    tol = 2 * 4 * steps * dt * (M + 2) * u * norm * np.abs(V).max() * np.exp(steps * dt * norm)
    assert np.abs(a.cpu().numpy() - want).max() <= tol
