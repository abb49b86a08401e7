"""Blocks of states on the default tiles at the edges of their rule (row tiles of
16 below M = 3000, 32 below 8200, 64 beyond; slabs from one to nine; remainders of
a slab of fewer than 16 and 32 columns), FP64 and FP32, against the oracle; and
states that share a call with others keep their bits.

Tolerance: with u = 2^-53 (2^-24 for FP32, whose rounding of Q adds as much again)
a stage's row sum is off by at most (M + 2) u ||Q||_inf max|x|, enters v
with weight h, and a step's combination adds at most 8 * 2^-53 max|v|; n steps grow
an error by at most exp(n h ||Q||_inf). Twice that, one for each side."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("M", [65, 129, 257, 304, 640, 2499, 2500, 2999, 3000, 3001, 8199, 8200])
@pytest.mark.parametrize("B,fp32", [(2, False), (17, False), (64, False), (3, True), (32, True), (50, True)])
def test_default_tiles_match_oracle(lb, oracle, M, B, fp32):
    if not fp32 and M <= 256 and B * M <= 4096:
        pytest.skip("the one-workgroup path")
    n, h = 2, 0.01
    g = np.random.default_rng(M + B)
    Q = g.standard_normal((M, M))
    Q /= np.abs(Q).sum(1).max()
    if fp32:
        Q = Q.astype(np.float32).astype(np.float64)
    K, V = g.standard_normal(M) * 0.1, g.standard_normal((B, M))
    print("[gpu] tiles M=%d B=%d fp32=%d" % (M, B, fp32), flush=True)
    Qd = torch.zeros(M, lb.default_ldq(M), dtype=torch.float32 if fp32 else torch.float64, device="cuda")
    Qd[:, :M] = torch.from_numpy(Q).cuda().to(Qd.dtype)
    Kd, Vd = torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda()
    prec = lb.FP32 if fp32 else lb.FP64
    args = (None if fp32 else Qd, Kd)
    with lb.Context(0) as ctx:
        out = lb.lindblad_propagate(ctx, *args, Vd.clone(), h, n, prec, Qd if fp32 else None)
        two = lb.lindblad_propagate(ctx, *args, Vd[:2].clone(), h, n, prec, Qd if fp32 else None)
        ctx.sync()
        # padded to the same 16 states: the same slabs, the same bits
        if B <= 16:
            assert torch.equal(two, out[:2])
    ref = oracle.rk4_dense(Q, K, V, h, n)
    top = max(np.abs(V).max(), np.abs(ref).max())
    u = 2.0 ** -24 if fp32 else 2.0 ** -53
    tol = 2 * np.exp(n * h) * n * (h * 2 * (M + 2) * u + 8 * 2.0 ** -53) * top
    assert np.abs(out.cpu().numpy() - ref).max() <= tol
