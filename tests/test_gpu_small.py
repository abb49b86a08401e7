"""The one-workgroup-per-state RK4 (M <= 256, B M <= 4096) against the oracle at
the edges of its column chunks (16), row tiles (64), kernels (64, 128, 192, 256
rows) and state limit, with odd leading dimensions and Q on an 8-byte boundary;
a state's result does not depend on the states and systems that share its call.

Tolerance: with u = 2^-53 a stage's row sum is off by at most (M + 2) u ||Q||_inf
max|x|, enters v with weight h, and a step's combination adds at most 8 u max|v|;
n steps grow an error by at most exp(n h ||Q||_inf). Twice that, one for each
side."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


def _problem(M, B, seed):
    g = np.random.default_rng(seed)
    Q = g.standard_normal((M, M)) * (0.7 / np.sqrt(M)) - np.eye(M)
    K = g.standard_normal(M) / M
    V = g.standard_normal((B, M))
    return Q, K, V


def _device_q(Q, ldq, shift):
    """Q with leading dimension ldq, starting `shift` doubles past an allocation; NaN around it."""
    M = Q.shape[0]
    buf = torch.full((shift + M * ldq + 8,), float("nan"), dtype=torch.float64, device="cuda")
    view = buf[shift:shift + M * ldq].view(M, ldq)
    view[:, :M] = torch.from_numpy(Q).cuda()
    return buf, view


@pytest.mark.parametrize("M,B", [(3, 1), (8, 64), (15, 2), (16, 5), (17, 1), (48, 3), (63, 16), (64, 64), (65, 1),
                                 (80, 51), (127, 4), (128, 32), (129, 1), (143, 17), (191, 2), (192, 21), (193, 1),
                                 (224, 18), (255, 16), (256, 1), (256, 16)])
@pytest.mark.parametrize("pad,shift", [(0, 0), (1, 1), (32, 0)])
def test_small_matches_oracle(lb, oracle, M, B, pad, shift):
    n, h = 23, 0.02
    Q, K, V = _problem(M, B, 1000 * M + B)
    print("[gpu] small M=%d B=%d pad=%d shift=%d" % (M, B, pad, shift), flush=True)
    buf, Qd = _device_q(Q, M + pad, shift)
    with lb.Context(0) as ctx:
        Vd = torch.from_numpy(V).cuda()
        lb.lindblad_propagate(ctx, Qd, torch.from_numpy(K).cuda(), Vd, h, n)
        ctx.sync()
        one = torch.from_numpy(V[B - 1:]).cuda()
        lb.lindblad_propagate(ctx, Qd, torch.from_numpy(K).cuda(), one, h, n)
        ctx.sync()
    assert torch.equal(one[0], Vd[B - 1])  # alone or with B - 1 others: the same bits
    ref = oracle.rk4_dense(Q, K, V, h, n)
    qn = np.abs(Q).sum(1).max()
    top = max(np.abs(V).max(), np.abs(ref).max())
    tol = 2 * np.exp(n * h * qn) * n * 2.0 ** -53 * (h * (M + 2) * qn + 8) * top
    assert np.abs(Vd.cpu().numpy() - ref).max() <= tol


@pytest.mark.parametrize("M,R", [(63, 3), (224, 2)])
def test_small_batched_equals_alone(lb, M, R):
    n, h, B = 11, 0.02, 3
    probs = [_problem(M, B, 7 * M + r) for r in range(R)]
    qs = [_device_q(Q, M, 0)[1].clone() for Q, _, _ in probs]
    ks = [torch.from_numpy(K).cuda() for _, K, _ in probs]
    vs = [torch.from_numpy(V).cuda() for _, _, V in probs]
    print("[gpu] small batched M=%d R=%d" % (M, R), flush=True)
    with lb.Context(0) as ctx:
        alone = [lb.lindblad_propagate(ctx, q, k, v.clone(), h, n) for q, k, v in zip(qs, ks, vs)]
        lb.lindblad_propagate_batched(ctx, qs, ks, vs, h, n)
        ctx.sync()
    for a, v in zip(alone, vs):
        assert torch.equal(a, v)
