"""Blocks of states of a small FP64 system, a stage in one launch, against the two
launches that a tile set by hand uses and against the oracle: M at the edges of the 16
rows of a workgroup, of the eight waves' columns (multiples of 64) and of their steps
of 8 and 32 columns, the largest sizes of each number of states and the next ones,
even, odd and minimal leading dimensions (with NaN beyond M), states that fill their
tiles or not; and one system alone, in a batch of three, from a graph and from the
allocation-free call give the same bits.

Tolerance: with u = 2^-53 a stage's row sum is off by at most (M + 2) u ||Q||_inf
max|x|, enters v with weight h, and n steps grow an error by at most
exp(n h ||Q||_inf); twice for the two sides."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

STEPS, DT = 3, 0.02


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


def system(M, ldq, B, seed):
    g = np.random.default_rng(seed)
    Q = g.standard_normal((M, M)) * (0.5 / M ** 0.5) - np.eye(M)
    Qd = torch.full((M, ldq), float("nan"), dtype=torch.float64, device="cuda")
    Qd[:, :M] = torch.from_numpy(Q)
    K, V = g.standard_normal(M) / M, g.standard_normal((B, M))
    return Q, K, V, Qd, torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda()


def bound(Q, V):
    M = Q.shape[0]
    norm = np.abs(Q).sum(1).max()
    return 2 * 4 * STEPS * DT * (M + 2) * 2.0 ** -53 * norm * np.abs(V).max() * np.exp(STEPS * DT * norm)


@pytest.mark.parametrize("M,B", [(65, 64), (72, 64), (80, 60), (127, 40), (128, 64), (255, 17), (257, 2), (287, 5), (288, 16), (289, 17), (319, 32), (320, 33),
                                 (321, 64), (511, 3), (513, 20), (1023, 64), (2047, 40), (2048, 64), (2049, 64),
                                 (2703, 16), (2704, 32), (2705, 9)])
@pytest.mark.parametrize("pad", [0, 1, 2])
def test_whole_stage(lb, oracle, M, B, pad):
    Q, K, V, Qd, Kd, Vd = system(M, M + pad, B, M + B)
    print("[gpu] whole stage M=%d ldq=%d B=%d" % (M, M + pad, B), flush=True)
    a, b = Vd.clone(), Vd.clone()
    torch.cuda.synchronize()
    with lb.Context(0) as ctx:
        lb.lindblad_propagate(ctx, Qd, Kd, a, DT, STEPS)
    with lb.Context(0) as ctx:
        lb.lindblad_set_tile(ctx, M, B, 16, 64, 1)
        lb.lindblad_propagate(ctx, Qd, Kd, b, DT, STEPS)
    torch.cuda.synchronize()
    tol = bound(Q, V)
    assert torch.isfinite(a).all() and (a - b).abs().max().item() <= tol
    if pad == 0:
        assert np.abs(a.cpu().numpy() - oracle.rk4_dense(Q, K, V, DT, STEPS)).max() <= tol


@pytest.mark.parametrize("M,B", [(289, 3), (1025, 32), (2048, 64), (2704, 16)])
def test_same_bits_every_way(lb, M, B):
    print("[gpu] whole stage M=%d B=%d: batch, graph, noalloc" % (M, B), flush=True)
    Q, K, V, Qd, Kd, Vd = system(M, lb.default_ldq(M), B, M)
    Qd[:, M:] = 0
    ways = [Vd.clone() for _ in range(4)]
    extra = [Vd.flip(0).contiguous(), Vd * 0.5]
    torch.cuda.synchronize()
    with lb.Context(0) as ctx:
        lb.lindblad_propagate(ctx, Qd, Kd, ways[0], DT, STEPS)
        lb.lindblad_propagate_batched(ctx, [Qd] * 3, [Kd] * 3, [extra[0], ways[1], extra[1]], DT, STEPS)
        lb.lindblad_propagate_graph(ctx, Qd, Kd, ways[2], DT, STEPS)
        ctx.sync()
        lb.lindblad_propagate_noalloc(ctx, Qd, Kd, ways[3], DT, STEPS)
        torch.cuda.synchronize()
    assert not torch.equal(ways[0], Vd)
    assert all(torch.equal(ways[0], w) for w in ways[1:])
    assert torch.equal(extra[0].flip(0), ways[0])
