"""One state of a mid-size system (256 < M <= 4096, Q resident on the chip for all
steps) against the launch-per-stage kernels that a captured graph runs: the same
row sums in the same order, so the same bits, at the edges of its column steps
(128 u), of its rows per wave (4) and workgroup (16) and of its range, with even
and odd leading dimensions; against the oracle; without a step and with one; and
from two threads at once.

Tolerance against the oracle: with u = 2^-53 a stage's row sum is off by at most
(M + 2) u ||Q||_inf max|x|, enters v with weight h, and a step's combination adds
at most 8 u max|v|; n steps grow an error by at most exp(n h ||Q||_inf). Twice
that, one for each side."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


def _system(M, ldq, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    Q = torch.full((M, ldq), float("nan"), dtype=torch.float64, device="cuda")
    Q[:, :M] = torch.randn(M, M, dtype=torch.float64, device="cuda", generator=g) * (0.5 / M ** 0.5)
    Q.diagonal()[:] -= 1.0
    K = torch.randn(M, dtype=torch.float64, device="cuda", generator=g) / M
    V = torch.randn(1, M, dtype=torch.float64, device="cuda", generator=g)
    torch.cuda.synchronize()
    return Q, K, V


@pytest.mark.parametrize("M", [257, 258, 512, 513, 528, 768, 769, 1023, 1025, 1368, 1537, 2049, 2560, 2561, 3073,
                               3585, 4095, 4096, 4097])
@pytest.mark.parametrize("pad", [0, 1, 32])
def test_resident_equals_launch_per_stage(lb, M, pad):
    if pad == 0 and M % 2:
        pad = 3
    Q, K, V = _system(M, M + pad, M)
    print("[gpu] resident M=%d ldq=%d" % (M, M + pad), flush=True)
    with lb.Context(0) as ctx:
        for steps in (1, 2, 5, 6):
            a, b = V.clone(), V.clone()
            lb.lindblad_propagate(ctx, Q, K, a, 1e-2, steps)
            lb.lindblad_propagate_graph(ctx, Q, K, b, 1e-2, steps)
            ctx.sync()
            assert torch.isfinite(a).all()
            assert torch.equal(a, b), (M, steps)
            lb.lindblad_graph_clear(ctx)


@pytest.mark.parametrize("M", [288, 1368, 4095])
def test_resident_matches_oracle(lb, oracle, M):
    n, h = 9, 0.01
    Q, K, V = _system(M, lb.default_ldq(M), 3 * M)
    print("[gpu] resident oracle M=%d" % M, flush=True)
    Qh, Kh, Vh = Q[:, :M].cpu().numpy(), K.cpu().numpy(), V.cpu().numpy()
    with lb.Context(0) as ctx:
        lb.lindblad_propagate(ctx, Q, K, V, h, 0)
        ctx.sync()
        assert np.array_equal(V.cpu().numpy(), Vh)
        lb.lindblad_propagate(ctx, Q, K, V, h, n)
        ctx.sync()
    ref = oracle.rk4_dense(Qh, Kh, Vh, h, n)
    qn = np.abs(Qh).sum(1).max()
    top = max(np.abs(Vh).max(), np.abs(ref).max())
    tol = 2 * np.exp(n * h * qn) * n * 2.0 ** -53 * (h * (M + 2) * qn + 8) * top
    assert np.abs(V.cpu().numpy() - ref).max() <= tol


def test_resident_from_two_threads(lb):
    """Each thread has its stream, context and system; both get what they get alone."""
    sizes, steps, calls = (1368, 2600), 40, 6
    data = [_system(M, lb.default_ldq(M), 11 + M) for M in sizes]
    with lb.Context(0) as ctx:
        want = [lb.lindblad_propagate(ctx, Q, K, V.clone(), 1e-2, steps) for Q, K, V in data]
        ctx.sync()
    print("[gpu] resident two threads", flush=True)
    out, errors = [[], []], []

    def work(i):
        try:
            s = torch.cuda.Stream()
            Q, K, V = data[i]
            with torch.cuda.stream(s), lb.Context(0, s) as ctx:
                for _ in range(calls):
                    out[i].append(lb.lindblad_propagate(ctx, Q, K, V.clone(), 1e-2, steps))
                ctx.sync()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not errors, errors
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(o, want[i]) for o in out[i])
