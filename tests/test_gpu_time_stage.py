"""lindblad_time_stage times what propagate runs: its figure, times the stages of a run,
is no more than twice the run's own time and no less than a third of it (the other
kernels of a stage, launches and the load of Q make up the rest), for one state held on
the chip, blocks whose stage is one launch, one and several systems, and larger ones;
and it leaves the states as they are."""
import time

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

STEPS = 150


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("M,B,R", [(1368, 1, 1), (4095, 1, 1), (4900, 1, 1), (899, 16, 2), (2048, 64, 1), (2700, 20, 3),
                                   (3599, 16, 1)])
def test_time_is_that_of_the_run(lb, M, B, R):
    print("[gpu] time stage M=%d B=%d R=%d" % (M, B, R), flush=True)
    ldq = lb.default_ldq(M)
    Qs = [torch.zeros(M, ldq, dtype=torch.float64, device="cuda") for _ in range(R)]
    for Q in Qs:
        Q.diagonal()[:] = -1.0
    Ks = [torch.ones(M, dtype=torch.float64, device="cuda") for _ in range(R)]
    Vs = [torch.ones(B, M, dtype=torch.float64, device="cuda") for _ in range(R)]
    torch.cuda.synchronize()
    with lb.Context(0) as ctx:
        lb.lindblad_time_stage(ctx, Qs, Ks, Vs, iters=20)
        ms = min(lb.lindblad_time_stage(ctx, Qs, Ks, Vs, iters=20) for _ in range(3))
        assert all((v == 1.0).all() for v in Vs)
        best = 1e9
        for _ in range(4):
            ctx.sync()
            t0 = time.perf_counter()
            lb.lindblad_propagate_batched(ctx, Qs, Ks, Vs, 1e-3, STEPS)
            ctx.sync()
            best = min(best, time.perf_counter() - t0)
    run = best * 1e3 / (4 * STEPS)
    print("[gpu] stage %.4f ms, run %.4f ms a stage" % (ms, run), flush=True)
    assert run / 3 <= ms <= 2 * run
