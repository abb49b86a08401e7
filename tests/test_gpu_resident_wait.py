"""The one-state integration with Q on the chip (256 < M <= 4096) where it does not
get the chip: its workgroups leave before they start (a wait of 0 for the chip), or at
the first wait for each other (0 there), or find a part of the chip held by another
stream for longer than they wait; and with the allocation-free call. V has the bits of
the launch-per-stage kernels every time; and a context that does not try at all has
them too. M: one workgroup more than a multiple of 16 rows, ragged, the largest, even
and odd leading dimensions.

None of these needs a tolerance: every way forms the same sums in the same order."""
import threading

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

STEPS, DT = 6, 1e-2


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


def _system(M, ldq, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    Q = torch.zeros((M, ldq), dtype=torch.float64, device="cuda")
    Q[:, :M] = torch.randn(M, M, dtype=torch.float64, device="cuda", generator=g) * (0.5 / M ** 0.5)
    Q.diagonal()[:] -= 1.0
    K = torch.randn(M, dtype=torch.float64, device="cuda", generator=g) / M
    V = torch.randn(1, M, dtype=torch.float64, device="cuda", generator=g)
    torch.cuda.synchronize()
    return Q, K, V


@pytest.mark.parametrize("M,pad", [(257, 1), (512, 0), (899, 3), (1368, 8), (2047, 1), (2049, 31), (3599, 1), (4095, 1),
                                   (4096, 0)])
def test_leaving_gives_the_same_bits(lb, M, pad):
    Q, K, V = _system(M, M + pad, M)
    with lb.Context(0) as ctx:
        want = V.clone()
        lb.lindblad_propagate_graph(ctx, Q, K, want, DT, STEPS)
        ctx.sync()
        assert torch.isfinite(want).all() and not torch.equal(want, V)
        for start, stage in ((0.0, 2000.0), (1000.0, 0.0), (0.0, 0.0), (-1.0, 2000.0), (2.0, 2000.0)):
            print("[gpu] resident M=%d waits %g / %g ms" % (M, start, stage), flush=True)
            lb.lindblad_set_resident_wait(ctx, start, stage)
            for call in (lb.lindblad_propagate, lb.lindblad_propagate_noalloc):
                for _ in range(2):
                    got = V.clone()
                    call(ctx, Q, K, got, DT, STEPS)
                    ctx.sync()
                    assert torch.equal(got, want), (M, start, stage, call.__name__)


def test_chip_held_by_another_stream(lb):
    """64 compute units run another context's small system for longer than the wait for the chip; a run of
    M = 4095, which needs all of them, comes out as on the idle chip."""
    Q, K, V = _system(4095, 4096, 5)
    q, k, v = _system(63, 64, 6)
    states = v.repeat(64, 1).contiguous()
    with lb.Context(0) as ctx:
        want = lb.lindblad_propagate(ctx, Q, K, V.clone(), DT, STEPS)
        ctx.sync()
    other = torch.cuda.Stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    print("[gpu] resident beside a kernel that holds compute units", flush=True)
    with torch.cuda.stream(other), lb.Context(0, other) as ctx:
        lb.lindblad_propagate(ctx, q, k, states, 1e-6, 10)
        e0.record()
        lb.lindblad_propagate(ctx, q, k, states, 1e-6, 60000)  # 0.2 us a stage: about 50 ms
        e1.record()
        mine = torch.cuda.Stream()
        with torch.cuda.stream(mine), lb.Context(0, mine) as me:
            got = [lb.lindblad_propagate(me, Q, K, V.clone(), DT, STEPS) for _ in range(4)]
            me.sync()
        ctx.sync()
    torch.cuda.synchronize()
    assert e0.elapsed_time(e1) > 10.0  # longer than the wait for the chip (2 ms)
    assert all(torch.equal(g, want) for g in got)


@pytest.mark.parametrize("steps", [4096, 4097, 8195])
def test_long_runs_in_pieces(lb, steps):
    """One piece, two and three: on the chip, left at once, and a launch per stage."""
    Q, K, V = _system(300, 300, 8)
    out = []
    print("[gpu] resident %d steps" % steps, flush=True)
    with lb.Context(0) as ctx:
        for start in (2.0, 0.0, -1.0):
            lb.lindblad_set_resident_wait(ctx, start)
            out.append(lb.lindblad_propagate(ctx, Q, K, V.clone(), 1e-3, steps))
            ctx.sync()
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


@pytest.mark.parametrize("M,threads", [(288, 8), (1368, 6), (2600, 4)])
def test_many_threads(lb, M, threads):
    """Side by side where they fit on the chip, one after the other or leaving where not."""
    steps, calls = 20, 8
    data = [_system(M, lb.default_ldq(M), 31 + i) for i in range(threads)]
    with lb.Context(0) as ctx:
        want = [lb.lindblad_propagate(ctx, Q, K, V.clone(), DT, steps) for Q, K, V in data]
        ctx.sync()
    print("[gpu] resident M=%d from %d threads" % (M, threads), flush=True)
    out, errors = [[] for _ in data], []

    def work(i):
        try:
            s = torch.cuda.Stream()
            Q, K, V = data[i]
            with torch.cuda.stream(s), lb.Context(0, s) as ctx:
                for _ in range(calls):
                    out[i].append(lb.lindblad_propagate(ctx, Q, K, V.clone(), DT, steps))
                ctx.sync()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(threads)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not errors, errors
    torch.cuda.synchronize()
    for i in range(threads):
        assert len(out[i]) == calls and all(torch.equal(o, want[i]) for o in out[i])


def test_allocation_free_call_allocates_nothing(lb):
    """One state, M = 2303: the first resident run of a process may come through this call."""
    Q, K, V = _system(2303, 2304, 9)
    with lb.Context(0) as ctx, lb.Context(0) as fresh:
        a, b = V.clone(), V.clone()
        torch.cuda.synchronize()
        lb.lindblad_propagate_noalloc(ctx, Q, K, a, DT, STEPS)  # loads every kernel once
        ctx.sync()
        free = torch.cuda.mem_get_info()[0]
        lb.lindblad_propagate_noalloc(fresh, Q, K, b, DT, STEPS)
        fresh.sync()
        assert torch.cuda.mem_get_info()[0] == free
        assert torch.equal(a, b)


def test_bad_waits_are_refused(lb):
    with lb.Context(0) as ctx:
        for start, stage in ((float("nan"), 1.0), (1.0, float("nan")), (1.0, -1.0), (1e10, 1.0), (1.0, 1e10)):
            with pytest.raises(lb.LindbladError):
                lb.lindblad_set_resident_wait(ctx, start, stage)


@pytest.mark.parametrize("M,start,stage", [(899, 0.0, 2000.0), (899, 1000.0, 0.0), (4095, 0.0, 0.0)])
def test_stage_time_of_runs_that_leave(lb, M, start, stage):
    """Where the timed runs leave, a launch per stage is timed: no less than a read of Q from the
    last-level cache at 20 TB/s, more than it delivers, takes, and no more than 1 ms (V as it was)."""
    print("[gpu] stage time of runs that leave M=%d" % M, flush=True)
    Q, K, V = _system(M, lb.default_ldq(M), M)
    with lb.Context(0) as ctx:
        lb.lindblad_set_resident_wait(ctx, start, stage)
        v = V.clone()
        for _ in range(3):
            ms = lb.lindblad_time_stage(ctx, [Q], [K], [v], iters=20)
            assert 8e3 * M * M / 20e12 < ms < 1.0
        assert torch.equal(v, V)
