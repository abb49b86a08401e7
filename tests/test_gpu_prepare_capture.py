"""lindblad_prepare on a stream that is being captured is refused before anything is
synchronized or freed: the capture goes on and its graph runs, whether the workspace
would have had to grow or not, below and beyond the one-launch size (N = 80)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1912_01491_amd import workloads as wl  # noqa: E402


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("N,first,check", [(12, None, False), (12, 12, False), (81, None, False), (81, 12, True)])
def test_refused_and_the_capture_goes_on(lb, N, first, check):
    print("[gpu] prepare under capture N=%d after %s" % (N, first), flush=True)
    H, gamma = [torch.from_numpy(x).cuda() for x in wl.random_lindbladian(N, 3)]
    M = N * N - 1
    Q = torch.full((M, lb.default_ldq(M)), 7.0, dtype=torch.float64, device="cuda")
    K = torch.full((M,), 7.0, dtype=torch.float64, device="cuda")
    x = torch.zeros(1000, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s), lb.Context(0, s) as ctx:
        if first:
            a, b = [torch.from_numpy(y).cuda() for y in wl.random_lindbladian(first, 4)]
            lb.lindblad_prepare(ctx, a, b)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            x.add_(1.0)
            with pytest.raises(lb.LindbladError) as e:
                lb.lindblad_prepare(ctx, H, gamma, Q=Q, K=K, check_hermitian=check)
            x.add_(2.0)
        assert e.value.code == -4
        for i in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert (x == 3.0 * (i + 1)).all()
        assert (Q == 7.0).all() and (K == 7.0).all()
        Q1, K1 = lb.lindblad_prepare(ctx, H, gamma, Q=Q, K=K)
        ctx.sync()
        assert torch.isfinite(Q1[:, :M]).all() and torch.isfinite(K1).all() and not (K1 == 7.0).any()
