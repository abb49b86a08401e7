"""The tile-cache file (LB_TUNE_CACHE) and lindblad_set_tile: a tile that was set stays,
whether the file names the same size or not and before anything else has read it (the
bits of the set tile, at a size that runs a stage in one launch and at one that does
not); the file's tile is reported before it is first used, and used at the size beyond
the one launch."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

STEPS, DT = 2, 0.02


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


@pytest.mark.parametrize("M,B", [(899, 16), (2303, 64)])
def test_set_tile_beats_the_file(lb, monkeypatch, tmp_path, M, B):
    print("[gpu] tile cache M=%d B=%d" % (M, B), flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    Q = torch.zeros(M, lb.default_ldq(M), dtype=torch.float64, device="cuda")
    Q[:, :M] = torch.randn(M, M, dtype=torch.float64, device="cuda", generator=g) * (0.5 / M ** 0.5)
    Q.diagonal()[:] -= 1.0
    K = torch.randn(M, dtype=torch.float64, device="cuda", generator=g) / M
    V = torch.randn(B, M, dtype=torch.float64, device="cuda", generator=g)
    torch.cuda.synchronize()

    def run(prepare):
        out = V.clone()
        with lb.Context(0) as ctx:
            prepare(ctx)
            lb.lindblad_propagate(ctx, Q, K, out, DT, STEPS)
            torch.cuda.synchronize()
        return out

    set_tile = (32, 96, 1)
    monkeypatch.delenv("LB_TUNE_CACHE", raising=False)
    default = run(lambda ctx: None)
    want = run(lambda ctx: lb.lindblad_set_tile(ctx, M, B, *set_tile))
    cached = run(lambda ctx: lb.lindblad_set_tile(ctx, M, B, 32, 160, 2))
    assert not torch.equal(want, default) and not torch.equal(want, cached)
    path = tmp_path / "tiles"
    path.write_text("%d %d 0 32 160 2\n" % (M, 16 if B <= 16 else 64))
    monkeypatch.setenv("LB_TUNE_CACHE", str(path))
    assert torch.equal(run(lambda ctx: lb.lindblad_set_tile(ctx, M, B, *set_tile)), want)

    def look(ctx):
        info = lb.lindblad_tile_info(ctx, M, B)
        assert (info["rows"], info["kslab"], info["waves"], bool(info["tuned"])) == (32, 160, 2, True)

    assert torch.equal(run(look), default if M == 899 else cached)
