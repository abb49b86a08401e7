"""Blocks of states of many small FP64 systems: where there are workgroups enough, or
the systems' Q exceed the last-level cache, a workgroup takes two tiles of 16 rows
instead of one. Every system then has the bits it has alone (one tile), at rows that
fill the second tile, reach into it or end before it, with even and odd leading
dimensions, for each padded number of states; and the tile path's row rule of several
systems keeps the bits of one (M = 2808: rows of 16 alone, of 32 in a batch).

No tolerance: the sums are formed in the same order."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

STEPS, DT = 2, 0.02


@pytest.fixture(scope="module")
def lb():
    import paper_1912_01491_amd as lb
    lb.load()
    return lb


# 64 states: two tiles from 769 workgroups of 16 rows on. 2 to 32 states: from 256 MB of Q on.
@pytest.mark.parametrize("M,B,R,pad", [(65, 64, 160, 3), (72, 60, 154, 0), (80, 64, 154, 0), (96, 50, 129, 1),
                                       (255, 33, 49, 1), (1599, 64, 8, 1), (2048, 40, 6, 0), (2048, 40, 7, 0),
                                       (1599, 16, 14, 1), (2033, 2, 9, 3), (2704, 32, 5, 0), (2695, 17, 5, 2),
                                       (2808, 16, 3, 8), (2808, 64, 2, 8), (2115, 64, 3, 13), (2915, 32, 2, 13)])
def test_batch_has_the_bits_of_one(lb, M, B, R, pad):
    print("[gpu] block rows M=%d B=%d R=%d" % (M, B, R), flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + B)
    ldq = M + pad
    Qs, Ks, Vs = [], [], []
    for _ in range(R):
        Q = torch.full((M, ldq), float("nan"), dtype=torch.float64, device="cuda")
        Q[:, :M] = torch.randn(M, M, dtype=torch.float64, device="cuda", generator=g) * (0.5 / M ** 0.5)
        Q.diagonal()[:] -= 1.0
        Qs.append(Q)
        Ks.append(torch.randn(M, dtype=torch.float64, device="cuda", generator=g) / M)
        Vs.append(torch.randn(B, M, dtype=torch.float64, device="cuda", generator=g))
    out = [v.clone() for v in Vs]
    torch.cuda.synchronize()
    with lb.Context(0) as ctx:
        lb.lindblad_propagate_batched(ctx, Qs, Ks, out, DT, STEPS)
        for r in sorted({0, 1, R // 2, R - 1}):
            one = Vs[r].clone()
            torch.cuda.synchronize()
            lb.lindblad_propagate(ctx, Qs[r], Ks[r], one, DT, STEPS)
            ctx.sync()
            assert torch.isfinite(one).all() and not torch.equal(one, Vs[r])
            assert torch.equal(out[r], one), r


# 2 to 32 states, M > 2048, more than 512 workgroups of 32 rows and 256 MB of Q: the tile GEMM, a slab
# for each wave of the one launch. Whole and partial last slabs, rows and columns; the fewest systems.
@pytest.mark.parametrize("M,B,R,pad", [(2049, 16, 8, 15), (2115, 16, 8, 13), (2176, 2, 8, 0), (2208, 9, 8, 1),
                                       (2303, 32, 8, 1), (2305, 17, 8, 3), (2600, 16, 7, 2), (2704, 32, 7, 16)])
def test_many_large_systems_have_the_bits_of_one(lb, M, B, R, pad):
    assert R * ((M + 31) // 32) > 512 and R * M * (M + pad) * 8 > 256 << 20
    test_batch_has_the_bits_of_one(lb, M, B, R, pad)
