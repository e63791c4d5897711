"""Transforms of plans so small that a field is one workgroup.

Both stages then run in one launch, with the steps and sums of the two kernels
that larger plans, tilings set by the caller and batches run, so the results
are the same bits.  The shapes have lane groups of 16 and 32 pairs, full and
not, odd latitude counts, every row length, orders longer than a segment of 32
degrees, latitudes that start late, and plans on both sides of the limits.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (lmax, mmax, nlat, nphi, fields)
SHAPES = [
    (7, 7, 8, 16, 1), (7, 4, 9, 16, 3), (7, 7, 64, 16, 2), (15, 15, 16, 32, 1), (15, 15, 63, 32, 5), (20, 20, 33, 64, 1),
    (31, 31, 31, 64, 2), (31, 31, 32, 64, 1), (31, 31, 32, 64, 70), (31, 31, 33, 64, 1), (40, 20, 41, 64, 2),
    (31, 12, 32, 128, 1), (100, 7, 60, 16, 2), (70, 15, 64, 32, 1), (7, 7, 65, 16, 1),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_one_launch_matches_two(shape):
    from paper_1202_6522_amd.shtn import Plan
    L, M, nlat, nphi, nf = shape
    one = Plan(L, M, nlat, nphi, device="cuda:0")
    two = Plan(L, M, nlat, nphi, device="cuda:0")
    t = two.tiling()
    two.set_tiling(t["synth_lp"], t["analys_lp"], t["analys_waves"], 1, t["m_pairing"], t["split"])
    gen = torch.Generator(device="cuda:0").manual_seed(sum(shape))
    g = torch.randn((nf, nlat, nphi), dtype=torch.float64, device="cuda:0", generator=gen)
    Q = two.analys(g)
    for name, x in (("analys", g), ("synth_adj", g), ("synth", Q), ("analys_adj", Q)):
        assert torch.equal(getattr(one, name)(x), getattr(two, name)(x)), name


def test_captured_and_replayed():
    from paper_1202_6522_amd.shtn import Plan
    plan = Plan(31, device="cuda:0")
    Q = plan.analys(torch.randn((2, 32, 64), dtype=torch.float64, device="cuda:0"))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        plan.analys(plan.synth(Q))
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            grid = plan.synth(Q)
            back = plan.analys(grid)
    torch.cuda.synchronize()
    for k in range(3):
        Q.mul_(1.5)
        graph.replay()
        torch.cuda.synchronize()
        want = plan.synth(Q)
        assert torch.equal(grid, want) and torch.equal(back, plan.analys(want)), k
