"""Stored-P transforms: the automatic decomposition against the others.

The waves of a workgroup share an order's inputs through LDS.  The order of the
sums does not depend on the tiles per wave, so every decomposition gives the
same bits, and the on-the-fly kernels the same values to rounding (the bound
the repository uses between analysis tilings, 1e-13 of the largest value).  The
shapes have pair and degree counts on both sides of a tile (16) and of a
workgroup (64 to 256), odd latitude counts, and orders of a single degree.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (lmax, mmax, nlat, nphi, fields)
SHAPES = [
    (1, 1, 2, 4, 1), (15, 15, 16, 32, 8), (16, 9, 33, 32, 9), (31, 31, 32, 64, 16), (32, 32, 35, 128, 17),
    (63, 63, 64, 128, 3), (64, 64, 129, 256, 24), (127, 127, 128, 256, 16), (128, 100, 135, 256, 5),
    (255, 255, 257, 512, 16), (300, 299, 301, 1024, 12), (40, 40, 600, 128, 8),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_decompositions_agree(shape):
    from paper_1202_6522_amd.shtn import Plan
    L, M, nlat, nphi, nf = shape
    otf = Plan(L, M, nlat, nphi, device="cuda:0")
    plan = Plan(L, M, nlat, nphi, device="cuda:0")
    plan.set_algorithm("stored")
    gen = torch.Generator(device="cuda:0").manual_seed(sum(shape))
    g = torch.randn((nf, nlat, nphi), dtype=torch.float64, device="cuda:0", generator=gen)
    Q = otf.analys(g)
    calls = (("synth", Q), ("analys", g), ("synth_adj", g), ("analys_adj", Q))
    first = {}
    for name, x in calls:
        first[name] = getattr(plan, name)(x)
        ref = getattr(otf, name)(x)
        assert float((first[name] - ref).abs().max()) <= 1e-13 * float(ref.abs().max()), name
        one = getattr(plan, name)(x[nf - 1])
        assert torch.equal(one, first[name][nf - 1]), name
    for tiles in ((1, 1, 1, 1), (2, 2, 2, 2), (4, 1, 4, 1), (4, 2, 4, 2)):
        plan.set_ptable_tiling(*tiles)
        for name, x in calls:
            assert torch.equal(getattr(plan, name)(x), first[name]), (name, tiles)
