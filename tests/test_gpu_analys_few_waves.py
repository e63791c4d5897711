"""Analysis of several fields whose units are too few for the matrix-core kernel.

Such calls run the vector kernel, with the bits of a set tiling (one field per
wave)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1023, 40, 1024, 128, 4), (300, 200, 1000, 512, 4), (511, 200, 512, 512, 4),
                                   (1023, 10, 1024, 32, 12), (1023, 20, 1024, 64, 8)])
def test_vector_kernel_is_taken(shape):
    from paper_1202_6522_amd.shtn import Plan
    L, M, nlat, nphi, nf = shape
    plan, vec = (Plan(L, M, nlat, nphi, device="cuda:0") for _ in range(2))
    t = vec.tiling()
    vec.set_tiling(t["synth_lp"], t["analys_lp"], t["analys_waves"], 1, 1, t["split"])
    gen = torch.Generator(device="cuda:0").manual_seed(sum(shape))
    g = torch.randn((nf, nlat, nphi), dtype=torch.float64, device="cuda:0", generator=gen)
    assert torch.equal(plan.analys(g), vec.analys(g))
    assert torch.equal(plan.synth_adj(g), vec.synth_adj(g))
