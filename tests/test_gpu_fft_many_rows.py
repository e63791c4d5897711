"""Calls of very many short rows: more of them per FFT workgroup, the same bits."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (lmax, mmax, nlat, nphi, fields): row lengths 1 to 64 complex points, rows per
# workgroup from the first step past eight to the most, latitudes that fill the
# last workgroup and do not
SHAPES = [
    (3, 0, 1000, 2, 40), (3, 0, 4096, 2, 130), (2, 1, 333, 4, 500), (5, 3, 130, 8, 900), (40, 3, 1025, 8, 70),
    (9, 7, 513, 16, 200), (20, 15, 700, 32, 60), (31, 31, 99, 64, 1000), (63, 63, 64, 128, 600),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_many_rows_match_few(shape):
    from paper_1202_6522_amd.shtn import Batch, Plan
    L, M, nlat, nphi, nf = shape
    plan = Plan(L, M, nlat, nphi, device="cuda:0")
    t = plan.tiling()
    gen = torch.Generator(device="cuda:0").manual_seed(sum(shape))
    g = torch.randn((nf, nlat, nphi), dtype=torch.float64, device="cuda:0", generator=gen)
    few = Plan(L, M, nlat, nphi, device="cuda:0")
    few.set_tiling(t["synth_lp"], t["analys_lp"], t["analys_waves"], 1, 1, t["split"], t["fft_rows"])
    Q = few.analys(g)
    s = few.synth(Q)
    assert torch.equal(plan.synth(Q), s)
    assert torch.equal(plan.synth_adj(g), few.synth_adj(g))
    assert torch.equal(plan.analys(g), Q)
    batch = Batch([(L, M, nlat, nphi)] * nf, device="cuda:0")
    assert torch.equal(batch.synth(torch.view_as_real(Q).reshape(-1).view(torch.complex128)), s.reshape(-1))
    assert torch.equal(batch.analys(g.reshape(-1)).reshape(nf, -1), Q)
