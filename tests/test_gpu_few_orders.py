"""Synthesis of many fields with few orders: a unit's field groups run on the
XCDs in turn, with the same results."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# orders on both sides of the line and of a multiple of the XCDs, field groups
# that divide by the XCDs and do not
@pytest.mark.parametrize("shape", [(200, 0, 1025, 2, 50), (300, 2, 300, 8, 33), (100, 8, 600, 32, 64), (70, 63, 71, 128, 45),
                                   (70, 64, 71, 256, 45)])
def test_fields_match_single_calls(shape):
    from paper_1202_6522_amd import inputs
    from paper_1202_6522_amd.shtn import Plan
    L, M, nlat, nphi, nf = shape
    rng = inputs.np.random.default_rng(sum(shape))
    plan = Plan(L, M, nlat, nphi, device="cuda:0")
    Q, T = (torch.from_numpy(inputs.draw_spectrum(rng, L, M, 1.5, nf)).to("cuda:0") for _ in range(2))
    g, h = plan.synth(Q), plan.analys_adj(Q)
    v = plan.vec_synth(Q, T)
    for f in range(nf):
        assert torch.equal(g[f], plan.synth(Q[f])) and torch.equal(h[f], plan.analys_adj(Q[f])), f
        assert all(torch.equal(a[f], b) for a, b in zip(v, plan.vec_synth(Q[f], T[f]))), f
