"""Inputs that are infinite or not a number.

Every kernel that may serve a call gives the same results for them: plans whose
fields fit a workgroup and calls of several fields against the kernels of a set
tiling.  Terms that the polar threshold drops take no part in the sums, whatever
their input.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (lmax, mmax, nlat, nphi, threshold exponent)
CASES = [(31, 31, 32, 64, -200), (31, 31, 32, 64, -20), (15, 15, 63, 32, -4), (40, 12, 24, 32, -3), (24, 20, 2, 64, -2),
         (7, 7, 64, 16, -1),
         (31, 31, 2, 64, -1), (60, 50, 6, 128, -6)]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 1e308])
def test_dropped_terms_stay_dropped(case, bad):
    from paper_1202_6522_amd.shtn import Plan
    shape, polar = case[:4], case[4]
    L, M, nlat, nphi = shape
    one = Plan(*shape, device="cuda:0", polar_log2=polar)
    two = Plan(*shape, device="cuda:0", polar_log2=polar)
    t = two.tiling()
    two.set_tiling(t["synth_lp"], t["analys_lp"], t["analys_waves"], 1, 1, t["split"])
    gen = torch.Generator(device="cuda:0").manual_seed(nlat)
    g = torch.randn((3, nlat, nphi), dtype=torch.float64, device="cuda:0", generator=gen)
    Q = two.analys(g)
    g[0, 0, 1] = bad          # the latitude next to the pole
    g[1, nlat // 2, 2] = bad  # one near the equator
    Q[0, one.lm_index(L, min(M, 5))] = bad
    Q[1, one.lm_index(M, M)] = bad
    for name, x in (("analys", g), ("synth_adj", g), ("synth", Q), ("analys_adj", Q)):
        a, b = (torch.view_as_real(r) if r.is_complex() else r
                for r in (getattr(one, name)(x), getattr(two, name)(x)))
        assert torch.equal(a.isnan(), b.isnan()), name
        assert torch.equal(a.nan_to_num(nan=0.0), b.nan_to_num(nan=0.0)), name


# fields that the matrix-core analysis takes (many coefficients, latitudes and
# fields); pairs past the last one in the last lanes of a wave, and none
@pytest.mark.parametrize("shape", [(255, 255, 300, 512, 13), (255, 255, 256, 512, 16), (400, 300, 401, 1024, 5),
                                   (600, 600, 1201, 2048, 4)])
def test_bad_values_in_several_fields(shape):
    from paper_1202_6522_amd.shtn import Plan
    L, M, nlat, nphi, nf = shape
    plans = [Plan(L, M, nlat, nphi, device="cuda:0") for _ in range(2)]
    t = plans[1].tiling()
    plans[1].set_tiling(t["synth_lp"], t["analys_lp"], t["analys_waves"], 1, 1, t["split"])
    gen = torch.Generator(device="cuda:0").manual_seed(nlat)
    g = torch.randn((nf, nlat, nphi), dtype=torch.float64, device="cuda:0", generator=gen)
    g[0, 0, 1] = float("nan")
    g[1, nlat - 1, 0] = float("inf")
    g[2, nlat // 2, 2] = float("inf")
    for name in ("analys", "synth_adj"):
        a, b = (torch.view_as_real(getattr(p, name)(g)) for p in plans)
        assert torch.equal(a.isfinite(), b.isfinite()), name
        assert bool(a[3:].isfinite().all())
        v, w = ([torch.view_as_real(r) for r in getattr(p, "vec_" + name)(g, g)] for p in plans)
        for a, b in zip(v, w):
            assert torch.equal(a.isfinite(), b.isfinite()), name
