"""Analysis of several fields at once (sums on the matrix cores).

Calls of enough fields run a kernel whose units take four or eight fields and
whose waves cover 64 to 256 latitude pairs.  The shapes reach every built
combination, with ragged latitude counts (odd ones among them), orders that end
inside a group of eight degrees, a last group of fields that is not full, and
latitudes that start late.  Each result is compared with one-field calls, which
run the vector kernel: the same products summed in another order, so within the
bound the repository uses between analysis tilings, 1e-13 of the largest value.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (lmax, mmax, nlat, nphi, fields): four or eight fields per unit, pairs per
# lane x waves
SHAPES = [
    (511, 511, 100, 1024, 12),   # four, 1 x 1
    (511, 500, 201, 1024, 12),   # four, 2 x 1
    (511, 511, 512, 1024, 4),    # four, 4 x 1
    (509, 301, 1001, 1024, 4),   # four, 4 x 2
    (300, 300, 2047, 1024, 11),  # four, 4 x 4
    (200, 200, 4096, 512, 4),    # four, 4 x 8
    (127, 127, 128, 256, 115),   # eight, 1 x 1
    (255, 255, 257, 512, 15),    # eight, 2 x 2
    (255, 250, 256, 512, 16),    # eight, 2 x 1
    (301, 301, 999, 1024, 7),    # eight, 2 x 4
    (150, 150, 2048, 512, 8),    # eight, 2 x 8
]


@pytest.mark.parametrize("shape", SHAPES)
def test_fields_together_match_fields_alone(shape):
    from paper_1202_6522_amd.shtn import Plan
    L, M, nlat, nphi, nf = shape
    dev = torch.device("cuda:0")
    plan = Plan(L, M, nlat, nphi, device=dev)
    gen = torch.Generator(device=dev).manual_seed(L + nlat)
    g = torch.randn((nf, nlat, nphi), dtype=torch.float64, device=dev, generator=gen)
    for fn in (plan.analys, plan.synth_adj):
        got = fn(g)
        ref = torch.stack([fn(g[f]) for f in range(nf)])
        err = float((got - ref).abs().max() / ref.abs().max())
        assert err <= 1e-13, (fn.__name__, err)
        assert torch.all(got[:, :L + 1].imag == 0)
        assert torch.equal(fn(g), got)  # the order of the sums is fixed


def test_round_trip_of_many_fields():
    from paper_1202_6522_amd import inputs
    from paper_1202_6522_amd.shtn import Plan
    L = 383
    dev = torch.device("cuda:0")
    plan = Plan(L, L, L + 1, 1024, device=dev)
    Q = inputs.draw_spectrum(np.random.default_rng(L), L, L, 1.5, 16)
    R = plan.analys(plan.synth(torch.from_numpy(Q).to(dev))).cpu().numpy()
    assert np.max(np.abs(R - Q)) <= 1e-10 * np.max(np.abs(Q))
