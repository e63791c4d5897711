"""Synthesis kernel paths: fields per wave, group and segment edges.

The coefficients of an order are read in groups of 16 degrees (two start
checkpoints of 8) and segments of 32; a call of several fields runs one, two
or four of them per wave.  Each output element sums the same products in the
same order whatever the path, so a call of several fields has to give exactly
the grids of one-field calls; those are compared with the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_1202_6522_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# orders of 1 ... 65 degrees around the group and segment edges (every order
# of a plan has its own length), one and several latitude blocks, and lanes
# that join late (lmax 255 and up)
SHAPES = [(7, 7, 8, 16), (16, 16, 17, 64), (32, 32, 33, 128), (48, 40, 131, 128), (64, 64, 200, 256),
          (255, 255, 256, 512), (383, 300, 400, 1024)]


@pytest.mark.parametrize("shape", SHAPES)
def test_fields_together_equal_fields_alone(shape):
    from paper_1202_6522_amd.shtn import Plan
    L, M, nlat, nphi = shape
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(L + nlat)
    Q = torch.from_numpy(inputs.draw_spectrum(rng, L, M, 1.0, 17)).to(dev)
    plan = Plan(L, M, nlat, nphi, device=dev)
    one = torch.stack([plan.synth(Q[f]) for f in range(17)])
    adj = torch.stack([plan.analys_adj(Q[f]) for f in range(17)])
    for nf in (2, 3, 4, 5, 17):
        assert torch.equal(plan.synth(Q[:nf].contiguous()), one[:nf]), nf
        assert torch.equal(plan.analys_adj(Q[:nf].contiguous()), adj[:nf]), nf
    ref = oracle.synth(Q[:1].cpu().numpy(), L, M, nlat, nphi)
    got = one[:1].cpu().numpy()
    # the parity bar of the repository: 1e-11 up to lmax 255, 1e-10 at 511
    assert np.max(np.abs(got - ref)) <= (1e-11 if L <= 255 else 1e-10) * np.max(np.abs(ref))
    for lp, fw in ((1, 1), (1, 2), (1, 4), (2, 1), (2, 2), (2, 4), (4, 1), (4, 2)):
        plan.set_tiling(lp, 8, fw=fw)
        assert torch.equal(plan.synth(Q), one), (lp, fw)
