"""Longitude stage over its row lengths and rows per workgroup.

Every row length has kernels of its own, workgroups hold four or eight rows
unless the caller sets them, and batches of mixed lengths run one kernel for
all.  The arithmetic of a row does not depend on any of this, so results are
compared bit for bit; the first of them with the transform of a field whose
grid is known in closed form.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (lmax, mmax, nlat, nphi): nphi = 2 K points per row
SHAPES = [
    (1, 0, 3, 2), (1, 1, 2, 4), (3, 3, 4, 8), (7, 6, 9, 16), (15, 15, 16, 32), (15, 12, 21, 32), (31, 31, 33, 64),
    (63, 60, 65, 128), (127, 127, 131, 256), (200, 180, 211, 512), (255, 250, 257, 1024), (300, 120, 303, 2048),
    (150, 150, 153, 4096), (40, 40, 43, 8192),
]


def _grids(shape, nf):
    gen = torch.Generator(device="cuda:0").manual_seed(sum(shape))
    return torch.randn((nf, shape[2], shape[3]), dtype=torch.float64, device="cuda:0", generator=gen)


@pytest.mark.parametrize("shape", SHAPES)
def test_rows_per_workgroup_do_not_matter(shape):
    from paper_1202_6522_amd.shtn import Plan
    base = Plan(*shape, device="cuda:0")
    t = base.tiling()
    g = _grids(shape, 2)
    Q = base.analys(g)
    s = base.synth(Q)
    for rows in (1, 2, 3, 4, 8, 4096):
        plan = Plan(*shape, device="cuda:0")
        plan.set_tiling(t["synth_lp"], t["analys_lp"], t["analys_waves"], t["fw"], t["m_pairing"], t["split"], rows)
        assert torch.equal(plan.synth(Q), s), rows
        assert torch.equal(plan.analys(g), Q), rows


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[1] >= 1])
def test_known_field(shape):
    # cos(phi + a) sin(theta) is of degree 1 and order 1 alone
    from paper_1202_6522_amd.shtn import Plan
    plan = Plan(*shape, device="cuda:0")
    L, M, nlat, nphi = shape
    x = torch.from_numpy(np.polynomial.legendre.leggauss(nlat)[0][::-1].copy()).to("cuda:0")
    phi = torch.arange(nphi, dtype=torch.float64, device="cuda:0") * (2 * np.pi / nphi)
    g = torch.sqrt(1 - x * x)[:, None] * torch.cos(phi + 0.3)[None, :]
    Q = plan.analys(g)
    # largest of the other coefficients, and the way back, in units of the
    # field's maximum 1: rounding of nodes and sums
    rest = Q.clone()
    rest[L + 1] = 0
    assert float(rest.abs().max()) <= 1e-13
    assert float((plan.synth(Q) - g).abs().max()) <= 1e-12


@pytest.mark.parametrize("shapes", [SHAPES[:-2], SHAPES, SHAPES[2:6]])
def test_mixed_row_lengths(shapes):
    from paper_1202_6522_amd.shtn import Batch, Plan
    grids = [_grids(s, 1)[0] for s in shapes]
    batch = Batch(shapes, device="cuda:0")
    gp = torch.cat([g.reshape(-1) for g in grids])
    Qp = batch.analys(gp)
    sp = batch.synth(Qp)
    for i, s in enumerate(shapes):
        plan = Plan(*s, device="cuda:0")
        Q = plan.analys(grids[i])
        assert torch.equal(Qp[batch.q_off[i] // 2:batch.q_off[i + 1] // 2], Q), s
        assert torch.equal(sp[batch.g_off[i]:batch.g_off[i + 1]], plan.synth(Q).reshape(-1)), s
