"""set_tiling with what an untouched plan or batch reports: the same launches."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _launches(call):
    from paper_1202_6522_amd import shtn as S
    S.shtn_profile_reset()
    S.shtn_profile_enable(True)
    out = call()
    n = [S.shtn_profile_read(k)[1] for k in (1, 2, 3, 4)]
    S.shtn_profile_enable(False)
    return n, out


def _same(a, b):
    a, b = (x if isinstance(x, tuple) else (x,) for x in (a, b))
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("shape", [(31, 31, 32, 64, 1), (255, 255, 256, 512, 16)])
def test_plan(shape):
    from paper_1202_6522_amd.shtn import Plan
    ref, plan = (Plan(*shape[:4], device="cuda:0") for _ in range(2))
    t = plan.tiling()
    plan.set_tiling(**dict(t, m_pairing=1))
    other = plan.tiling()
    assert other == dict(t, m_pairing=1)
    plan.set_tiling(**t)
    assert plan.tiling() == t
    g = torch.randn((shape[4], shape[2], shape[3]), dtype=torch.float64, device="cuda:0")
    Q = ref.analys(g)
    for call in (lambda p: p.analys(g), lambda p: p.synth(Q), lambda p: p.vec_analys(g, g), lambda p: p.vec_synth(Q, Q)):
        (n, a), (m, b) = _launches(lambda: call(ref)), _launches(lambda: call(plan))
        assert n == m and _same(a, b)


# decompositions next to the reported one, which the kernels of one direction
# take as they are set
@pytest.mark.parametrize("tiles", [(4, 2, 4, 2), (4, 2, 1, 1), (1, 1, 4, 2)])
@pytest.mark.parametrize("nf", [1, 9, 24])
def test_stored_table(tiles, nf):
    from paper_1202_6522_amd.shtn import Plan
    ref, plan = (Plan(100, 90, 103, 256, device="cuda:0") for _ in range(2))
    plan.set_ptable_tiling(1, 2, 2, 1)
    plan.set_ptable_tiling(*tiles)
    for p in (ref, plan):
        p.set_algorithm("stored")
    gen = torch.Generator(device="cuda:0").manual_seed(nf)
    g = torch.randn((nf, 103, 256), dtype=torch.float64, device="cuda:0", generator=gen)
    Q = ref.analys(g)
    assert torch.equal(plan.analys(g), Q)
    assert torch.equal(plan.synth(Q), ref.synth(Q))


def test_batch():
    from paper_1202_6522_amd.shtn import Batch
    shapes = [(63, 63, 64, 128)] * 5 + [(40, 30, 41, 64)] * 2
    b = Batch(shapes, device="cuda:0")
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    g = torch.randn(b.g_off[-1], dtype=torch.float64, device="cuda:0", generator=gen)
    Q = b.analys(g)
    s = b.synth(Q)
    t = b.tiling()
    b.set_tiling(2, 4, 1, 1)
    b.set_tiling(**t)
    assert b.tiling() == t == dict(synth_lp=1, fw=1, m_pairing=0, analys_merge=0)
    assert torch.equal(b.analys(g), Q) and torch.equal(b.synth(Q), s)
