"""Batches of fields whose latitudes take several waves per order: the bits of
one-field calls, wherever a unit stands in the batch's list."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(60, 60, 1500, 128), (100, 70, 2047, 256), (40, 40, 2500, 128), (63, 63, 4096, 128), (31, 31, 32, 64)]


def test_batch_matches_plans():
    from paper_1202_6522_amd.shtn import Batch, Plan
    batch = Batch(SHAPES + SHAPES[::-1], device="cuda:0")
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    g = torch.randn(batch.g_off[-1], dtype=torch.float64, device="cuda:0", generator=gen)
    Q = batch.analys(g)
    s = batch.synth(Q)
    for i, shape in enumerate(batch.shapes):
        plan = Plan(*shape, device="cuda:0")
        q = Q[batch.q_off[i] // 2:batch.q_off[i + 1] // 2]
        assert torch.equal(q, plan.analys(g[batch.g_off[i]:batch.g_off[i + 1]].reshape(shape[2:]))), shape
        assert torch.equal(s[batch.g_off[i]:batch.g_off[i + 1]], plan.synth(q).reshape(-1)), shape
