"""A plan whose geometry has grown since it was made, until its (group, item) pairs
pass 32 bits: the run drops what does not fit, says so and stays in its buffers, and
the plan gives its first result again once the geometry is back."""
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu

# 255 groups a view.  Nine tenths of the Gaussians grow over all of them; the rest stay
# small and lie behind, so that a view's items end with some thousand blocks of them.
# The pairs pass 2^32 within the third view: 2 x 0.9 N x 255 lie below, 3 x above.
N, W, H, VIEWS = 8_450_000, 960, 1088, 3
GROW = 9 * N // 10


def test_pairs_past_32_bits():
    import torch
    from paper_2604_17155_amd import gsc
    assert 2 * GROW * 255 + VIEWS * 4 * N < 2 ** 32 < 3 * GROW * 255
    cam = syn.look_at((0.0, -3.0, 0.0), W, H, 50.0, up=(0.0, 0.0, 1.0))
    gen = torch.Generator(device="cuda").manual_seed(4)
    m = 0.8 * torch.rand((N, 3), generator=gen, device="cuda") - 0.4
    m[GROW:, 1] += 0.8  # depth is y + 3
    s = torch.full((N, 3), 2e-4, device="cuda")
    q = torch.zeros((N, 4), device="cuda")
    q[:, 0] = 1.0
    o = torch.full((N,), 0.05, device="cuda")
    y = torch.rand((W * H, 1), generator=gen, device="cuda")
    ctx = gsc.Context(bin_size=16, batch_items=2 ** 26)
    plan = gsc.Plan(ctx, [(0, N, 0, VIEWS)], m, s, q, o, [cam] * VIEWS, 1, 0, offsets=[0] * VIEWS)
    first, _ = plan.run(y, [1e-4])
    info = plan.info()
    assert info.batches == 1 and info.dropped_pairs == 0 and info.contributions > 0
    s[:GROW] = 100.0
    grown, _ = plan.run(y, [1e-4])
    assert plan.info().dropped_pairs > 0 and bool(grown.isfinite().all())
    s.fill_(2e-4)
    again, _ = plan.run(y, [1e-4])
    assert plan.info().dropped_pairs == 0
    # sums of at most a few hundred pixels a Gaussian, added in another order
    assert float((again - first).abs().max()) <= 1e-4 * float(first.abs().max())
