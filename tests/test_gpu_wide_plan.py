"""Plans of 33 to 64 BF16 channels: an untuned one takes its tiles from a queue past 2048
of them (as a call does) and says so, autotune times the form that an untuned plan runs,
and each gives a call's result."""
import numpy as np
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu


# tiles of a launch: 16 views of 180x180 2304, 14 of them 2016
@pytest.mark.parametrize("views,queue", [(16, 256), (14, 0)])
@pytest.mark.parametrize("C", [33, 64])
def test_wide_plan(C, views, queue):
    import torch
    from paper_2604_17155_amd import gsc
    geo = [torch.from_numpy(a).cuda() for a in syn.blob_geometry(np.random.default_rng(C), 3000)]
    cams = syn.hemisphere_cams(views, 3.0, 180, 180)
    y = torch.rand((views * 180 * 180, C), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda").bfloat16()
    ctx = gsc.Context(bin_size=16)
    ref, st = ctx.colorize(*geo, cams, y, 0, [1e-4])
    plan = gsc.Plan(ctx, [(0, 3000, 0, views)], *geo, cams, C, 0)
    tol = 1e-5 * float(ref.abs().max())
    c, s = plan.run(y, [1e-4])
    info = plan.info()
    assert info.accumulate_variant == 128 + 64 + queue
    assert float((c - ref).abs().max()) <= tol and torch.equal(s, st)
    c, s = plan.autotune(y, [1e-4])
    assert {128 + 64, 256 + 128 + 64} <= set(plan.info().tuned_variant)
    assert float((c - ref).abs().max()) <= tol and torch.equal(s, st)
    c, s = plan.run(y, [1e-4])
    assert float((c - ref).abs().max()) <= tol and torch.equal(s, st)
