"""Group pairs are taken in windows whose size follows their count: from a single splat
(windows of 4 pairs) to thousands (256) in views of several sizes, against the oracle;
and the time of a few splats in many views, which must not exceed that of a hundred
times as many."""
import numpy as np
import pytest

import oracle
from paper_2604_17155_amd import synthetic as syn
from tests import parity

pytestmark = pytest.mark.gpu


# about 1.3 groups a splat and view, 140 groups of 4x4 bins of 16 pixels
@pytest.mark.parametrize("bin_size", [16, 32])
@pytest.mark.parametrize("n", [1, 60, 200, 800, 1600, 6400])
def test_windows(n, bin_size):
    import torch
    from paper_2604_17155_amd import gsc
    sc = syn.make_plain(n=n, n_cams=2, res=64)
    rng = np.random.default_rng(n)
    sc.means, sc.scales, sc.quats, sc.opacities = syn.blob_geometry(rng, n)
    sc.opacities = (0.3 * sc.opacities + 0.004).astype(np.float32)
    sc.cams = syn.hemisphere_cams(5, 3.0, 300, 200) + syn.hemisphere_cams(2, 2.5, 210, 301)
    y = rng.uniform(size=(sc.n_pixels, 3)).astype(np.float32)
    ref = oracle.colorize(sc, y)
    ctx = gsc.Context(bin_size=bin_size)
    geo = gsc.scene_tensors(sc)
    yd = parity.to_device_targets(y)
    c, st, x = ctx.colorize(*geo, sc.cams, yd, 0, list(sc.lam), extras={"counts"})
    stats = ctx.stats()
    print(parity.check_colorize(c.cpu().numpy(), st.cpu().numpy(), ref, count_gpu=stats.contributions,
                                cnt_gpu=x["counts"].cpu().numpy(), label=f"{n} splats, bins {bin_size}"), flush=True)
    plan = gsc.Plan(ctx, [(0, n, 0, len(sc.cams))], *geo, list(sc.cams), 3, 0)
    pc, ps = plan.run(yd, list(sc.lam))
    info = plan.info()
    assert info.dropped_pairs == 0 and info.pair_capacity == stats.pairs
    assert info.contributions == stats.contributions and torch.equal(ps, st)
    assert float((pc - c).abs().max()) <= 1e-5 * float(c.abs().max())


def test_time_of_few_splats():
    import torch
    from paper_2604_17155_amd import gsc
    cams = syn.hemisphere_cams(20, 3.0, 512, 512)
    y = torch.ones((20 * 512 * 512, 1), device="cuda")
    us = {}
    for n in (10, 1000):
        geo = [torch.from_numpy(a).cuda() for a in syn.blob_geometry(np.random.default_rng(3), n)]
        ctx = gsc.Context()
        t = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ctx.colorize(*geo, cams, y, 0, [1e-4])
            b.record()
            b.synchronize()
            t.append(1e3 * a.elapsed_time(b))
        us[n] = sorted(t)[7]
    print(us, flush=True)
    assert us[10] <= us[1000]
