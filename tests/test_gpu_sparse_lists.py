"""Few splats in many groups of bins: a window of group pairs then spans whole views of
groups without any.  The lists against the oracle, and the time of two splats far
apart against two close together (the walk of a window must not pass over the groups
between them one by one)."""
import numpy as np
import pytest

import oracle
from paper_2604_17155_amd import synthetic as syn
from tests import parity, tiny

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bin_size", [16, 32])
@pytest.mark.parametrize("n,views", [(1, 3), (23, 9)])
def test_sparse_lists(n, views, bin_size):
    import torch  # noqa: F401  (before the library: one HIP runtime)
    from paper_2604_17155_amd import gsc
    sc = syn.make_plain(n=n, n_cams=2, res=64)
    sc.cams = syn.hemisphere_cams(views, 3.0, 1031, 709)
    rng = np.random.default_rng(n)
    sc.scales = np.full((n, 3), 0.01, np.float32)
    y = rng.uniform(size=(sc.n_pixels, 3)).astype(np.float32)
    ref = oracle.colorize(sc, y)
    ctx = gsc.Context(bin_size=bin_size)
    geo = gsc.scene_tensors(sc)
    c, st, x = ctx.colorize(*geo, sc.cams, parity.to_device_targets(y), 0, list(sc.lam), extras={"counts"})
    print(parity.check_colorize(c.cpu().numpy(), st.cpu().numpy(), ref, count_gpu=ctx.stats().contributions,
                                cnt_gpu=x["counts"].cpu().numpy(), label=f"{n} in {views} views"), flush=True)
    plan = gsc.Plan(ctx, [(0, n, 0, views)], *geo, list(sc.cams), 3, 0)
    pc, _ = plan.run(parity.to_device_targets(y), list(sc.lam))
    assert plan.info().dropped_pairs == 0
    assert float((pc - c).abs().max()) <= 1e-5 * float(c.abs().max())


def test_time_of_distant_splats():
    import torch
    from paper_2604_17155_amd import gsc
    S = 16384  # 65536 groups of 64 pixels
    cam = tiny.axis_camera(S, S)
    at = lambda px, py: [(px - S / 2) * 4.0 / cam.fx, (py - S / 2) * 4.0 / cam.fx, 0.0]
    y = torch.ones((S * S, 1), dtype=torch.bfloat16, device="cuda")
    ms = {}
    for name, second in (("near", (100.0, 100.0)), ("far", (S - 20.0, S - 20.0))):
        sc = tiny.scene([at(20.0, 20.0), at(*second)], np.full((2, 3), 1e-4), tiny.identity_quats(2), [0.8, 0.8], [cam])
        geo = gsc.scene_tensors(sc)
        ctx = gsc.Context(bin_size=16)
        t = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            c, _ = ctx.colorize(*geo, sc.cams, y, 0, [1e-4])
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        assert bool((c > 0.1).all())
        ms[name] = sorted(t)[3]
    print(ms, flush=True)
    assert ms["far"] <= 2.0 * ms["near"]
