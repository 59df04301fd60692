"""The matrix-core accumulate of 33 to 64 channels (one block a tile) and the
split layout of sums over views: channel counts around its blocks of 16, both
bin sizes and tile schedules, per-view sums (interleaved rows), lists of zero to
several gathers of 256 entries, images that end inside a block.  The gate is the
oracle's (float64, 1e-4 plus the bound of near-threshold decisions)."""
import numpy as np
import pytest

import oracle
from paper_2604_17155_amd import synthetic as syn
from tests import parity

pytestmark = pytest.mark.gpu


def _scene(C, L, n, width, height):
    sc = syn.make_features(n=n, n_cams=5, width=width, height=height, C=C)
    if L:
        rng = np.random.default_rng(C)
        sc.sh_deg, sc.lam = L, np.array([1e-4 * 4.0 ** k for k in range(L + 1)], np.float32)
        sc.gt = [rng.normal(0.0, 0.2, (n, (L + 1) ** 2, C))]
    return sc


@pytest.mark.parametrize("C,L,n,width,height,bin_size,schedule", [
    (33, 0, 6000, 131, 75, 32, 0), (48, 0, 6000, 131, 75, 16, 1), (49, 1, 4000, 97, 61, 32, 2),
    (64, 0, 20000, 70, 41, 16, 2), (64, 0, 20000, 70, 41, 32, 1), (64, 1, 3000, 64, 64, 32, 0),
    (64, 0, 300, 200, 16, 32, 0), (16, 0, 6000, 131, 75, 32, 0), (32, 0, 6000, 131, 75, 16, 0)])
def test_wide_accumulate(C, L, n, width, height, bin_size, schedule):
    import torch
    from paper_2604_17155_amd import gsc
    sc = _scene(C, L, n, width, height)
    y = oracle.make_targets(sc)
    assert y.dtype == np.uint16
    ref = oracle.colorize(sc, y)
    m, s, q, o = gsc.scene_tensors(sc)
    ctx = gsc.Context(bin_size=bin_size, schedule=schedule)
    c, st, x = ctx.colorize(m, s, q, o, sc.cams, parity.to_device_targets(y), L, list(sc.lam), extras={"counts"})
    label = f"C={C} L={L} n={n} {width}x{height} bin {bin_size} schedule {schedule}"
    print(parity.check_colorize(c.cpu().numpy(), st.cpu().numpy(), ref, tol=1e-4,
                                count_gpu=int(ctx.stats().contributions), cnt_gpu=x["counts"].cpu().numpy(),
                                label=label), flush=True)
    assert torch.isfinite(c).all()
    if L == 0:  # per-view sums kept for the caller: the interleaved layout
        c2, st2, x2 = ctx.colorize(m, s, q, o, sc.cams, parity.to_device_targets(y), L, list(sc.lam),
                                   extras={"view_sums"})
        parity.check_colorize(c2.cpu().numpy(), st2.cpu().numpy(), ref, tol=1e-4, label=label + " view sums")
        assert x2["view_sums"].shape == (len(sc.cams), n, C + 1)
