"""dL/do of colorize where the launches of many channels add up, against the FP64 oracle at
the same coefficients.  With one Gaussian the fit does not depend on its opacity: the
derivative is 0 but for the rounding of those coefficients.

Constant targets, so that beta^T y and delta nearly agree at every pixel.  Each
launch takes its channels' part of delta: its u = beta^T y - delta is a sum of at most 15
products (16 with one wave a tile) and rounds by at most 16 x 2^-24 of them, and the
running sums are as small as u.  So dL/do is off by at most 1e-6 of the sum of all terms'
sizes, sum_p (w_p / o) sum_c beta_c y_c.  (All of delta in one launch leaves running
sums of that size through the others: 64000 atomics, each off by up to 2^-25 of it.)"""
import numpy as np
import pytest

import oracle
from paper_2604_17155_amd import synthetic as syn
from tests import tiny

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [200, 400])  # 3200 tiles: a wave a block; 6400: a wave a tile
@pytest.mark.parametrize("C", [31, 64])
def test_rounding_between_launches(C, views):
    import torch
    from paper_2604_17155_amd import gsc
    sc = tiny.scene([[0.0, 0.0, 0.0]], [[0.6, 0.6, 0.6]], tiny.identity_quats(1), [0.5],
                    syn.hemisphere_cams(views, 3.0, 64, 64), C=C)
    geo = gsc.scene_tensors(sc)
    y = (0.5 + 0.01 * torch.arange(C, device="cuda", dtype=torch.float32)).expand(sc.n_pixels, C).contiguous()
    ctx = gsc.Context(bin_size=16)
    c, _ = ctx.colorize(*geo, sc.cams, y, 0, [1e-4])
    gt, go = ctx.colorize_backward(*geo, sc.cams, y, 0, [1e-4], c, torch.ones_like(c))
    terms = float((gt.double() * y.double()).sum()) / 0.5
    _, ro = oracle.colorize_backward(sc, y.cpu().numpy(), c.cpu().numpy().astype(np.float64), np.ones((1, 1, C)))
    off = abs(float(go[0]) - float(np.asarray(ro)[0]))
    print(f"{C} channels, {views} views: dL/do {float(go[0]) / terms:.1e} of its terms, off by {off / terms:.1e}", flush=True)
    assert terms > 0 and off <= 1e-6 * terms
