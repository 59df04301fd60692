"""The pass that lists the observed Gaussians: their views' bits by one launch (up to 24
views) or two, words of 64 views, and the zeros of the unobserved ones, short rows and
long.  Against the oracle; the time of the zeros against their bytes, and of many views
against few."""
import numpy as np
import pytest

import oracle
from paper_2604_17155_amd import synthetic as syn
from tests import parity, tiny

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,C,views,n", [(1, 3, 24, 70), (1, 4, 25, 1030), (2, 2, 64, 65), (1, 17, 65, 1),
                                         (3, 5, 130, 64), (2, 3, 3, 2049)])
def test_observed(L, C, views, n):
    import torch
    from paper_2604_17155_amd import gsc
    rng = np.random.default_rng(views)
    m, s, q, o = syn.blob_geometry(rng, n)
    if n > 1:
        o[rng.uniform(size=n) < 0.4] = 0.0  # never observed
    lam = [1e-3 * 2.0 ** k for k in range(L + 1)]
    sc = tiny.scene(m, s, q, o, syn.hemisphere_cams(views, 3.0, 40, 30), sh_deg=L, C=C, lam=lam)
    y = rng.uniform(size=(sc.n_pixels, C)).astype(np.float32)
    ref = oracle.colorize(sc, y)
    geo = gsc.scene_tensors(sc)
    coeffs = torch.full((n, (L + 1) ** 2, C), 7.0, device="cuda")
    c, st = gsc.Context().colorize(*geo, sc.cams, parity.to_device_targets(y), L, list(sc.lam), coeffs=coeffs)
    c, st = c.cpu().numpy(), st.cpu().numpy()
    print(parity.check_colorize(c, st, ref, label=f"L={L} C={C}, {views} views of {n}"), flush=True)
    assert (c[(st & 1) == 1] == 0.0).all() and ((st & 1) == 1)[o == 0.0].all()


def _solve_ms(n, views, res, L, C, observed):
    import torch
    from paper_2604_17155_amd import gsc
    m, s, q, o = (torch.from_numpy(a).cuda() for a in syn.blob_geometry(np.random.default_rng(3), n))
    ctx = gsc.Context(flags=gsc.GSC_FLAG_PROFILE)
    y = torch.ones((views * res * res, C), device="cuda")
    t = []
    for _ in range(9):
        ctx.colorize(m, s, q, o * float(observed), syn.hemisphere_cams(views, 3.0, res, res), y, L, [1e-3] * (L + 1))
        torch.cuda.synchronize()
        t.append(ctx.stats().stage_dict()["solve"])
    return sorted(t)[4]


def test_time_of_unobserved():
    n, row = 300000, 16 * 64
    ms = _solve_ms(n, 2, 16, 3, 64, False)
    print(f"{1e3 * ms:.0f} us for {4e-6 * n * row:.0f} MB", flush=True)
    assert 1e-3 * ms < 4 * n * row / 1e12


def test_time_of_many_views():
    few, many = _solve_ms(4290, 22, 64, 1, 3, True), _solve_ms(4290, 166, 64, 1, 3, True)
    print(f"{1e3 * few:.0f} us for 22 views, {1e3 * many:.0f} us for 166", flush=True)
    assert many <= 2.75 * few
