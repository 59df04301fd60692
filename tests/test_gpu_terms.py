"""Per-item colours and adjoint terms: block edges (127..129 Gaussians), sets of
four views with a remainder, channel counts whose coefficients fit the staging
area at once or in several parts, every degree.

The oracle runs in float64 with the smooth options (no thresholds), so what
differs is FP32 rounding: weights to about 1e-5 of the largest at these depths
(the exponent's argument carries a few ulps at |q| < 18), terms to NB 2^-24.
With one Gaussian every weight is linear in its opacity, so the fit does not
depend on it and d/do of colorize is exactly zero: no relative error there."""
import numpy as np
import pytest

import oracle
from tests import tiny

pytestmark = pytest.mark.gpu
SMOOTH = dict(alpha_min=0.0, t_min=0.0, sigma_cut=6.0)
TOL = 1e-4


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("L,C,views,n", [(0, 7, 1, 5), (3, 3, 5, 127), (3, 20, 9, 129), (2, 12, 4, 128),
                                         (1, 33, 3, 300), (3, 7, 2, 1), (2, 5, 6, 513)])
def test_terms_against_oracle(L, C, views, n):
    import torch
    from paper_2604_17155_amd import gsc
    rng = np.random.default_rng(100 * L + C)
    lam = [1e-3 * 2.0 ** k for k in range(L + 1)]
    sc = tiny.random_scene(3 + n, n=n, n_cams=views, sh_deg=L, C=C, lam=lam)
    c = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
    gi = rng.standard_normal((sc.n_pixels, C)).astype(np.float32)
    y = rng.random((sc.n_pixels, C), dtype=np.float32)
    opts = oracle.Options(**SMOOTH)
    ctx = gsc.Context(**SMOOTH)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    m, s, q, o = gsc.scene_tensors(sc)
    out = {}
    out["images"] = (ctx.render(m, s, q, o, sc.cams, dev(c)), oracle.render(sc, c.astype(np.float64), opts=opts))
    g = ctx.render_backward(m, s, q, o, sc.cams, dev(c), dev(gi))
    r = oracle.render_backward(sc, c.astype(np.float64), gi.astype(np.float64), opts=opts)
    out["render d/dc"], out["render d/do"] = (g[0], r[0]), (g[1], r[1])
    fit = oracle.colorize(sc, y, opts=opts)["coeffs"].astype(np.float32)
    g = ctx.colorize_backward(m, s, q, o, sc.cams, dev(y), L, list(sc.lam), dev(fit), dev(c))
    r = oracle.colorize_backward(sc, y, fit.astype(np.float64), c.astype(np.float64), opts=opts)
    out["colorize d/dy"] = (g[0], r[0])
    if n > 1:
        out["colorize d/do"] = (g[1], r[1])
    errs = {k: _rel(a.cpu().numpy().astype(np.float64).reshape(b.shape), b) for k, (a, b) in out.items()}
    print(f"L={L} C={C} {views} views of {n}: " + ", ".join(f"{k} {e:.1e}" for k, e in errs.items()), flush=True)
    assert max(errs.values()) <= TOL
