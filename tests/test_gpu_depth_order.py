"""Depth order of a view's items at the sizes where the sort changes form (one
block in LDS up to 4096 and 24576 items, tiles of 2048 and 8192 keys, segments
of more than 64 tiles), with many equal depths (ties go to the lower index),
culled items among them, and views of different sizes in one batch.  A wrong
order shows in the contribution counts and coefficients, which are compared
with the oracle's for every Gaussian."""
import numpy as np
import pytest

import oracle
from paper_2604_17155_amd import synthetic as syn
from tests import parity

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    sc = syn.make_plain(n=max(n, 2), n_cams=1, res=16)
    rng = np.random.default_rng(seed)
    means, scales, quats, opac = syn.blob_geometry(rng, n)
    # depths along the cameras' axes on a coarse grid; some behind a camera
    means[:, :] = np.round(means * 8.0) / 8.0 + np.float32(0.01) * rng.integers(0, 3, size=(n, 3))
    means[rng.random(n) < 0.02, 0] = 4.0
    opac[rng.random(n) < 0.02] = 0.001  # below the alpha floor
    if n > 30000:  # faint enough that pixels stay open through the list
        opac = (0.06 * opac + 0.004).astype(np.float32)
    sc.means, sc.scales, sc.quats, sc.opacities = means.astype(np.float32), scales, quats, opac.astype(np.float32)
    sc.cams = [syn.look_at((3.0, 0.0, 0.0), 24, 20), syn.look_at((0.5, 2.5, 1.0), 19, 23)]
    return sc, rng.uniform(0.0, 1.0, size=(sc.n_pixels, 3)).astype(np.float32)


@pytest.mark.parametrize("n", [1, 63, 4096, 4097, 24576, 24577, 140_001, 530_001])
def test_order_of_one_scene(n):
    import torch
    from paper_2604_17155_amd import gsc
    sc, y = _scene(n, n)
    ref = oracle.colorize(sc, y)
    ctx = gsc.Context()
    c, st, x = ctx.colorize(*gsc.scene_tensors(sc), sc.cams, parity.to_device_targets(y), 0, list(sc.lam),
                            extras={"counts"})
    print(parity.check_colorize(c.cpu().numpy(), st.cpu().numpy(), ref, cnt_gpu=x["counts"].cpu().numpy(),
                                label=f"{n} Gaussians"), flush=True)


@pytest.mark.parametrize("sizes", [(900, 4100, 17), (30_000, 1200, 150_000)])
def test_order_of_uneven_scenes(sizes):
    import torch
    from paper_2604_17155_amd import gsc
    parts = [_scene(n, n + 1) for n in sizes]
    table, cams, g0 = [], [], 0
    for sc, _ in parts:
        table.append((g0, sc.N, len(cams), len(sc.cams)))
        cams += list(sc.cams)
        g0 += sc.N
    cat = lambda f: torch.from_numpy(np.ascontiguousarray(np.concatenate([getattr(sc, f) for sc, _ in parts]))).cuda()
    geo = [cat(f) for f in ("means", "scales", "quats", "opacities")]
    ctx = gsc.Context()
    plan = gsc.Plan(ctx, table, *geo, cams, 3, 0)
    c, st = plan.run(parity.to_device_targets(np.concatenate([y for _, y in parts])), list(parts[0][0].lam))
    assert plan.info().dropped_pairs == 0 and plan.info().batches == 1
    for (sc, y), (g, n, _, _) in zip(parts, table):
        print(parity.check_colorize(c[g:g + n].cpu().numpy(), st[g:g + n].cpu().numpy(), oracle.colorize(sc, y),
                                    label=f"plan, {n} Gaussians"), flush=True)
