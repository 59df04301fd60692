"""Adjoints of a few splats in large images: tiles without entries read no pixel values
(dL/do alone then takes less time than their bytes would at 8 TB/s), and dL/dy is zero
there whatever the image held."""
import numpy as np
import pytest

import oracle
from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu


def test_time_of_empty_tiles():
    import torch
    from paper_2604_17155_amd import gsc
    geo = [torch.from_numpy(a).cuda() for a in syn.blob_geometry(np.random.default_rng(3), 10)]
    cams = syn.hemisphere_cams(20, 3.0, 1024, 1024)
    C = 16
    y = torch.ones((20 * 1024 * 1024, C), device="cuda")  # 1.34 GB
    co = torch.ones((10, 1, C), device="cuda")
    ctx = gsc.Context(bin_size=16, flags=gsc.GSC_FLAG_PROFILE)
    t = []
    for _ in range(7):
        ctx.render_backward(*geo, cams, co, y, want_coeffs=False)
        torch.cuda.synchronize()
        t.append(ctx.stats().stage_dict()["blend_adjoint"])
    ms = sorted(t)[3]
    print(f"{1e3 * ms:.0f} us, {4e-9 * y.numel() / 8e3 * 1e6:.0f} us to read the images", flush=True)
    assert ms * 1e-3 < 4 * y.numel() / 8e12


# blending options under which no decision at a threshold moves a weight by more than
# about 1e-8 (no alpha floor, no early stop, footprints of six sigma), FP32 sums of few
# terms: relative L2 error at most 1e-4, as in the other adjoint tests
@pytest.mark.parametrize("views", [1, 40])  # a wave a block of few tiles, and a wave a tile
@pytest.mark.parametrize("C", [3, 17])
def test_gradients_of_sparse_scenes(C, views):
    import torch
    from paper_2604_17155_amd import gsc
    rng = np.random.default_rng(C)
    sc = syn.make_plain(n=12, n_cams=1, res=64)
    sc.means, sc.scales, sc.quats, sc.opacities = syn.blob_geometry(rng, 12)
    sc.C = C
    sc.cams = syn.hemisphere_cams(views, 3.0, 250, 230)  # 240 tiles each
    opts = oracle.Options(alpha_min=0.0, t_min=0.0, sigma_cut=6.0)
    y = rng.uniform(size=(sc.n_pixels, C)).astype(np.float32)
    co = rng.uniform(size=(12, 1, C)).astype(np.float32)
    gc = rng.uniform(size=(12, 1, C)).astype(np.float32)
    rt, ro = oracle.colorize_backward(sc, y, co.astype(np.float64), gc.astype(np.float64), opts=opts)
    geo = gsc.scene_tensors(sc)
    ctx = gsc.Context(bin_size=16, alpha_min=0.0, t_min=0.0, sigma_cut=6.0)
    dev = lambda a: torch.from_numpy(a).cuda()
    gt, go = ctx.colorize_backward(*geo, sc.cams, dev(y), 0, list(sc.lam), dev(co), dev(gc))
    gt, go, rt = gt.cpu().numpy(), go.cpu().numpy(), np.asarray(rt).reshape(gt.shape)
    empty = np.abs(rt).max(axis=1) == 0  # pixels that no splat reaches
    assert 0.1 < empty.mean() < 1.0
    assert np.linalg.norm(gt - rt) <= 1e-4 * np.linalg.norm(rt)
    assert np.linalg.norm(go - ro) <= 1e-4 * np.linalg.norm(ro)
    assert np.abs(gt[empty]).max() <= 1e-6 * np.abs(rt).max()
