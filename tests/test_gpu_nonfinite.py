"""A Gaussian with non-finite colours or gradients marks the pixel blocks that its
footprint reaches and no others.  Two small splats in different 8x8 blocks of one
16x16 tile, the front one with NaN or infinite values: the other's pixels and
gradients are those of a scene in which the front one's values are zero."""
import numpy as np
import pytest

from tests import tiny

pytestmark = pytest.mark.gpu


def _scene(views):
    cam = tiny.axis_camera(32, 32)
    at = lambda px, py, z: [(px - 16.0) * z / cam.fx, (py - 16.0) * z / cam.fx, z - 4.0]
    means = [at(3.5, 3.5, 3.0), at(11.5, 11.5, 3.5)]  # blocks 0 and 3 of the first tile
    return tiny.scene(means, np.full((2, 3), 1e-3), tiny.identity_quats(2), [0.8, 0.7], [cam] * views)


@pytest.mark.parametrize("bin_size", [16, 32])
@pytest.mark.parametrize("C", [1, 3, 7, 9])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_nonfinite_values_stay_in_their_blocks(bad, C, bin_size):
    import torch
    from paper_2604_17155_amd import gsc
    sc = _scene(1)
    geo = gsc.scene_tensors(sc)
    ctx = gsc.Context(bin_size=bin_size)
    gen = torch.Generator(device="cuda").manual_seed(C)
    rnd = lambda *s: torch.rand(s, generator=gen, device="cuda") + 0.5
    colours, grad = rnd(2, 1, C), rnd(32 * 32, C)
    clean = colours.clone()
    clean[0] = 0.0
    colours[0] = bad
    far = torch.ones((32, 32), dtype=torch.bool, device="cuda")
    far[:8, :8] = False  # the block the front splat reaches
    far = far.reshape(-1)
    img, ref = (ctx.render(*geo, sc.cams, c) for c in (colours, clean))
    # (the other splat's centre pixel holds at least 0.5 Y_0 0.7 = 0.0987)
    assert float(ref[far].abs().max()) > 0.09 and torch.equal(img[far], ref[far])
    go, go_ref = (ctx.render_backward(*geo, sc.cams, c, grad, want_coeffs=False)[1] for c in (colours, clean))
    assert float(go_ref[1]) != 0.0 and torch.equal(go[1], go_ref[1])
    # colorize's adjoint: the front splat's upstream gradient
    y = rnd(32 * 32, C)
    coeffs, _ = ctx.colorize(*geo, sc.cams, y, 0, [1e-4])
    res = [ctx.colorize_backward(*geo, sc.cams, y, 0, [1e-4], coeffs, g) for g in (colours, clean)]
    assert torch.equal(res[0][0][far], res[1][0][far]) and torch.equal(res[0][1][1], res[1][1][1])
