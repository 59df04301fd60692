"""Needles of 300 to 900 pixels sigma: the ellipse that the binning walks is the one
that the blend tests, so no pixel inside it is lost at a needle's ends.  The early
stop is off, so a Gaussian's count is its own.  It lies between two numbers found
here on the record formed in binary64: the pixels that pass the blend's binary32
test, and those of them in the 8x8 blocks that hold a pixel whose exact q is at most
9, all of which have to be listed (other blocks' pixels pass by the rounding of their
q alone, and may or may not be).
A conic coefficient within the binary64 rounding of a binary32 tie moves all of a
needle's q: the rounding is 2^-53 times the cancellation of the determinant, 7e5
here, so 8e-11 relative against 6e-8 or more between ties; three coefficients of 160
needles make at most 1.3 such needles likely, and more than 4 with 1%."""
import numpy as np
import pytest

from tests import tiny

pytestmark = pytest.mark.gpu

N, W, H = 160, 3001, 2603
K = -0.72134752044448170368
F = np.float32


def _fma(x, y, z):
    return (x.astype(np.float64) * y.astype(np.float64) + z.astype(np.float64)).astype(F)


def _scene():
    rng = np.random.default_rng(2)
    cam = tiny.axis_camera(W, H)
    z = 4.0
    px = rng.uniform([0.3 * W, 0.3 * H], [0.7 * W, 0.7 * H], size=(N, 2))
    means = np.concatenate([(px - [W / 2, H / 2]) * z / cam.fx, np.zeros((N, 1))], axis=1)
    scales = np.full((N, 3), 1e-4)
    scales[:, 0] = np.exp(rng.uniform(np.log(300.0), np.log(900.0), N)) * z / cam.fx
    # at least 10 degrees off the image axes: a row then crosses 2 * 10 pixels at most
    th = np.radians(rng.uniform(10.0, 80.0, N)) + np.pi / 2 * rng.integers(0, 2, N)
    quats = np.stack([np.cos(th / 2), 0 * th, 0 * th, np.sin(th / 2)], axis=1)
    return tiny.scene(means, scales, quats, np.full(N, 0.5), [cam]), cam


def _records(sc, cam):
    m, s, q = (a.astype(np.float64) for a in (sc.means, sc.scales, sc.quats))
    q = q / np.linalg.norm(q, axis=1, keepdims=True)
    w, x, y, z = q.T
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                  2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                  2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], axis=1).reshape(-1, 3, 3)
    S = np.einsum("nij,nj,nkj->nik", R, s * s, R)
    t = m + np.asarray(cam.t, np.float64)  # the camera looks along +z
    iz, fx = 1.0 / t[:, 2], float(F(cam.fx))
    J = np.zeros((N, 2, 3))
    J[:, 0, 0] = J[:, 1, 1] = fx * iz
    J[:, 0, 2], J[:, 1, 2] = -fx * t[:, 0] * iz * iz, -fx * t[:, 1] * iz * iz
    P = np.einsum("nai,nij,nbj->nab", J, S, J)
    sxx, sxy, syy = P[:, 0, 0] + float(F(0.3)), P[:, 0, 1], P[:, 1, 1] + float(F(0.3))
    inv = 1.0 / (sxx * syy - sxy * sxy)
    u, v = fx * t[:, 0] * iz + float(F(cam.cx)), fx * t[:, 1] * iz + float(F(cam.cy))
    return u, v, np.stack([K * syy * inv, -2.0 * K * sxy * inv, K * sxx * inv], axis=1).astype(F)


def _counts(u, v, conic):
    """Pixels of one record inside by the blend's test, and those of them in the
    blocks that have to be listed."""
    c0, c1, c2 = (float(c) for c in conic)
    ys = np.arange(H)[:, None]
    mid = u - 0.5 * c1 / c0 * (ys + 0.5 - v)  # the middle of the needle in the row
    xs = np.floor(mid).astype(np.int64) + np.arange(-14, 15)[None, :]

    def offset(p, c):
        hi = F(c)
        return (((16 * (p // 16) + 8).astype(F) - hi) - F(c - float(hi))) + ((p % 16).astype(F) - F(7.5))

    dx, dy = offset(xs, u), np.broadcast_to(offset(ys, v), xs.shape)
    a0 = conic[0] * dx * dx
    q2 = _fma(dy, _fma(np.full_like(dy, conic[2]), dy, conic[1] * dx), a0)
    passed = (xs >= 0) & (xs < W) & (q2 >= F(K * 9.0))
    ex, ey = xs + 0.5 - u, ys + 0.5 - v
    exact = (c0 * ex * ex + c1 * ex * ey + c2 * ey * ey) / K
    block = (ys // 8) * W + xs // 8
    sure = np.unique(block[(exact <= 9.0) & (xs >= 0) & (xs < W)])
    return int(passed.sum()), int((passed & np.isin(block, sure)).sum())


@pytest.mark.parametrize("bin_size", [16, 32])
def test_needles_keep_their_ends(bin_size):
    import torch
    from paper_2604_17155_amd import gsc
    sc, cam = _scene()
    u, v, conic = _records(sc, cam)
    most, least = np.array([_counts(u[g], v[g], conic[g]) for g in range(N)]).T
    assert least.min() > 1000
    ctx = gsc.Context(bin_size=bin_size, t_min=0.0)
    y = torch.ones((W * H, 1), device="cuda")
    _, _, x = ctx.colorize(*gsc.scene_tensors(sc), sc.cams, y, 0, [1e-4], extras={"counts"})
    got = x["counts"].cpu().numpy()
    off = (got < least) | (got > most)
    print(f"bins {bin_size}: {int(off.sum())} of {N} counts out of range, {int((got < least).sum())} of them short; "
          f"{int(got.sum())} in {int(least.sum())} .. {int(most.sum())}", flush=True)
    assert int(off.sum()) <= 4
