"""The fold and solve against the same normal equations formed in numpy's
float64 from the per-view sums the call returns: the numbers of views around
the quad's step of four and the 64 views of a mask word, Gaussians seen by few
of them, channel counts around the solve's step of four, every degree.  The
outputs are binary32, so a row differs by at most their rounding, 2^-24 of
each entry; twice that allows for the float64 solves (condition <= 1.3e5)."""
import numpy as np
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu


def _basis(d, L):
    x, y, z = d.T
    r = lambda a, b: np.sqrt(a / (b * np.pi))
    out = [np.full_like(x, r(1, 4)), r(3, 4) * y, r(3, 4) * z, r(3, 4) * x,
           r(15, 4) * x * y, r(15, 4) * y * z, r(5, 16) * (3 * z * z - 1), r(15, 4) * x * z, r(15, 16) * (x * x - y * y),
           r(35, 32) * y * (3 * x * x - y * y), r(105, 4) * x * y * z, r(21, 32) * y * (5 * z * z - 1),
           r(7, 16) * z * (5 * z * z - 3), r(21, 32) * x * (5 * z * z - 1), r(105, 16) * z * (x * x - y * y),
           r(35, 32) * x * (x * x - 3 * y * y)]
    return np.stack(out[:(L + 1) ** 2], 1)


@pytest.mark.parametrize("views,L,C", [(1, 3, 3), (3, 1, 1), (4, 2, 4), (5, 3, 5), (8, 3, 3), (8, 2, 9), (63, 1, 3),
                                       (64, 3, 3), (65, 2, 2), (131, 3, 7)])
def test_fold_against_float64(views, L, C):
    import torch
    from paper_2604_17155_amd import gsc
    rng = np.random.default_rng(views)
    n = 2500
    means, scales, quats, opac = syn.blob_geometry(rng, n)
    cams = syn.hemisphere_cams(views, 3.0, 53, 47)
    geo = [torch.from_numpy(a).cuda() for a in (means, scales, quats, opac)]
    y = torch.from_numpy(rng.random((views * 53 * 47, C), dtype=np.float32)).cuda()
    lam = [float(v) for v in syn.paper_lambda(L)]
    c, st, x = gsc.Context().colorize(*geo, cams, y, L, lam, extras={"view_sums", "visibility"})
    vs = x["view_sums"].double().cpu().numpy()
    nb = (L + 1) ** 2
    A, B, w = np.zeros((n, nb, nb)), np.zeros((n, nb, C)), np.zeros(n)
    for j, cam in enumerate(cams):
        R = np.asarray(cam.R, np.float32).astype(np.float64)
        d = means.astype(np.float64) + R.T @ np.asarray(cam.t, np.float32).astype(np.float64)
        phi = _basis(d / np.linalg.norm(d, axis=1, keepdims=True), L)
        A += (vs[j, :, :1] * phi)[:, :, None] * phi[:, None, :]
        B += phi[:, :, None] * vs[j, :, None, 1:]
        w += vs[j, :, 0]
    seen = w > 0
    assert np.array_equal((st.cpu().numpy() & 1) == 0, seen) and 0 < seen.sum()
    lam32 = np.asarray(lam, np.float32).astype(np.float64)
    diag = np.repeat(lam32, [2 * l + 1 for l in range(L + 1)])
    ref = np.zeros((n, nb, C))
    ref[seen] = np.linalg.solve(A[seen] + w[seen, None, None] * np.diag(diag), B[seen])
    got = c.double().cpu().numpy()
    assert not got[~seen].any()
    e = np.linalg.norm((got - ref).reshape(n, -1), axis=1) / np.maximum(np.linalg.norm(ref.reshape(n, -1), axis=1), 1e-30)
    counts = (vs[:, :, 0] > 0).sum(0)
    print(f"{views} views, L={L}, C={C}: {int(seen.sum())} observed, seen by {counts[seen].min()}..{counts.max()} views, "
          f"max {e[seen].max():.2e}", flush=True)
    assert e[seen].max() <= 2.0 * 2.0 ** -24
    assert np.allclose(x["visibility"].cpu().numpy(), w, rtol=2.0 ** -23, atol=0.0)
