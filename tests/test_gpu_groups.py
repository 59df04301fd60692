"""Group pairs sorted view by view: views of 20 to 255 groups (one pass over
segments) and of 256 (the general sort), views without pairs at the start, in the
middle and at the end, too few pairs for segments, both bin sizes, and a plan with
scenes of different size.  A call over all views against calls over one view each,
which sort at most 8 bits in one segment: contribution counts are equal, binary32
sums differ by the order of their additions (about sqrt(tiles) 2^-24, 1e-5 allows
for every tile of a view)."""
import numpy as np
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu


def _cams(sizes, away):
    out = []
    for k, (w, h) in enumerate(sizes):
        p = np.array([3.0 * np.cos(0.7 * k), 3.0 * np.sin(0.7 * k), 0.6])
        out.append(syn.look_at(p, w, h, target=tuple(2.0 * p) if k in away else (0.0, 0.0, 0.0)))
    return out


def _single(gsc, ctx, geo, cam, y):
    c, st, x = ctx.colorize(*geo, [cam], y, 1, [1e-3, 1e-3], extras={"counts", "view_sums"})
    return x["counts"].cpu().numpy().astype(np.int64), x["view_sums"][0].double().cpu().numpy()


@pytest.mark.parametrize("n,sizes,away,bins", [
    (20000, [(640, 640)] * 4, (), 16), (20000, [(640, 640), (320, 200), (960, 1088), (640, 640)], (1,), 16),
    (20000, [(960, 1088)] * 3, (0,), 16), (20000, [(1024, 1024), (640, 640)], (), 16),
    (30000, [(1280, 1280)] * 5, (4,), 32), (300, [(640, 640)] * 4, (), 16)])
def test_views_together_and_alone(n, sizes, away, bins):
    import torch
    from paper_2604_17155_amd import gsc
    rng = np.random.default_rng(n + bins)
    geo = [torch.from_numpy(a).cuda() for a in syn.blob_geometry(rng, n)]
    cams = _cams(sizes, away)
    ys = [torch.from_numpy(rng.random((w * h, 3), dtype=np.float32)).cuda() for w, h in sizes]
    ctx = gsc.Context(bin_size=bins)
    c, st, x = ctx.colorize(*geo, cams, torch.cat(ys), 1, [1e-3, 1e-3], extras={"counts", "view_sums"})
    counts, sums = x["counts"].cpu().numpy().astype(np.int64), x["view_sums"].double().cpu().numpy()
    alone = [_single(gsc, ctx, geo, cam, y) for cam, y in zip(cams, ys)]
    assert np.array_equal(counts, sum(a for a, _ in alone)) and counts.sum() > 0
    for k, (_, ref) in enumerate(alone):
        assert np.all(ref == 0.0) == (k in away)
        assert np.all(np.abs(sums[k] - ref) <= 1e-5 * np.abs(ref)), k
    print(f"{n} Gaussians, {sizes}, bins {bins}: {int(counts.sum())} contributions", flush=True)


def test_plan_of_uneven_scenes():
    import torch
    from paper_2604_17155_amd import gsc
    rng = np.random.default_rng(5)
    ns, cams, ys, table, parts = [9000, 25000], [], [], [], []
    for n in ns:
        own = _cams([(640, 512), (512, 640), (640, 640)], ())
        table.append((sum(ns[:len(parts)]), n, len(cams), len(own)))
        parts.append(syn.blob_geometry(rng, n))
        cams += own
        ys += [torch.from_numpy(rng.random((c.width * c.height, 3), dtype=np.float32)).cuda() for c in own]
    geo = [torch.from_numpy(np.concatenate(a)).cuda() for a in zip(*parts)]
    ctx = gsc.Context(bin_size=16)
    plan = gsc.Plan(ctx, table, *geo, cams, 3, 0)
    c, st = plan.run(torch.cat(ys), [1e-3])
    assert plan.info().dropped_pairs == 0
    for k, (g0, n, c0, nc) in enumerate(table):
        ref, sref, _ = ctx.colorize(*[a[g0:g0 + n].contiguous() for a in geo], cams[c0:c0 + nc],
                                    torch.cat(ys[c0:c0 + nc]), 0, [1e-3], extras={"counts"})
        assert torch.equal(st[g0:g0 + n], sref)
        assert torch.all((c[g0:g0 + n] - ref).abs() <= 1e-5 * ref.abs())
