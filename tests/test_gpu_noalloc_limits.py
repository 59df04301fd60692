"""The allocation-free call accepts what fits its 64 MiB and refuses what cannot."""
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu

SCRATCH = 64 << 20


def _call(gsc, ctx, geo, cams, y, sh_deg=0, offsets=None):
    import torch
    N, C, nb = int(geo[0].shape[0]), int(y.shape[1]), (sh_deg + 1) ** 2
    c = torch.empty((N, nb, C), device="cuda")
    st = torch.empty((N,), dtype=torch.uint8, device="cuda")
    ctx.colorize_noalloc(*geo, cams, y, sh_deg, [1e-4], c, st, offsets=offsets)
    return c, st


@pytest.mark.parametrize("batch_items", [0, 200_000])
def test_items_that_miss_the_image(batch_items):
    """48 bytes an item of the first view batch, 64 a Gaussian: views whose items
    mostly miss the image are accepted up to that, and refused past it without any
    work."""
    import torch
    from paper_2604_17155_amd import gsc
    n = 20_000
    sc = syn.make_plain(n=n, n_cams=1, res=48)
    geo = gsc.scene_tensors(sc)
    geo[0][100:, 2] += 50.0
    cams = syn.circle_cams(64, 3.0, 48, 48)
    y = torch.rand((64 * 48 * 48, 1), device="cuda")
    ctx = gsc.Context(batch_items=batch_items)
    assert 64 * 64 * n > SCRATCH > 48 * 64 * n + 64 * n
    c, st = _call(gsc, ctx, geo, cams, y)
    assert 50 < int((st == 0).sum()) <= 100
    ref, rst = gsc.Context(batch_items=batch_items).colorize(*geo, cams, y, 0, [1e-4])
    assert torch.equal(st, rst) and float((c - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
    # 72 views in one batch need 48 * 72 * n bytes
    many = syn.circle_cams(72, 3.0, 48, 48)
    y = torch.rand((72 * 48 * 48, 1), device="cuda")
    assert 48 * 72 * n > SCRATCH
    if batch_items:
        _, st = _call(gsc, ctx, geo, many, y)
        assert 50 < int((st == 0).sum()) <= 100
    else:
        for flags in (0, gsc.GSC_FLAG_VALIDATE_ONLY):
            with pytest.raises(gsc.GscError) as e:
                _call(gsc, gsc.Context(flags=flags), geo, many, y)
            assert e.value.status == gsc.GSC_ERR_CAPACITY
