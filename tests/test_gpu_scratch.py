"""A call's scratch stays within what one (bin, item) pair with its key in two buffers
takes (16 bytes) and 72 bytes an item, though lists are built through groups: the
list buffer is sized by the count of its entries in all but small calls."""
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [12, 25])
def test_scratch_of_a_call(views):
    import numpy as np
    import torch
    from paper_2604_17155_amd import gsc
    n, res = 100_000, 512
    m, s, q, o = (torch.from_numpy(a).cuda() for a in syn.blob_geometry(np.random.default_rng(3), n))
    cams = syn.hemisphere_cams(views, 3.0, res, res)
    y = torch.rand((views * res * res, 3), device="cuda")
    c = torch.empty((n, 1, 3), device="cuda")
    st = torch.empty((n,), dtype=torch.uint8, device="cuda")
    small = gsc.Context(bin_size=16)  # loads the kernels
    small.colorize(m, s, q, o, cams[:1], y, 0, [1e-4], coeffs=c, status=st)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx = gsc.Context(bin_size=16)
    ctx.colorize(m, s, q, o, cams, y, 0, [1e-4], coeffs=c, status=st)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    pairs = int(ctx.stats().pairs)
    # geometry, sums, ranges, order and sort counters: 64 + 16 bytes a splat, 24 a tile;
    # allocations are an eighth larger than asked for
    tiles = views * (res // 16) ** 2
    bound = 16 * pairs + 72 * views * n + 80 * n + 24 * tiles
    print(f"{views} views: {pairs} pairs, {used / 2 ** 20:.0f} MiB of {bound * 9 / 8 / 2 ** 20:.0f}", flush=True)
    assert 0 < used <= bound * 9 / 8
