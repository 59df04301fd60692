"""The few-tile accumulate takes 15 channels a launch and the rest in a launch of 3, 7
or 15: the channel counts around those widths, against one channel a launch."""
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu

U = 2.0 ** -24  # binary32 unit roundoff


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("C", [3, 4, 7, 8, 15, 16, 18, 19, 22, 23, 30, 31, 33, 37, 38])
def test_widths(C, bf16):
    import torch
    from paper_2604_17155_amd import gsc
    sc = syn.make_plain(n=900, n_cams=2, res=96)
    geo = gsc.scene_tensors(sc)
    gen = torch.Generator(device="cuda").manual_seed(C)
    y = torch.rand((sc.n_pixels, C), generator=gen, device="cuda")
    y = y.bfloat16() if bf16 else y
    code = C if C <= 4 else (8 if C <= 8 else 16)  # the automatic vector code
    _, _, x = gsc.Context(bin_size=16, accumulate_variant=code).colorize(*geo, sc.cams, y, 0, [1e-4], extras={"view_sums"})
    _, _, r = gsc.Context(bin_size=16, accumulate_variant=1).colorize(*geo, sc.cams, y, 0, [1e-4],
                                                                      extras={"view_sums", "counts"})
    a, b = x["view_sums"].double(), r["view_sums"].double()
    # sums of at most `counts` pixels, each in its own order, terms of at most a weight
    bound = 2.0 * (r["counts"].double()[None, :, None] + 16.0) * U * b[:, :, :1]
    assert float(b[:, :, 1:].max()) > 1.0 and bool(((a - b).abs() <= bound).all())
