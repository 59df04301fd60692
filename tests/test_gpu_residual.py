"""The residual of a refinement pass: formed by the render's stores where one launch
writes all channels, else by a pass of its own, each target row once."""
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("many", [False, True])
def test_shared_and_scattered_rows(C, many):
    """Views that share their target rows, and views whose rows lie apart, give the
    result of views with rows of their own, one after the other."""
    import torch
    from paper_2604_17155_amd import gsc
    sc = syn.make_plain(n=400, n_cams=1, res=64)
    geo = gsc.scene_tensors(sc)
    res = 512 if many else 64  # 5 x 1024 tiles are more than the few-tile form's
    cams = syn.circle_cams(4, 3.0, res, res)
    cams = [cams[0], cams[0], cams[1], cams[2], cams[3]]
    P = res * res
    gen = torch.Generator(device="cuda").manual_seed(C)
    y = torch.rand((4, P, C), generator=gen, device="cuda")
    gap = torch.full((37, C), float("nan"), device="cuda")
    ref, _ = gsc.Context(bin_size=16).colorize_refine(*geo, cams, torch.cat([y[0], y[0], y[1], y[2], y[3]]), 0, [1e-4], 3)
    shared = torch.cat([y[1], gap, y[0], y[3], gap, y[2]])
    at = [P + 37, P + 37, 0, 3 * P + 74, 2 * P + 37]
    got, _ = gsc.Context(bin_size=16).colorize_refine(*geo, cams, shared, 0, [1e-4], 3, offsets=at)
    # sums in another order, through three passes that shrink the residual
    assert float((got - ref).abs().max()) <= 2e-5 * float(ref.abs().max())


def test_time_of_many_channels():
    """A pass costs about a render and a colorize of the same channels."""
    import torch
    from paper_2604_17155_amd import gsc
    n, C = 700, 48
    sc = syn.make_plain(n=n, n_cams=1, res=64)
    geo = gsc.scene_tensors(sc)
    cams = syn.circle_cams(18, 3.0, 531, 382)
    y = torch.rand((18 * 531 * 382, C), device="cuda")
    co = torch.rand((n, 1, C), device="cuda")
    ctx = gsc.Context()
    img = torch.empty_like(y)

    def ms(f):
        t = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return sorted(t)[3]

    col = ms(lambda: ctx.colorize(*geo, cams, y, 0, [1e-4]))
    ren = ms(lambda: ctx.render(*geo, cams, co, images=img))
    ref = ms(lambda: ctx.colorize_refine(*geo, cams, y, 0, [1e-4], 2))
    print(f"colorize {col:.2f} ms, render {ren:.2f} ms, two passes {ref:.2f} ms", flush=True)
    assert ref <= 1.2 * (3.0 * col + 2.0 * ren)
