"""What the statistics say: the pairs of a reused binning after another call on the
context; the launches of a call whose batches are split, and of the blends."""
import pytest

from paper_2604_17155_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counted", [False, True])
def test_pairs_of_a_reused_binning(counted):
    """A reusing call reports the pairs of the binning that it reuses, whether they
    were read back (counted: a pair limit that the batch just meets) or not, and
    whatever an allocation-free call on the context counted in between."""
    import torch
    from paper_2604_17155_amd import gsc
    sc, other = syn.make_plain(n=700, n_cams=3, res=64), syn.make_plain(n=90, n_cams=2, res=48)
    geo, og = gsc.scene_tensors(sc), gsc.scene_tensors(other)
    y = torch.rand((sc.n_pixels, 3), device="cuda")
    ctx = gsc.Context(bin_size=16)
    c, _ = ctx.colorize(*geo, sc.cams, y, 0, [1e-4])
    want = int(ctx.stats().pairs)
    assert want > 1000
    if counted:
        ctx = gsc.Context(bin_size=16, batch_pairs=want)
        c, _ = ctx.colorize(*geo, sc.cams, y, 0, [1e-4])
        st = ctx.stats()
        assert int(st.pairs) == want and st.view_batches == 1
    yo = torch.rand((other.n_pixels, 3), device="cuda")
    ctx.colorize_noalloc(*og, other.cams, yo, 0, [1e-4], torch.empty((other.N, 1, 3), device="cuda"))
    assert 0 < int(ctx.stats().pairs) != want
    img = ctx.render(*geo, sc.cams, c, reuse_binning=True)
    assert int(ctx.stats().pairs) == want
    ctx.render_backward(*geo, sc.cams, c, torch.ones_like(img), reuse_binning=True)
    assert int(ctx.stats().pairs) == want


@pytest.mark.parametrize("n_refine", [None, 2])
@pytest.mark.parametrize("part", [2.5, 9.0, 60.0])
def test_batches_are_split_before_their_pairs_are_made(part, n_refine):
    """A batch over the caller's pair limit is split when its pairs have been counted,
    before they take memory: pairs are emitted once a batch and pass."""
    import torch
    from paper_2604_17155_amd import gsc
    sc = syn.make_plain(n=3000, n_cams=24, res=96)
    geo = gsc.scene_tensors(sc)
    y = torch.rand((sc.n_pixels, 3), device="cuda")
    one = gsc.Context(bin_size=16)
    ref, _ = one.colorize(*geo, sc.cams, y, 0, [1e-4]) if n_refine is None else \
        one.colorize_refine(*geo, sc.cams, y, 0, [1e-4], n_refine)
    pairs = int(one.stats().pairs)
    ctx = gsc.Context(bin_size=16, batch_pairs=int(pairs / part), flags=gsc.GSC_FLAG_PROFILE)
    c, _ = ctx.colorize(*geo, sc.cams, y, 0, [1e-4]) if n_refine is None else \
        ctx.colorize_refine(*geo, sc.cams, y, 0, [1e-4], n_refine)
    st = ctx.stats()
    emitted = int(st.stage_launches[gsc.STAGES.index("emit")])
    print(f"{pairs} pairs, limit {int(pairs / part)}: {st.view_batches} batches, {emitted} emissions", flush=True)
    assert st.view_batches >= min(part, len(sc.cams)) and int(st.pairs) == pairs
    assert emitted == st.view_batches * (1 + (n_refine or 0))
    assert float((c - ref).abs().max()) <= 1e-4 * float(ref.abs().max())


# (C, BF16, many tiles, variant) -> accumulate launches: the few-tile form's 3, 7 or 15
# channels a launch for the automatic vector code, the code's own otherwise
@pytest.mark.parametrize("C,bf16,many,variant,launches", [
    (3, False, False, 0, 1), (7, False, False, 0, 1), (8, False, False, 0, 1), (64, False, False, 0, 5),
    (64, False, True, 0, 4), (8, False, False, 4, 2), (8, False, False, 8, 1), (64, False, False, 8, 8),
    (16, True, False, 0, 1), (16, True, False, 16, 2), (64, True, False, 128 + 32, 2), (64, True, True, 0, 1)])
def test_accumulate_launches(C, bf16, many, variant, launches):
    """The launches that the statistics report, by the kernels' own channel counts; and
    the same result whichever form runs."""
    import torch
    from paper_2604_17155_amd import gsc
    sc = syn.make_plain(n=500, n_cams=1, res=64)
    geo = gsc.scene_tensors(sc)
    cams = syn.circle_cams(70 if many else 3, 3.0, 128, 128)  # 64 tiles each
    gen = torch.Generator(device="cuda").manual_seed(C)
    y = torch.rand((len(cams) * 128 * 128, C), generator=gen, device="cuda")
    y = y.bfloat16() if bf16 else y
    ctx = gsc.Context(bin_size=16, accumulate_variant=variant, flags=gsc.GSC_FLAG_PROFILE)
    blend = gsc.STAGES.index("blend")
    c, _ = ctx.colorize(*geo, cams, y, 0, [1e-4])
    assert int(ctx.stats().stage_launches[blend]) == launches
    ref, _ = gsc.Context(bin_size=16, accumulate_variant=1).colorize(*geo, cams, y, 0, [1e-4])
    assert float((c - ref).abs().max()) <= 1e-4 * float(ref.abs().max())
    plan = gsc.Plan(ctx, [(0, sc.N, 0, len(cams))], *geo, cams, C, 0)
    plan.run(y, [1e-4])
    assert int(ctx.stats().stage_launches[blend]) == launches
    # a render: the view colours, then 4 channels a launch (8 of few tiles past 4)
    ctx.render(*geo, cams, c)
    assert int(ctx.stats().stage_launches[blend]) == 1 + (C + 7) // 8 if C > 4 and not many else 1 + (C + 3) // 4


def test_autotune_times_what_it_names():
    """A plan of few tiles: the automatic vector code runs the few-tile form and the
    others their own, so that no two names stand for one kernel; whichever is taken
    gives the first run's result."""
    import torch
    from paper_2604_17155_amd import gsc
    sc = syn.make_plain(n=4000, n_cams=8, res=64)
    geo = gsc.scene_tensors(sc)
    y = torch.rand((sc.n_pixels, 16), device="cuda").bfloat16()
    ctx = gsc.Context(bin_size=16, flags=gsc.GSC_FLAG_PROFILE)
    plan = gsc.Plan(ctx, [(0, sc.N, 0, 8)], *geo, sc.cams, 16, 0)
    ref, _ = plan.run(y, [1e-4])
    c, _ = plan.autotune(y, [1e-4])
    info = plan.info()
    names = [v for v in info.tuned_variant if v]
    assert {16, 8, 4} <= set(names) and info.accumulate_variant in names
    assert float((c - ref).abs().max()) <= 1e-4 * float(ref.abs().max())
    ctx.stats()
    plan.run(y, [1e-4])
    want = {16: 2, 8: 2, 4: 4}.get(info.accumulate_variant & 127 if info.accumulate_variant & 128 == 0 else 0, 1)
    if info.accumulate_variant == 16 + 256:
        want = 1  # the persistent grid of the tile form
    assert int(ctx.stats().stage_launches[gsc.STAGES.index("blend")]) == want
