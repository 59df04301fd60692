"""What the statistics say: the pairs of a reused binning after another call on the
context; the launches of a call whose batches are split."""
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
