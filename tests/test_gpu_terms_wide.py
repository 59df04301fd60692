"""Per-item terms of many channels: blocks of 64 to 4 Gaussians (the coefficients that
fit the staging area), whose threads share a Gaussian's views; and their time against
the bytes that they cannot do without.  Bounds as for the narrow ones."""
import numpy as np
import pytest

from paper_2604_17155_amd import synthetic as syn
from tests.test_gpu_terms import test_terms_against_oracle as terms_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,C,views,n", [(3, 5, 37, 65), (3, 11, 3, 33), (3, 22, 70, 17), (3, 43, 2, 9),
                                         (2, 64, 33, 130), (1, 64, 1, 70), (0, 64, 9, 129)])
def test_wide_terms_against_oracle(L, C, views, n):
    terms_against_oracle(L, C, views, n)


def test_time_of_wide_terms():
    import torch
    from paper_2604_17155_amd import gsc
    n, V, C = 50000, 32, 64
    m, s, q, o = (torch.from_numpy(a).cuda() for a in syn.blob_geometry(np.random.default_rng(3), n))
    o = o * 0  # nothing is listed: the adjoint stage is the terms alone
    cams = syn.hemisphere_cams(V, 3.0, 16, 16)
    y = torch.ones((V * 256, C), device="cuda")
    co = torch.ones((n, 16, C), device="cuda")
    ctx = gsc.Context(flags=gsc.GSC_FLAG_PROFILE)
    t = []
    for _ in range(7):
        ctx.colorize_backward(m, s, q, o, cams, y, 3, [1e-3] * 4, co, co)
        torch.cuda.synchronize()
        t.append(1e-3 * ctx.stats().stage_dict()["blend_adjoint"])
    need = 4 * (2 * co.numel() + n * V * (C + 1))  # both sets read, every item written
    print(f"{1e6 * sorted(t)[3]:.0f} us for {1e-6 * need:.0f} MB", flush=True)
    assert sorted(t)[3] < need / 0.5e12
