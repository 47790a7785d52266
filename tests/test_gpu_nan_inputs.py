"""FP32 models of width 64: an input that is not a number spoils its own query's or point's result and no
other's.  The other results equal those of the call without it bit for bit."""
import numpy as np
import pytest
import torch

from paper_2412_04634_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nirc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_04634_amd import nirc as m
    m.lib()
    return m


# one and four query tiles per pass
@pytest.mark.parametrize("Q", [100, 40001])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_infer(nirc, Q, value):
    P = 300
    dp = nirc.Points.from_workload(wl.make_points(3, P))
    model = nirc.Model(wl.make_weights(3, 64), max_batch=0)
    g = torch.Generator().manual_seed(3)
    idx = torch.randint(0, P, (Q,), generator=g, dtype=torch.int32).cuda()
    d = torch.nn.functional.normalize(torch.randn(Q, 3, generator=g), dim=1)
    clean = nirc.nirc_infer(model, dp, nirc.Queries.from_dirs(d.cuda(), idx))
    bad = [0, 5, 37, Q // 2, Q - 1]
    d[bad, 1] = value
    got = nirc.nirc_infer(model, dp, nirc.Queries.from_dirs(d.cuda(), idx))
    good = torch.ones(Q, dtype=torch.bool)
    good[bad] = False
    assert torch.equal(got[good.cuda()], clean[good.cuda()])
    if np.isnan(value):
        assert got[bad].isnan().all()


@pytest.mark.parametrize("traced", [False, True])
@pytest.mark.parametrize("N", [1, 3, 4, 8, 16, 31, 32])
def test_estimate(nirc, N, traced):
    P = 300
    pts, lob = wl.make_points(4, P), wl.make_lobes(4).packed()
    model = nirc.Model(wl.make_weights(4, 64), max_batch=0)
    dp = nirc.Points.from_workload(pts)
    res = torch.rand((P, 3), device="cuda") if traced else None   # the caller's own residual radiance
    clean = nirc.tlmc_estimate(model, dp, lob, N, 4, 1, parts=True, residual=res)
    bad = [0, 18, 130, P - 1]
    pts.px[bad] = np.nan
    dp = nirc.Points.from_workload(pts)
    got = nirc.tlmc_estimate(model, dp, lob, N, 4, 1, parts=True, residual=res)
    good = torch.ones(P, dtype=torch.bool)
    good[bad] = False
    good = good.cuda()
    for a, b in zip(got, clean):
        assert torch.equal(a[good], b[good])
        assert a[bad].isnan().all()
    if traced:
        return
    out = torch.empty((P, 3), dtype=torch.float32, device="cuda")
    batch = nirc.Batch()
    batch.set([dict(model=model, points=dp, lobes=lob, n_cache=N, seed=4, frame=1, out_tl=out)])
    batch.launch()
    assert torch.equal(out[good], got[0][good]) and out[bad].isnan().all()
