"""Estimates and inference around the call sizes at which units of work (16 points, or 16 queries) go to
the workgroups in turn or by neighbours: a point's result does not depend on how many points the call
has, so a shorter call's results equal the longer one's bit for bit.  (FP32 inference of width 64 takes
one or four query tiles per pass by the size of the call, two forms of the same operations, each within
1e-5 of the exact value: 2e-5 of each other.)
"""
import pytest
import torch

import oracle
from paper_2412_04634_amd import workload as wl

pytestmark = pytest.mark.gpu
LONG = 140_000
# one unit; a workgroup per unit; 2,048 and 1,024 units (256 workgroups of 8 and of 4 waves) and one more or less
SIZES = [1, 17, 4096, 4097, 16384, 16385, 32767, 32768, 32769, 65537]


@pytest.fixture(scope="module")
def nirc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_04634_amd import nirc as m
    m.lib()
    return m


def prefix(nirc, points, n):
    return nirc.Points([t[:n].contiguous() for t in points.t])


@pytest.mark.parametrize("prec,width", [(0, 64), (1, 64), (0, 128), (1, 128)])
def test_estimate_and_infer(nirc, prec, width):
    pts, lob = wl.make_points(95, LONG), wl.make_lobes(95).packed()
    dp = nirc.Points.from_workload(pts)
    model = nirc.Model(wl.make_weights(95, width), nirc.make_config(width=width, precision=prec), max_batch=0)
    whole = nirc.tlmc_estimate(model, dp, lob, 3, 96, 1)
    q, _ = nirc.tlmc_train_batch(dp, lob, LONG, 97, 0, 0)
    d = torch.stack([q.wx, q.wy, q.wz], 1)
    rgb = nirc.nirc_infer(model, dp, q)
    for n in SIZES:
        print(f"prec={prec} width={width} n={n}", flush=True)
        assert torch.equal(nirc.tlmc_estimate(model, prefix(nirc, dp, n), lob, 3, 96, 1), whole[:n])
        sub = nirc.Queries.from_dirs(d[:n], q.point[:n])
        got = nirc.nirc_infer(model, dp, sub)
        if prec == 0 and width == 64:
            assert ((got - rgb[:n]).norm() <= 2e-5 * rgb[:n].norm()).item()
        else:
            assert torch.equal(got, rgb[:n])


@pytest.mark.parametrize("prec", [0, 1])
def test_hash_estimate(nirc, prec):
    pts, lob = wl.make_points(98, LONG), wl.make_lobes(98).packed()
    dp = nirc.Points.from_workload(pts)
    grid = (14, 8, 1.3)
    model = nirc.HashModel(wl.make_hash_weights(98, 64, 2 * oracle.hash_entries(grid), 0.5),
                           cfg=nirc.make_config(precision=prec), grid=nirc.make_hash_grid(*grid), max_batch=0)
    whole = nirc.nirc_hash_estimate(model, dp, lob, 3, 99, 1)
    for n in SIZES:
        print(f"hash prec={prec} n={n}", flush=True)
        assert torch.equal(nirc.nirc_hash_estimate(model, prefix(nirc, dp, n), lob, 3, 99, 1), whole[:n])
