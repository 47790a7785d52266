"""Direction counts that divide neither a 16-query tile nor a pass: every point's cache level and
residual against the FP64 oracle, point by point (one query of 65 left out or counted twice moves
a point by about 1.5 %, above every per-point bound used)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_04634_amd import workload as wl
from tests.common import check_estimate_points, host, residual_prediction

pytestmark = pytest.mark.gpu
PRECS = {"fp32": 0, "bf16": 1, "fp16": 2}


@pytest.mark.parametrize("prec,width", [("fp32", 64), ("bf16", 64), ("fp16", 64), ("fp16", 128)])
@pytest.mark.parametrize("N", [3, 5, 6, 7, 9, 12, 15, 17, 31, 33, 63, 65])
def test_direction_counts(prec, width, N):
    print(f"{prec} W={width} N={N}", flush=True)
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_04634_amd import nirc
    P, seed, frame = 37, 60 + N, 5
    pts = wl.make_points(seed, P)
    lob = wl.make_lobes(seed).packed()
    w0 = wl.make_weights(seed, width)
    model = nirc.Model(w0, cfg=nirc.make_config(width=width, precision=PRECS[prec]), max_batch=0)
    tl, c, r = (host(t) for t in nirc.tlmc_estimate(model, nirc.Points.from_workload(pts), lob, N, seed, frame,
                                                    parts=True))
    o_tl, o_c, o_r = oracle.estimate(pts, lob, w0, width, N, seed, frame)
    y_r = residual_prediction(pts, w0, width, N, seed, frame)
    check_estimate_points(f"{prec} W={width} N={N}", tl, c, r, o_tl, o_c, o_r, y_r, prec)
    assert np.isfinite(tl).all()
