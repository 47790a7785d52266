"""Training of 16-bit models of width 64 over the batch sizes that choose how partial sums are formed
(one chunk of 64 samples per slab, two that the reduction adds first, up to 256 slabs of several), and
frames (FP32 ones too) whose samples are drawn inside the gradient kernel.

Drawn samples are those of tlmc_train_batch bit for bit, and a frame's step does the arithmetic of
nirc_train_step on them: weights are equal bit for bit, alone and in a list.

Tolerance of a batch's gradient against its parts of 4096 samples (one chunk per slab): the loss's factor
per sample differs by two FP32 roundings between batch sizes, which moves a 16-bit delta to its
neighbour (2^-8 of it) with probability 2^-14; the sum of n samples moves by 2^-7 2^-8 of a sample's
norm times sqrt(n), 3e-5 of the sum when the samples' gradients are uncorrelated.  2e-4 allows for the
layers below; a lost chunk of 64 samples of 40,001 shows at 1.6e-3 or more.
"""
import numpy as np
import pytest
import torch

from paper_2412_04634_amd import workload as wl
from tests.common import Samples, host, rel_l2

pytestmark = pytest.mark.gpu
PRECS = {"bf16": 1, "fp16": 2}


@pytest.fixture(scope="module")
def nirc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_04634_amd import nirc as m
    m.lib()
    return m


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("B", [8192, 8193, 12345, 16384, 16385, 40001])
def test_gradient_is_the_sum_of_parts(nirc, prec, B):
    print(f"{prec} B={B}", flush=True)
    pts, lob = wl.make_points(81, 3000), wl.make_lobes(81).packed()
    dp = nirc.Points.from_workload(pts)
    s = Samples(pts, lob, B, 82, 0, 0)
    w = wl.make_weights(81, 64)
    model = nirc.Model(w, nirc.make_config(precision=PRECS[prec]), max_batch=B)
    loss, grad = nirc.nirc_loss_grad(model, dp, s.queries(nirc), s.target())
    gs, ls = np.zeros(model.n_params), 0.0
    for b0 in range(0, B, 4096):
        sl = slice(b0, min(B, b0 + 4096))
        n = sl.stop - sl.start
        part = Samples(pts, lob, B, 82, 0, 0)
        part.select(sl)
        l, g = nirc.nirc_loss_grad(model, dp, part.queries(nirc), part.target())
        gs += host(g).astype(np.float64) * n / B
        ls += float(l) * n / B
    assert rel_l2(host(grad), gs) <= 2e-4
    assert abs(float(loss) - ls) <= 1e-5 * ls


@pytest.mark.parametrize("prec", ["fp32", *PRECS])
@pytest.mark.parametrize("output", [0, 1, 2])
def test_drawn_frame_equals_its_steps(nirc, prec, output):
    pts, lob = wl.make_points(83, 2000), wl.make_lobes(83).packed()
    dp = nirc.Points.from_workload(pts)
    reqs, want = [], []
    for B in [1, 63, 8192, 8193, 16385, 140000]:   # the last: five rounds, drawn four at a time
        print(f"{prec} output={output} B={B}", flush=True)
        cfg = nirc.make_config(precision=PRECS.get(prec, 0), output=output)
        a, b, c = (nirc.Model(wl.make_weights(83, 64), cfg, max_batch=B) for _ in range(3))
        nirc.nirc_train_frame(a, dp, lob, B, 3, 84, 7)
        for k in range(3):
            q, t = nirc.tlmc_train_batch(dp, lob, B, 84, 7, k, output=output)
            nirc.nirc_train_step(b, dp, q, t)
        assert torch.equal(a.get_weights(), b.get_weights()), B
        reqs.append(dict(model=c, points=dp, lobes=lob, batch=B, seed=84, frame=7))
        want.append(a.get_weights())
    if prec == "fp32":   # lists take 16-bit models
        return
    tlist = nirc.TrainBatch(140000)
    tlist.set(reqs)
    tlist.launch(3)
    for r, w in zip(reqs, want):
        assert torch.equal(r["model"].get_weights(), w), r["batch"]


def test_drawn_hash_frame_equals_its_steps(nirc):
    pts, lob = wl.make_points(85, 2000), wl.make_lobes(85).packed()
    dp = nirc.Points.from_workload(pts)
    import oracle
    grid = (14, 8, 1.3)
    w = wl.make_hash_weights(85, 64, 2 * oracle.hash_entries(grid), 0.5)
    for prec in (0, 1, 2):
        for B in (1, 12345, 40001):
            print(f"hash prec={prec} B={B}", flush=True)
            a, b = (nirc.HashModel(w, cfg=nirc.make_config(precision=prec), grid=nirc.make_hash_grid(*grid), max_batch=B)
                    for _ in range(2))
            nirc.nirc_hash_train_frame(a, dp, lob, B, 2, 86, 3)
            for k in range(2):
                q, t = nirc.tlmc_train_batch(dp, lob, B, 86, 3, k)
                nirc.nirc_hash_train_step(b, dp, q, t)
            assert torch.equal(a.get_weights(), b.get_weights()), (prec, B)
