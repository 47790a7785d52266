"""FP32 models of width 64 on the two-term FP16 products, and the models that take the FP32 chain
instead, against the FP64 oracle.

Tolerances: predictions rel-L2 <= 1e-6 (five layer sums, each rounded to about 2^-23 of its size,
and the exponential: about 5 x 1.2e-7 with a margin of 1.7), and the per-query bound of the FP32
chain."""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_04634_amd import workload as wl
from tests.common import check_estimate_points, check_query_points, host, rel_l2, residual_prediction

pytestmark = pytest.mark.gpu
W = 64


@pytest.fixture(scope="module")
def nirc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_04634_amd import nirc as m
    m.lib()
    return m


def mats(w):
    """Views of the five weight matrices of a canonical vector."""
    out, o = [], 0
    for r, c in wl.layer_shapes(W):
        out.append(w[o:o + r * c].reshape(r, c))
        o += r * c
    return out


def queries(P, Q, seed):
    g = torch.Generator().manual_seed(seed)
    idx = torch.randint(0, P, (Q,), generator=g, dtype=torch.int32)
    return idx, torch.nn.functional.normalize(torch.randn(Q, 3, generator=g), dim=1)


# one tile and its edges, the last count of one-tile passes (2,048 tiles) and the first of four
@pytest.mark.parametrize("Q", [1, 15, 16, 17, 127, 129, 32768, 32769, 40001])
def test_infer(nirc, Q):
    P = 300
    pts, w = wl.make_points(Q, P), wl.make_weights(Q, W)
    idx, d = queries(P, Q, Q)
    model = nirc.Model(w, max_batch=0)
    y = host(nirc.nirc_infer(model, nirc.Points.from_workload(pts), nirc.Queries.from_dirs(d.cuda(), idx.cuda())))
    ref = oracle.infer(pts, idx.numpy(), d.double().numpy(), w, W)
    assert rel_l2(y, ref) <= 1e-6
    check_query_points(f"split Q={Q}", y, ref, "fp32")


def reshape_weights(kind, w):
    """The same function in other magnitudes (powers of two along the ReLU chain), or a model whose
    rows differ widely."""
    m = mats(w)
    if kind == "balanced":        # the split scales follow
        m[0] *= 2.0 ** 18
        m[1] *= 2.0 ** -18
        m[4] *= 2.0 ** -9
        m[3] *= 2.0 ** 9
    elif kind == "beyond_norms":  # layer norms outside 2^+-30: the FP32 chain
        m[0] *= 2.0 ** 40
        m[1] *= 2.0 ** -40
    elif kind == "wide_rows":     # a row 2^-13 and less of its layer's largest weight: the FP32 chain
        m[1][7] *= 2.0 ** -16
        m[2][:, 7] *= 2.0 ** 16
    elif kind == "edge_rows":     # just inside: rows a few binades below the largest weight
        m[1][7] *= 2.0 ** -9
        m[2][:, 7] *= 2.0 ** 9
    elif kind == "dead_rows":     # zero rows are no small rows
        m[1][3] = 0.0
        m[3][60:] = 0.0
    elif kind == "zero_layer":
        m[2][:] = 0.0
    return w


@pytest.mark.parametrize("kind", ["balanced", "beyond_norms", "wide_rows", "edge_rows", "dead_rows", "zero_layer"])
def test_weight_ranges(nirc, kind):
    P, N, seed = 130, 8, 9
    pts, lob = wl.make_points(seed, P), wl.make_lobes(seed).packed()
    w = reshape_weights(kind, wl.make_weights(seed, W))
    idx, d = queries(P, 1000, seed)
    model, dp = nirc.Model(w, max_batch=0), nirc.Points.from_workload(pts)
    y = host(nirc.nirc_infer(model, dp, nirc.Queries.from_dirs(d.cuda(), idx.cuda())))
    ref = oracle.infer(pts, idx.numpy(), d.double().numpy(), w, W)
    assert rel_l2(y, ref) <= 1e-6, kind
    tl, c, r = (host(t) for t in nirc.tlmc_estimate(model, dp, lob, N, seed, 2, parts=True))
    o_tl, o_c, o_r = oracle.estimate(pts, lob, w, W, N, seed, 2)
    check_estimate_points(kind, tl, c, r, o_tl, o_c, o_r, residual_prediction(pts, w, W, N, seed, 2), "fp32")
    out = torch.empty((P, 3), dtype=torch.float32, device="cuda")
    batch = nirc.Batch()
    batch.set([dict(model=model, points=dp, lobes=lob, n_cache=N, seed=seed, frame=2, out_tl=out)])
    batch.launch()
    assert np.array_equal(host(out), tl)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_non_finite_weights(nirc, value):
    """A weight that is not finite: whatever stays finite in plain FP32 arithmetic does here too."""
    P, seed = 64, 4
    pts, w = wl.make_points(seed, P), wl.make_weights(seed, W)
    m = mats(w)
    m[3][5, 9] = value
    idx, d = queries(P, 500, seed)
    y = host(nirc.nirc_infer(nirc.Model(w, max_batch=0), nirc.Points.from_workload(pts),
                             nirc.Queries.from_dirs(d.cuda(), idx.cuda())))
    with np.errstate(all="ignore"):
        ref = oracle.infer(pts, idx.numpy(), d.double().numpy(), w, W)
    if np.isneginf(value):   # the unit is off wherever its input is positive
        ok = np.isfinite(ref).all(axis=1)
        assert ok.any() and rel_l2(y[ok], ref[ok]) <= 1e-6
    else:
        assert not np.isfinite(y).all()
