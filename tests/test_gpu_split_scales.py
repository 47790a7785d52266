"""FP32 models of width 64 whose neurons differ widely, in several layers at once: the two-term products
must hold every neuron's bits, or leave the model to the FP32 chain.  Against the FP64 oracle.

Tolerance: predictions rel-L2 <= 1e-6, as for plain models, where the model is a Glorot model rewritten by
powers of two (FP32 arithmetic then gives a plain model's error); for the sums that cancel, four times the
error of the same chain in numpy's FP32 (another order of the same roundings), and 1e-6 if that is more."""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_04634_amd import workload as wl
from tests import npref
from tests.common import check_estimate_points, host, rel_l2, residual_prediction

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
    out, o = [], 0
    for r, c in wl.layer_shapes(W):
        out.append(w[o:o + r * c].reshape(r, c))
        o += r * c
    return out


def reshape(kind, w):
    m = mats(w)

    def stretch(l, unit, e):   # unit of hidden layer l + 1 by 2^e, its outgoing weights by 2^-e
        m[l][unit] *= 2.0 ** e
        m[l + 1][:, unit] *= 2.0 ** -e

    if kind == "one_unit":
        stretch(1, 7, 10)
    elif kind == "unit_per_layer":
        for l in (1, 2, 3):
            stretch(l, 7 + l, 9)
    elif kind == "two_layers":
        for l in (1, 2):
            stretch(l, 7 + l, 9)
    elif kind == "four_layers":
        for l, e in ((0, 9), (1, 2), (2, 9), (3, 2)):
            stretch(l, 7 + l, e)
    elif kind == "every_unit":
        for l in range(4):
            for unit in range(W):
                stretch(l, unit, (5 * unit + 3 * l) % 17 - 8)
    elif kind == "far_units":
        for l in range(4):
            stretch(l, 11 + l, 40)
            stretch(l, 31 + l, -40)
    elif kind == "rarely_on":   # large units that are off almost everywhere
        for l in (1, 2, 3):
            m[l][5] = -256 * np.abs(m[l][5])
            m[l][5, :4] *= -1
    elif kind == "paired":      # equal units in pairs, whose large outgoing weights cancel
        for l in range(4):
            m[l][1::2] = m[l][0::2]
            m[l + 1][:, 0::2] += 8
            m[l + 1][:, 1::2] -= 8
    return w


def fp32_chain(pts, idx, d, w):
    """The predictions with every layer in numpy's FP32.  The library's ReLU is an integer maximum: it keeps
    a NaN weight's NaN and takes that of 0 x inf, whose sign bit is set, to 0."""
    keep = np.isnan(w).any()
    h = npref.encode(npref.inputs_of(pts, idx, d)).astype(np.float32)
    ms = [m.astype(np.float32) for m in mats(w)]
    for m in ms[:4]:
        h = (np.maximum if keep else np.fmax)(h @ m.T, np.float32(0))
    return np.exp((h @ ms[4].T).astype(np.float64))


KINDS = ["one_unit", "unit_per_layer", "two_layers", "four_layers", "every_unit", "far_units", "rarely_on", "paired"]


@pytest.mark.parametrize("kind", KINDS)
def test_neurons_far_apart(nirc, kind):
    P, N, Q, seed = 130, 8, 4000, 9
    pts, lob = wl.make_points(seed, P), wl.make_lobes(seed).packed()
    w = reshape(kind, wl.make_weights(seed, W))
    g = torch.Generator().manual_seed(seed)
    idx = torch.randint(0, P, (Q,), generator=g, dtype=torch.int32)
    d = torch.nn.functional.normalize(torch.randn(Q, 3, generator=g), dim=1)
    model, dp = nirc.Model(w, max_batch=0), nirc.Points.from_workload(pts)
    y = host(nirc.nirc_infer(model, dp, nirc.Queries.from_dirs(d.cuda(), idx.cuda())))
    ref = oracle.infer(pts, idx.numpy(), d.double().numpy(), w, W)
    tol = 1e-6
    if kind == "paired":
        tol = max(tol, 4 * rel_l2(fp32_chain(pts, idx.numpy(), d.double().numpy(), w), ref))
    err = rel_l2(y, ref)
    print(f"{kind}: rel-L2 {err:.2e} (bound {tol:.1e})", flush=True)
    assert err <= tol
    tl, c, r = (host(t) for t in nirc.tlmc_estimate(model, dp, lob, N, seed, 2, parts=True))
    o_tl, o_c, o_r = oracle.estimate(pts, lob, w, W, N, seed, 2)
    check_estimate_points(kind, tl, c, r, o_tl, o_c, o_r, residual_prediction(pts, w, W, N, seed, 2), "fp32")
    out = torch.empty((P, 3), dtype=torch.float32, device="cuda")
    batch = nirc.Batch()
    batch.set([dict(model=model, points=dp, lobes=lob, n_cache=N, seed=seed, frame=2, out_tl=out)])
    batch.launch()
    assert np.array_equal(host(out), tl)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("layer", [1, 3, 4])
def test_non_finite_weight_of_a_dead_unit(nirc, layer, value):
    """A weight that is not finite shows as in plain FP32 arithmetic also behind a unit that is never on, whose
    column the scales drop."""
    P, Q, seed = 64, 500, 4
    pts, w = wl.make_points(seed, P), wl.make_weights(seed, W)
    m = mats(w)
    m[layer - 1][9] = 0.0 if layer == 1 else -np.abs(m[layer - 1][9])
    m[layer][2, 9] = value
    g = torch.Generator().manual_seed(seed)
    idx = torch.randint(0, P, (Q,), generator=g, dtype=torch.int32)
    d = torch.nn.functional.normalize(torch.randn(Q, 3, generator=g), dim=1)
    model, dp = nirc.Model(w, max_batch=0), nirc.Points.from_workload(pts)
    y = host(nirc.nirc_infer(model, dp, nirc.Queries.from_dirs(d.cuda(), idx.cuda())))
    with np.errstate(all="ignore"):
        ref = fp32_chain(pts, idx.numpy(), d.double().numpy(), w)
    ok = np.isfinite(ref)
    assert np.array_equal(np.isfinite(y), ok)
    assert rel_l2(y[ok], ref[ok]) <= 1e-6
