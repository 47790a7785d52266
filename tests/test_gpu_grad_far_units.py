"""FP32 loss gradients of width 64 of models whose units are far apart: every unit's gradient, however small
beside the others', against the FP64 oracle; and the choice of operands follows the weights.

Tolerance: a unit's gradient (its row of a weight matrix, or its column of the next) is compared with the
error that plain FP32 arithmetic makes of the same unit's: nirc_backward, whose products and sums are all FP32, on
the oracle's output gradient.  Operands of the sums over the samples have 22 bits where FP32 has 24, a factor of 4,
and the sums run in another order, another 2; beside that, 4 x 2^-22 sqrt(B) for the operands' own errors where
the samples' signs cancel (rel-L2 per unit, on samples without a ReLU decision within rounding of its
switch)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_04634_amd import workload as wl
from tests import npref
from tests.common import Samples, host, rel_l2

pytestmark = pytest.mark.gpu
W, P, SEED = 64, 4000, 91


@pytest.fixture(scope="module")
def nirc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_04634_amd import nirc as m
    m.lib()
    return m


def spread_units(exponent):
    """The Glorot model with hidden unit u of layer l scaled by 2^exponent(l, u) (the same function)."""
    w = wl.make_weights(SEED, W)
    m = npref.split_weights(w, W)
    for l in range(4):
        e = np.array([2.0 ** exponent(l, u) for u in range(W)])
        m[l] *= e[:, None]
        m[l + 1] /= e[None, :]
    return np.concatenate([a.ravel() for a in m]).astype(np.float32)


KINDS = {
    "near": lambda l, u: (5 * u + 3 * l) % 9 - 4,
    "within": lambda l, u: (5 * u + 3 * l) % 17 - 8,
    "apart": lambda l, u: (13 * u + 7 * l) % 41 - 20,
    "one_far_unit_per_layer": lambda l, u: 40 if u == 11 + l else -40 if u == 31 + l else 0,
}


def samples(pts, B):
    sm = Samples(pts, wl.make_lobes(SEED).packed(), B, 92, 0, 0)
    sm.drop_relu_ties(pts, wl.make_weights(SEED, W).astype(np.float64), W)   # (scaling by 2^e moves no decision)
    return sm


def unit_errors(got, ref):
    """rel-L2 of every row and column of the five weight matrices."""
    out = []
    for axis in (0, 1):
        for a, b in zip(npref.split_weights(got, W), npref.split_weights(ref, W)):
            out.append(np.linalg.norm(a - b, axis=axis) / np.maximum(np.linalg.norm(b, axis=axis), 1e-300))
    return np.concatenate(out)


@pytest.mark.parametrize("B", [300, 4096, 20000, 70000])
@pytest.mark.parametrize("kind", list(KINDS))
def test_every_units_gradient(nirc, kind, B):
    pts, w = wl.make_points(SEED, P), spread_units(KINDS[kind])
    sm = samples(pts, B)
    model = nirc.Model(w, nirc.make_config(), max_batch=len(sm.idx))
    loss, grad = nirc.nirc_loss_grad(model, nirc.Points.from_workload(pts), sm.queries(nirc), sm.target())
    ref_loss, ref = sm.loss_grad(pts, w.astype(np.float64), W)
    y = oracle.infer(pts, sm.idx, sm.d, w, W)
    d_rgb = 2.0 * (y - sm.t) / (y * y + 1e-2) / (3 * len(sm.idx))
    plain = nirc.nirc_backward(model, nirc.Points.from_workload(pts), sm.queries(nirc),
                               torch.from_numpy(d_rgb.astype(np.float32)).cuda())
    err, tol = unit_errors(host(grad), ref), 8 * unit_errors(host(plain), ref) + 4 * 2.0 ** -22 * np.sqrt(B)
    i = int((err / tol).argmax())
    print(f"{kind} B={B}: worst unit {err[i]:.1e} (bound {tol[i]:.1e})", flush=True)
    assert (err <= tol).all()
    assert rel_l2(host(grad), ref) <= 1e-5
    assert abs(float(loss) - float(ref_loss)) <= 1e-5 * abs(float(ref_loss))


def test_follows_the_weights(nirc):
    """The operands are chosen anew when weights or a state come in."""
    pts, near, apart = wl.make_points(SEED, P), spread_units(KINDS["near"]), spread_units(KINDS["apart"])
    sm = samples(pts, 3000)
    dp, q, t = nirc.Points.from_workload(pts), sm.queries(nirc), sm.target()
    models = {k: nirc.Model(w, nirc.make_config(), max_batch=4096) for k, w in (("near", near), ("apart", apart))}
    want = {k: nirc.nirc_loss_grad(m, dp, q, t)[1].clone() for k, m in models.items()}
    model = nirc.Model(near, nirc.make_config(), max_batch=4096)
    for k, w in (("apart", apart), ("near", near), ("apart", apart)):
        model.set_weights(torch.from_numpy(w).cuda())
        assert torch.equal(nirc.nirc_loss_grad(model, dp, q, t)[1], want[k])
    for k in ("near", "apart"):
        model.set_state(models[k].get_state())
        assert torch.equal(nirc.nirc_loss_grad(model, dp, q, t)[1], want[k])


@pytest.mark.parametrize("B", [5000, 40000])
def test_drawn_step(nirc, B):
    """A frame's step, which draws its samples in the gradient kernel, equals the step on the same samples."""
    pts, w, lob = wl.make_points(SEED, P), spread_units(KINDS["apart"]), wl.make_lobes(SEED).packed()
    dp = nirc.Points.from_workload(pts)
    a, b = (nirc.Model(w, nirc.make_config(), max_batch=B) for _ in range(2))
    nirc.nirc_train_frame(a, dp, lob, B, 1, 5, 2)
    q, t = nirc.tlmc_train_batch(dp, lob, B, 5, 2, 0)
    nirc.nirc_train_step(b, dp, q, t)
    assert torch.equal(a.get_weights(), b.get_weights()) and a.read_flags() == 0


def test_resumed_training_sums_as_the_saved(nirc):
    """Steps that take the weights over the line between the operands: a model resumed from the saved state
    continues bit for bit, where one made from the same weights takes the other operands."""
    pts, w = wl.make_points(SEED, P), wl.make_weights(SEED, W)
    m = npref.split_weights(w, W)
    m[2][:] = np.clip(m[2], -0.1249, 0.1249)   # exponents of the rows' largest: -4; after a step of 0.01 some -3
    m[2][7] = -1.5 * 2.0 ** -16                # never on, so it stays, 2^12 from the others and then 2^13
    w = np.concatenate([a.ravel() for a in m]).astype(np.float32)
    sm = Samples(pts, wl.make_lobes(SEED).packed(), 3000, 92, 0, 0)
    dp, q, t = nirc.Points.from_workload(pts), sm.queries(nirc), sm.target()
    make = lambda w: nirc.Model(w, nirc.make_config(lr=1e-2), max_batch=3000)
    saved, resumed = make(w), make(wl.make_weights(SEED + 1, W))
    for _ in range(3):
        nirc.nirc_train_step(saved, dp, q, t)
    blob = saved.get_state()
    resumed.set_state(blob)
    fresh = make(host(saved.get_weights()))
    grads = [nirc.nirc_loss_grad(k, dp, q, t)[1].clone() for k in (saved, resumed, fresh)]
    assert torch.equal(resumed.get_state(), blob)
    assert torch.equal(grads[1], grads[0])
    assert not torch.equal(grads[2], grads[0])
    assert rel_l2(host(grads[2]), host(grads[0])) <= 1e-5
    for k in (saved, resumed):
        nirc.nirc_train_step(k, dp, q, t)
    assert torch.equal(resumed.get_state(), saved.get_state())
