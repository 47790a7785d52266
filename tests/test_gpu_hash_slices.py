"""The grid-entry sums of a hash-model training step over the grid shapes that choose their path:
slices summed in LDS (one or many per level, of their own or shared by several workgroups) and, for
grids beyond them, global atomic sums; against the FP64 oracle, and the fused step against its parts.

Tolerance: on samples without a ReLU decision within FP32 rounding of its switch, the FP32 gradient
bound 1e-5 that the other gradient tests use (per level, whose entries are fewer, three times it), plus
12 x 2^-24 N_11 where the finest level's cells are smaller than FP32 positions resolve (the bound of the
grid lookup: a position product that rounds up to a cell's edge scatters to the next cell); the fused
step does the same arithmetic as the gradient and a separate Adam call, so its weights are equal
bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_04634_amd import workload as wl
from tests.common import UNIT_ROUNDOFF, Samples, hash_tie_free_samples, host, rel_l2

pytestmark = pytest.mark.gpu
PRECS = {"fp32": 0, "bf16": 1, "fp16": 2}
# one slice per level; a slice of exactly 8192 entries; hashed slices shared by workgroups; dense
# rows that do not fill a slice; the default; resolutions beyond a slice (global atomics)
GRIDS = [(10, 4, 1.5), (13, 16, 1.5), (14, 8, 1.3), (16, 16, 1.5), (17, 30, 1.1), (18, 16, 1.5), (14, 40, 2.0)]


@pytest.fixture(scope="module")
def nirc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_04634_amd import nirc as m
    m.lib()
    return m


def make(nirc, prec, grid, seed, max_batch):
    w = wl.make_hash_weights(seed, 64, 2 * oracle.hash_entries(grid), 0.5)
    return nirc.HashModel(w, cfg=nirc.make_config(precision=PRECS[prec]), grid=nirc.make_hash_grid(*grid),
                          max_batch=max_batch), w


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("B", [1, 700, 40001])
def test_entry_sums(nirc, grid, B):
    print(f"{grid} B={B}", flush=True)
    pts, lob = wl.make_points(71, 900), wl.make_lobes(71).packed()
    model, w = make(nirc, "fp32", grid, 71, B)
    sm, _ = hash_tie_free_samples(pts, lob, B, 72, 0, 0, w.astype(np.float64), grid, 16 * UNIT_ROUNDOFF["fp32"])
    _, grad = nirc.nirc_hash_loss_grad(model, nirc.Points.from_workload(pts), sm.queries(nirc), sm.target())
    _, ref = oracle.hash_loss_grad(pts, sm.idx, sm.d, sm.t, w.astype(np.float64), 64, grid)
    nm, g = oracle.hash_mlp_params(64), host(grad)
    res, off, _ = oracle.hash_levels(grid)
    fine = 12 * 2.0 ** -24 * res[11] if res[11] > 8192 else 0.0
    assert rel_l2(g[nm:], ref[nm:]) <= 1e-5 + fine
    if not fine:
        assert np.all(g[nm:][ref[nm:] == 0.0] == 0.0)
    ends = list(off[1:]) + [oracle.hash_entries(grid)]
    for l in range(12):   # a lost slice or part of one shows in its level
        a, b = nm + 2 * off[l], nm + 2 * ends[l]
        assert rel_l2(g[a:b], ref[a:b]) <= 3e-5 + fine, l


def parameters_and_moments(model):
    """The FP32 parameters and both Adam moments: the first three 256-byte aligned pieces of a state."""
    blob, n = model.get_state(), 4 * model.n_params
    step = (n + 255) // 256 * 256
    return [blob[k * step:k * step + n] for k in range(3)]


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("B", [65, 40001])
def test_fused_step_is_gradient_and_adam(nirc, prec, grid, B):
    print(f"{prec} {grid} B={B}", flush=True)
    pts, lob = wl.make_points(73, 900), wl.make_lobes(73).packed()
    dp = nirc.Points.from_workload(pts)
    one, _ = make(nirc, prec, grid, 73, B)
    two, _ = make(nirc, prec, grid, 73, B)
    for step in range(2):
        sm = Samples(pts, lob, B, 74, 0, step)
        nirc.nirc_hash_train_step(one, dp, sm.queries(nirc), sm.target())
        _, grad = nirc.nirc_hash_loss_grad(two, dp, sm.queries(nirc), sm.target())
        nirc.nirc_hash_adam_step(two, grad)
    for a, b in zip(parameters_and_moments(one), parameters_and_moments(two)):
        assert torch.equal(a, b)
    assert one.read_flags() == 0


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_batch_beyond_the_workspace(nirc, prec):
    """The gradient of a batch larger than the workspace was sized for (where its partial sums still
    fit) runs in parts; a batch that needs more partial sums is refused."""
    pts, lob = wl.make_points(75, 900), wl.make_lobes(75).packed()
    dp, grid, B = nirc.Points.from_workload(pts), (14, 8, 1.3), 50001
    small, w = make(nirc, prec, grid, 75, 16384)
    large, _ = make(nirc, prec, grid, 75, B)
    sm = Samples(pts, lob, B, 76, 0, 0)
    l0, g0 = nirc.nirc_hash_loss_grad(small, dp, sm.queries(nirc), sm.target())
    l1, g1 = nirc.nirc_hash_loss_grad(large, dp, sm.queries(nirc), sm.target())
    assert rel_l2(host(g0), host(g1)) <= 1e-5
    assert abs(float(l0) - float(l1)) <= 1e-6 * float(l1)
    nirc.nirc_hash_train_step(small, dp, sm.queries(nirc), sm.target())
    assert small.read_flags() == 0 and not torch.equal(small.get_weights(), torch.from_numpy(w).cuda())
    tiny, _ = make(nirc, prec, grid, 75, 64)
    with pytest.raises(nirc.NircError):
        nirc.nirc_hash_loss_grad(tiny, dp, sm.queries(nirc), sm.target())


@pytest.mark.parametrize("value", [1e30, float("inf"), float("nan")])
@pytest.mark.parametrize("grid", [GRIDS[0], GRIDS[5], GRIDS[6]])
def test_out_of_range_gradient_skips_the_step(nirc, grid, value):
    pts, lob = wl.make_points(77, 900), wl.make_lobes(77).packed()
    dp = nirc.Points.from_workload(pts)
    model, w = make(nirc, "fp32", grid, 77, 1000)
    sm = Samples(pts, lob, 1000, 78, 0, 0)
    t = sm.target().clone()
    t[567, 1] = value
    nirc.nirc_hash_train_step(model, dp, sm.queries(nirc), t)
    assert model.read_flags() == nirc.NIRC_FLAG_NONFINITE_GRAD
    assert torch.equal(model.get_weights(), torch.from_numpy(w).cuda())
    nirc.nirc_hash_train_step(model, dp, sm.queries(nirc), sm.target())
    assert not torch.equal(model.get_weights(), torch.from_numpy(w).cuda())
