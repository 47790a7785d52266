"""FP32 inference of width 64 takes one or four query tiles per pass by the size of the call: a query's
prediction has the same bits in both."""
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


# Glorot weights and larger ones (outputs over a wide range), both outputs, and a model of the FP32 chain
@pytest.mark.parametrize("kind", ["plain", "large", "sigmoid", "fp32_chain"])
def test_one_and_four_tiles(nirc, kind):
    P, Q = 500, 32769 + 4 * 16 * 3
    w = wl.make_weights(11, 64)
    if kind == "large":
        w = (1.3 * w).astype(np.float32)
    elif kind == "fp32_chain":   # a row far above the others, off almost everywhere
        m = w[64 * 160:64 * 160 + 4096].reshape(64, 64)
        m[5] = -2.0 ** 12 * np.abs(m[5])
        m[5, :4] *= -1
    dp = nirc.Points.from_workload(wl.make_points(11, P))
    model = nirc.Model(w, nirc.make_config(output=1 if kind == "sigmoid" else 0), max_batch=0)
    g = torch.Generator().manual_seed(11)
    idx = torch.randint(0, P, (Q,), generator=g, dtype=torch.int32).cuda()
    d = torch.nn.functional.normalize(torch.randn(Q, 3, generator=g), dim=1).cuda()
    whole = nirc.nirc_infer(model, dp, nirc.Queries.from_dirs(d, idx))
    for a, n in ((0, 32768), (1, 32768), (17, 1000), (Q - 5, 5)):
        part = nirc.nirc_infer(model, dp, nirc.Queries.from_dirs(d[a:a + n].contiguous(), idx[a:a + n].contiguous()))
        assert torch.equal(part, whole[a:a + n]), (kind, a, n)
