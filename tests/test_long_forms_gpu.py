"""The kernels that ordinary and large calls run (the forward's four-wave tiles,
the adjoint's pairs tiles apart and four bands per workgroup) at every frequency
count, at the smallest sizes that reach them, against the oracle.
tests/test_forms_host.py asserts that these shapes select those forms.

Bars: forward 1e-12 relative per output; adjoint per entry 1e-12 relative plus
1e-12 of the array's largest checked entry.
"""
import numpy as np
import pytest

import oracle
from paper_2008_11326_amd import inputs as I
from tests.gpu_helpers import assert_parity, mixed_pole_problem, say, to_device
from tests.test_bwd_gpu import ARRAYS, check_entries, gpu_grads

pytestmark = pytest.mark.gpu

# (number_bands, nvband, ncouls, ngpown, nfreq): two occupied bands, then at
# least four whole band groups of the hot loop and a band left over
FORWARD = [(11, 2, 2048, npw, nw) for nw, npw in
           zip(range(1, 9), (127, 191, 127, 65, 65, 65, 65, 65))]
PAIRS_APART = [(16, 1, 2048, 102, nw) for nw in range(1, 9)] + [(23, 9, 2048, 102, 5)]
# single tiles for few occupied bands, a shared tile for more; a ragged last one
FOUR_BANDS = [(260, 5, 8100, 2, nw) for nw in range(1, 9)] + \
             [(262, 14, 8100, 2, nw) for nw in (2, 5)]


@pytest.fixture(scope="module")
def gpp():
    import paper_2008_11326_amd as gpp
    return gpp


@pytest.mark.parametrize("shape", FORWARD, ids=str)
@pytest.mark.parametrize("low", [0.0, 0.01])
def test_forward(gpp, shape, low):
    """With low > 0 waves hold real poles, exact ones and nearly vanishing om
    (branch C) among ordinary lanes."""
    import torch
    prob = mixed_pole_problem(sum(shape), I.Dims(*shape), low)
    if low:
        rng = np.random.default_rng(sum(shape))
        prob.wtilde_array[rng.random(prob.wtilde_array.shape) < low / 4] = 1e-8 + 1e-8j
    say(f"[long forms] forward {shape} {low}")
    ach, asx = gpp.sigma_fwd(**to_device(prob), nvband=prob.dims.nvband)
    torch.cuda.synchronize()
    ref = oracle.sigma_fwd(prob)
    assert_parity(ach.cpu().numpy(), ref[0], ref[2], "achtemp")
    assert_parity(asx.cpu().numpy(), ref[1], ref[3], "asxtemp")


@pytest.mark.parametrize("shape", PAIRS_APART + FOUR_BANDS, ids=str)
def test_adjoint(gpp, shape):
    prob = I.make_problem(I.Dims(*shape), sum(shape) + 1, 0.02)
    nb, nv, ng, npw, nw = shape
    rng = np.random.default_rng(sum(shape))
    ga, gs = I.make_upstream_grad(nw, rng)
    say(f"[long forms] adjoint {shape}")
    grads = gpu_grads(gpp, prob, ga, gs)
    for name in ARRAYS:
        rows, cols = grads[name].shape
        used = npw if name == "aqsmtemp" else cols
        idx = np.stack([rng.integers(0, rows, 24), rng.integers(0, used, 24)], axis=1)
        edge = {(r, c) for r in (0, nv - 1, nv, rows - 2, rows - 1) if 0 <= r < rows
                for c in (0, used // 2, used - 1)}
        check_entries(name, grads[name], prob, ga, gs,
                      np.concatenate([idx, np.array(sorted(edge))]).astype(np.int64))
    assert np.all(grads["aqsmtemp"][:, npw:] == 0)
    part = gpu_grads(gpp, prob, ga, gs, want=(False, True, False, True))
    assert part["aqsmtemp"] is None and part["I_eps_array"] is None
    assert np.array_equal(part["aqsntemp"], grads["aqsntemp"])
    assert np.array_equal(part["wtilde_array"], grads["wtilde_array"])
