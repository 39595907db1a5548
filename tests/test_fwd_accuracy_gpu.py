"""Accuracy of the forward where the test's own inputs let one step of it be
seen, against exact or 80-bit long-double values."""
import numpy as np
import pytest

from paper_2008_11326_amd import inputs as I
from tests.gpu_helpers import say, to_device

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def gpp():
    import paper_2008_11326_amd as gpp
    return gpp


@pytest.mark.parametrize("scale", [1e3, 1e70, 1e80, 1e100])
@pytest.mark.parametrize("imag", [0.1, 0.0])
@pytest.mark.parametrize("nw", range(1, 9))
def test_exchange_far_from_the_poles(gpp, nw, imag, scale):
    """Every frequency far above every pole: 1/(|x - om|^2 |x + om|^2) passes
    below the smallest double while the exchange terms, e om^2 / (x^2 - om^2),
    are well inside the range.  All terms have positive real parts, so that
    sum |term| is the sum.  Bar: 40 roundings of one term and an addition per
    term (8 bands x 64 rows x 3 columns)."""
    nb, ng, npw = 8, 64, 3
    prob = I.make_problem(I.Dims(nb, nb, ng, npw, nw), nw)
    rng = np.random.default_rng(nw)
    for z in (prob.aqsmtemp, prob.aqsntemp, prob.I_eps_array):
        z[:] = rng.uniform(0.1, 0.5, z.shape)
    prob.wtilde_array[:] = (rng.uniform(0.5, 2.0, (npw, ng)) + imag * rng.uniform(1, 2, (npw, ng)) * 1j)
    prob.wx_array[:] = scale * rng.uniform(1.0, 2.0, (nw, nb))
    C = np.clongdouble
    om, e, v = prob.wtilde_array.astype(C), prob.I_eps_array.astype(C), prob.vcoul.astype(C)
    M = prob.aqsntemp.astype(C)[:, None, :] * prob.aqsmtemp[:, :npw].astype(C)[:, :, None]
    x = prob.wx_array.astype(C)[:, :, None, None]
    ref = (v * M * e * om * om / ((x - om) * (x + om))).sum(axis=(1, 2, 3))
    _, asx = gpp.sigma_fwd(**to_device(prob), nvband=nb)
    worst = float(np.max(np.abs(asx.cpu().numpy() - ref) / np.abs(ref))) / U
    bar = 40 + nb * ng * npw
    say(f"[fwd accuracy] exchange x ~ {scale:g} nfreq {nw}: {worst:.1f} u, bar {bar}")
    assert worst <= bar
