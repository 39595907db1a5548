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


@pytest.mark.parametrize("nw", range(1, 9))
@pytest.mark.parametrize("shape,draws", [((1, 64, 4), 40), ((8, 64, 4), 40), ((8, 4096, 160), 12)])
def test_reciprocals_of_occupied_bands(gpp, nw, shape, draws):
    """At x = 0 a Coulomb-hole term is om / (0 - om) = -1, every other factor
    here being 1 and every other term 0, formed as om (conj(0 - om) r) with r
    the reciprocal of |om|^2: apart from the roundings of two products its error
    is that of the reciprocal.  Bar: with r good to one rounding u, the real
    part, a sum of two products of one sign, is off by at most 4 u (r, the
    factor conj(0 - om) r, one product and the sum), the imaginary part, whose
    products are at most 1/2 and cancel, by at most u: 4.2 u together.  (A
    reciprocal from a batch alone is off by up to 20 u.)"""
    nb, ng, npw = shape
    rng = np.random.default_rng(nw + nb + ng)
    prob = I.make_problem(I.Dims(nb, nb, ng, npw, nw), 1)
    prob.aqsmtemp[:] = 1.0
    worst = 0.0
    for _ in range(draws):
        w, n, p, g = (rng.integers(k) for k in (nw, nb, npw, ng))
        prob.wtilde_array[:] = rng.uniform(0.6, 2, (npw, ng)) + 1j * rng.uniform(-1, 1, (npw, ng))
        prob.wx_array[:] = rng.uniform(-2, -0.1, (nw, nb))
        prob.wx_array[w, n] = 0.0
        for a, at, v in ((prob.aqsntemp, n, 1.0), (prob.I_eps_array, (p, g), 1.0),
                         (prob.vcoul, g, 2.0)):
            a[:] = 0.0
            a[at] = v
        ach, _ = gpp.sigma_fwd(**to_device(prob), nvband=nb)
        worst = max(worst, abs(complex(ach[w].item()) + 1.0))
    say(f"[fwd accuracy] reciprocals {shape} nfreq {nw}: {worst / U:.1f} u, bar 4.2")
    assert worst <= 4.2 * U


@pytest.mark.parametrize("nw", range(1, 9))
@pytest.mark.parametrize("shape,draws", [((8, 64, 4), 40), ((9, 4096, 160), 12)])
def test_reciprocals_of_real_poles(gpp, nw, shape, draws):
    """The same for unoccupied bands where every om is real, a fifth of them
    on a frequency of some band.  The term is there -(|om|^2 r), P1 = 0: one
    rounding of r and one of the product."""
    nb, ng, npw = shape
    rng = np.random.default_rng(nw + nb + ng)
    prob = I.make_problem(I.Dims(nb, 0, ng, npw, nw), 1)
    prob.aqsmtemp[:] = 1.0
    worst = 0.0
    for _ in range(draws):
        w, n, p, g = (rng.integers(k) for k in (nw, nb, npw, ng))
        prob.wx_array[:] = rng.uniform(-2, 2, (nw, nb))
        prob.wx_array[w, n] = 0.0
        om = rng.uniform(0.6, 2, (npw, ng))
        on = rng.random(om.shape) < 0.2
        om[on] = rng.choice(np.abs(prob.wx_array.ravel()), size=int(on.sum()))
        om[p, g] = rng.uniform(0.6, 2)
        prob.wtilde_array[:] = om
        for a, at, v in ((prob.aqsntemp, n, 1.0), (prob.I_eps_array, (p, g), 1.0),
                         (prob.vcoul, g, 2.0)):
            a[:] = 0.0
            a[at] = v
        ach, _ = gpp.sigma_fwd(**to_device(prob), nvband=0)
        worst = max(worst, abs(complex(ach[w].item()) + 1.0))
    say(f"[fwd accuracy] real poles {shape} nfreq {nw}: {worst / U:.1f} u, bar 2")
    assert worst <= 2 * U
