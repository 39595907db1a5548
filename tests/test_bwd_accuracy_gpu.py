"""Accuracy of the adjoint next to large poles: |om| is about 450 times
|x - om| (branch A ends at 500), so that a gradient formed from separate sums
of x and of om loses that factor.  Reference: the gradients term by term in
80-bit long double.

Bar per entry, with u = 2^-53 and the sum over its terms:
    |error| <= (64 + terms) u sum |term|
64 = 20 (one Newton step on a hardware reciprocal, 2.2e-15, shared by a batch)
+ 24 (two roundings per factor of a batch of at most 12) + 20 (the roundings of
one term's own products), and one addition per term.
"""
import numpy as np
import pytest

from paper_2008_11326_amd import inputs as I
from tests.gpu_helpers import say
from tests.test_bwd_gpu import gpu_grads

pytestmark = pytest.mark.gpu

C, U = np.clongdouble, 2.0 ** -53


@pytest.fixture(scope="module")
def gpp():
    import paper_2008_11326_amd as gpp
    return gpp


def large_pole_problem(dims, seed):
    nb, _, ng, npw, nw = dims.as_tuple()
    prob = I.make_problem(dims, seed)
    rng = np.random.default_rng(seed)
    prob.wtilde_array[:] = (450.0 + rng.uniform(-0.02, 0.02, (npw, ng))
                            + 1j * rng.uniform(-0.05, 0.05, (npw, ng)))
    prob.wx_array[:] = 451.0 + rng.uniform(-0.02, 0.02, (nw, nb))
    # every term on branch A, which the references below take for granted
    d2, o2 = 0.96 ** 2, 450.02 ** 2 + 0.05 ** 2
    assert d2 > 0.25 and o2 < 250000.0 * d2
    return prob


def references(prob, ga, rows):
    """Gradients at the given G rows (daqsmtemp: over all rows, so only where
    `rows` holds them all) and the sums of |term|, every band unoccupied."""
    nb, _, ng, npw, nw = prob.dims.as_tuple()
    # [n][p][g] per frequency
    om, e = prob.wtilde_array[:, rows].astype(C), prob.I_eps_array[:, rows].astype(C)
    v = prob.vcoul[rows].astype(np.longdouble)
    an, am = prob.aqsntemp[:, rows].astype(C), prob.aqsmtemp[:, :npw].astype(C)
    Mc = np.conj(an)[:, None, :] * am[:, :, None]
    ref = {k: 0 for k in ("aqsmtemp", "aqsntemp", "I_eps_array", "wtilde_array")}
    mag = dict(ref)
    for w in range(nw):
        x = prob.wx_array[w].astype(np.longdouble)[:, None, None]
        u = np.conj(1 / (x - om))
        h = C(ga[w]) / 2
        K = h * np.conj(om) * u
        vz = v * np.conj(e) * K
        for name, term, axis in (
                ("I_eps_array", v * Mc * K, 0),
                ("wtilde_array", v * np.conj(e) * Mc * h * x * u * u, 0),
                ("aqsntemp", am[:, :, None] * vz, 1),
                ("aqsmtemp", an[:, None, :] * np.conj(vz), 2)):
            ref[name] = ref[name] + term.sum(axis=axis)
            mag[name] = mag[name] + np.abs(term).sum(axis=axis)
    terms = {"I_eps_array": nb * nw, "wtilde_array": nb * nw, "aqsntemp": npw * nw,
             "aqsmtemp": len(rows) * nw}
    return ref, mag, terms


def check(got, ref, mag, terms, what):
    err = np.abs(got - ref)
    worst = float(np.max(err / (mag * U)))
    say(f"[bwd accuracy] {what}: {worst:.1f} u of the sum of |term|, bar {64 + terms}")
    assert worst <= 64 + terms, what


# dI_eps of bands that go through B1 - om A2 (up to four frequencies, whole
# groups) cancels, so there only one band, which is formed by itself
@pytest.mark.parametrize("nb,nw", [(1, nw) for nw in range(1, 9)] +
                         [(nb, nw) for nb in (3, 6) for nw in range(5, 9)])
def test_band_sums(gpp, nb, nw):
    prob = large_pole_problem(I.Dims(nb, 0, 70, 3, nw), 10 * nb + nw)
    ga, _ = I.make_upstream_grad(nw, np.random.default_rng(nw))
    g = gpu_grads(gpp, prob, ga, ga)
    ref, mag, terms = references(prob, ga, np.arange(70))
    for name in ("I_eps_array", "wtilde_array"):
        check(g[name], ref[name], mag[name], terms[name], f"{name} {nb} bands nfreq {nw}")


# one- and two-band tiles, and four-band ones (8448 waves of them)
@pytest.mark.parametrize("nw", range(1, 9))
@pytest.mark.parametrize("nb,ng,npw", [(3, 70, 3), (66, 1000, 6), (264, 8100, 2)])
def test_column_and_row_sums(gpp, nb, ng, npw, nw):
    prob = large_pole_problem(I.Dims(nb, 0, ng, npw, nw), nb + nw)
    ga, _ = I.make_upstream_grad(nw, np.random.default_rng(nw))
    g = gpu_grads(gpp, prob, ga, ga)
    only = gpu_grads(gpp, prob, ga, ga, want=(False, True, False, False))
    assert np.array_equal(only["aqsntemp"], g["aqsntemp"])
    rows = np.arange(ng) if ng <= 100 else np.r_[0:20, ng // 2:ng // 2 + 20, ng - 20:ng]
    ref, mag, terms = references(prob, ga, rows)
    check(g["aqsntemp"][:, rows], ref["aqsntemp"], mag["aqsntemp"], terms["aqsntemp"],
          f"aqsntemp {nb} x {ng} nfreq {nw}")
    if len(rows) == ng:
        check(g["aqsmtemp"][:, :npw], ref["aqsmtemp"], mag["aqsmtemp"], terms["aqsmtemp"],
              f"aqsmtemp {nb} x {ng} nfreq {nw}")
