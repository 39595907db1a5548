"""Host-only: the shapes of tests/test_long_forms_gpu.py select the forms they
are there for, and the GPU tests of small shapes the others, so that a change of
a threshold cannot take a kernel out of the tests unseen.  A small C++ shim calls
the library's own geometry functions (no device call)."""
import ctypes as C
import os
import random
import subprocess

import pytest

from paper_2008_11326_amd import _lib, build
from tests import test_grid_forms_gpu as grid
from tests import test_long_forms_gpu as forms

SHIM = """
#include "gpp_internal.h"
extern "C" void forms(int nb, int nv, int ng, int np, int nw, int *out)
{
    const gpp::Dims32 d{nb, nv, ng, np, nw};
    const gpp::FwdGeometry f = gpp::fwd_geometry(d);
    const gpp::BwdGeometry b = gpp::bwd_geometry(d);
    out[0] = f.waves;
    out[1] = f.nchunk;
    out[2] = b.share_pairs;
    out[3] = b.tile_bands;
    out[4] = b.single;
    out[5] = (int)(f.nblocks + f.red_blocks);
}
"""


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    (d / "shim.cpp").write_text(SHIM)
    lib = str(d / "shim.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1",
                    f"-I{build.CSRC}", f"-I{build.INCLUDE}", f"-isystem{rocm}/include",
                    str(d / "shim.cpp"), "-o", lib, _lib.LIB_PATH,
                    f"-Wl,-rpath,{os.path.dirname(os.path.abspath(_lib.LIB_PATH))}"], check=True)
    _lib.load()
    shim = C.CDLL(lib)

    def of(shape):
        out = (C.c_int * 6)()
        shim.forms(*shape, out)
        return dict(zip(("waves", "nchunk", "share", "tile", "single", "rows"), out))

    return of


def test_forward_shapes_take_the_four_wave_tiles(form):
    for shape in forms.FORWARD:
        f = form(shape)
        assert f["waves"] == 4 and f["nchunk"] == 1, (shape, f)


def test_adjoint_shapes_take_the_long_forms(form):
    for shape in forms.PAIRS_APART:
        assert form(shape)["share"] == 0, shape
    for shape in forms.FOUR_BANDS:
        f = form(shape)
        assert f["tile"] == 4 and f["single"] == (shape[1] if shape[1] <= 12 else 0), (shape, f)


def test_small_shapes_take_the_short_forms(form):
    """Every form of the short grids at every frequency count."""
    for nw in range(1, 9):
        small = [form(s) for s in grid.EACH_NFREQ + [(67, 3, 1000, 6, nw)] if s[4] == nw]
        assert {f["waves"] for f in small} == {16}
        assert {f["share"] for f in small} == {1}
        assert {f["tile"] for f in small} == {1, 2}


def need(shape):
    return int(_lib.load().gpp_sigma_fwd_workspace(C.byref(_lib.dims_struct(*shape))))


def random_shape(rng):
    nw, nb = rng.randint(1, 8), int(2 ** rng.uniform(0, 11))
    ng = int(2 ** rng.uniform(0, 17))
    return nb, 0, ng, max(1, min(ng, int(2 ** rng.uniform(0, 12)))), nw


def test_forward_workspace_holds_every_row(form):
    rng = random.Random(3)
    for _ in range(20000):
        shape = random_shape(rng)
        assert form(shape)["rows"] * 32 * shape[4] <= need(shape), shape


def test_forward_workspace_of_a_larger_call_serves_a_smaller_one():
    """A program that keeps one buffer for states of several sizes sizes it for
    the largest: no call with every size at most as large may need more."""
    rng = random.Random(4)
    for _ in range(100000):
        nb, nv, ng, npw, nw = small = random_shape(rng)
        grow = lambda n: int(n * rng.choice((1, 1, 1.05, 1.5, 2.5)))
        ng2 = grow(ng)
        large = (grow(nb), nv, ng2, max(npw, min(ng2, grow(npw))), min(8, nw + rng.randint(0, 2)))
        assert need(small) <= need(large), (small, large)
