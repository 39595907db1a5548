"""Host-only check of how the adjoint's pairs kernel deals bands out to waves
(csrc/gpp_bwd_shape.h): up to the largest band count the boundary accepts the
parts follow each other, cover every band once and cut whole groups."""
import ctypes as C
import subprocess

import pytest

from paper_2008_11326_amd import build

SHIM = """
#include "gpp_bwd_shape.h"
extern "C" int begin_of(int total, int k, int parts) { return gpp::share_begin(total, k, parts); }
extern "C" int first_band(int nb, int nocc, int group, int k, int parts)
{
    return gpp::share_first_band(nb, nocc, group, k, parts);
}
"""
MOST = 1 << 30  # GPP_MAX_NBANDS
TOTALS = sorted({0, 1, 2, 3, 4, 5, 7, 8, 63, 1000} |
                {t + d for t in (MOST >> 2, MOST >> 1, 3 * (MOST >> 2)) for d in range(-3, 4)} |
                {MOST - d for d in range(5)})


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    d = tmp_path_factory.mktemp("shape")
    (d / "shim.cpp").write_text(SHIM)
    lib = str(d / "shim.so")
    # -ftrapv: a product that passes 32 bits ends the process
    subprocess.run(["g++", "-std=c++17", "-ftrapv", "-fPIC", "-shared", "-Wall", "-Werror",
                    f"-I{build.CSRC}", str(d / "shim.cpp"), "-o", lib], check=True)
    return C.CDLL(lib)


def exact(total, k, parts):
    return total * k // parts


@pytest.mark.parametrize("parts", [1, 4])
def test_occupied_bands_are_dealt_out_once(shape, parts):
    for total in TOTALS:
        cuts = [shape.begin_of(total, k, parts) for k in range(parts + 1)]
        assert cuts == [exact(total, k, parts) for k in range(parts + 1)], total


@pytest.mark.parametrize("parts", [1, 4])
@pytest.mark.parametrize("group", [1, 2, 3, 4])
def test_unoccupied_bands_are_dealt_out_once(shape, group, parts):
    for nb in TOTALS:
        for nocc in {0, 1, nb // 3, nb - 1, nb} - {-1}:
            if nocc > nb:
                continue
            cuts = [shape.first_band(nb, nocc, group, k, parts) for k in range(parts + 1)]
            groups = -(-(nb - nocc) // group)
            assert cuts == [min(nb, nocc + exact(groups, k, parts) * group)
                            for k in range(parts + 1)], (nb, nocc)
            assert cuts[0] == nocc and cuts[-1] == nb and cuts == sorted(cuts), (nb, nocc)
            assert all((c - nocc) % group == 0 for c in cuts[:-1]), (nb, nocc)
