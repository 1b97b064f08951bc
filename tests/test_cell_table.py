"""The table of occupied cells (csrc/tlsph_internal.h), compiled for the host:
slots visited per cell when the cells of many specimens, of a plate, a bar and
a line are put into it, at most half full as the build makes it.  Host only."""
import ctypes as C
import os
import subprocess

import pytest

from paper_1901_07374_amd import build as B

SOURCE = r"""
#include <vector>
#include "tlsph_internal.h"
using namespace tlsph;
extern "C" double probes(int specs, int nx, int ny, int nz) {
    const int64_t n = (int64_t)specs * nx * ny * nz;
    int64_t H = 2, visited = 0;
    while (H < 2 * n) H <<= 1;
    std::vector<char> used(H, 0);
    for (int s = 0; s < specs; ++s)
        for (int z = 0; z < nz; ++z)
            for (int y = 0; y < ny; ++y)
                for (int x = 0; x < nx; ++x) {
                    int64_t h = cell_home(grid_key(s, x, y, z), table_shift(H));
                    for (++visited; used[h]; ++visited) h = (h + 1) & (H - 1);
                    used[h] = 1;
                }
    return (double)visited / n;
}
"""


@pytest.fixture(scope="module")
def probes(tmp_path_factory):
    d = tmp_path_factory.mktemp("cells")
    src = d / "cells.hip"
    src.write_text(SOURCE)
    so = str(d / "cells.so")
    subprocess.check_call([B.HIPCC, "--cuda-host-only", "-x", "hip", "-O2", "-std=c++17", "-fPIC",
                           "-shared", "-w", "-I", os.path.join(B.HERE, "csrc"), "-o", so, str(src)])
    lib = C.CDLL(so)
    lib.probes.restype = C.c_double
    return lib.probes


@pytest.mark.parametrize("specs,nx,ny,nz", [(70000, 2, 2, 2), (2000, 5, 5, 5), (64, 12, 12, 40),
                                            (1, 5, 107, 267), (1, 32, 32, 200), (1, 2, 2, 12000)])
def test_cells_spread_over_the_table(probes, specs, nx, ny, nz):
    # a random hash visits 1.5 slots at half full; lattices lie around that
    assert probes(specs, nx, ny, nz) < 4.0
