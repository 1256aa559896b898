"""The reaction scratch of the lane-group integrators (no GPU): what the
mechanism's handle holds in global memory is decided when it is loaded, what a
launch uses when it is made, and the two have to agree for every mechanism.
The library's own functions are called from a small program, over all species
counts and over the reaction counts around every limit, with and without
pressure-dependent reactions."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2312_13513_amd")

MAIN = r"""
#include <cstdio>
#include "bdf_wave.h"

// "K R n_pdep uses-global(64) uses-global(16) slots" per mechanism
int main()
{
    for (int K = 1; K <= 63; K++)
        for (int R = 0; R <= 2000; R++)
            for (int n_pdep = 0; n_pdep <= 1 && n_pdep <= R; n_pdep++)
                for (int table = 4096; table <= 24576; table += 20480) {
                    chem::DevMechView m{};
                    chem::set_view_sizes(m, K, R, n_pdep, table);
                    const bool w = chem::wave_uses_global_scratch(m, 64);
                    const bool t = K + 1 <= 16 && chem::wave_uses_global_scratch(m, 16);
                    std::printf("%d %d %d %d %d %d\n", K, R, n_pdep, w, t,
                                chem::wave_scratch_slots(m, size_t(1) << 28));
                }
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    import numpy as np

    from paper_2312_13513_amd import chem
    chem.lib()
    d = tmp_path_factory.mktemp("scratch")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), str(src), "-o", str(exe),
                    os.path.join(PKG, "libchem.so"), "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib", "-L",
                    "/opt/rocm/lib", "-lamdhip64"], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120).stdout
    return np.array([[int(x) for x in line.split()] for line in out.splitlines()])


def test_scratch_is_held_where_a_launch_uses_it(rows):
    used = (rows[:, 3] | rows[:, 4]).astype(bool)
    assert (rows[used, 5] >= 64).all() and (rows[used, 5] <= 4096).all()
    assert (rows[~used, 5] == 0).all()


def test_limits_of_the_wave_kernel(rows):
    """The reaction counts from which the wave kernel's scratch is in global
    memory; the GPU tests of that kernel rely on them."""
    for pdep, first in ((0, 878), (1, 769)):
        r = rows[(rows[:, 0] > 15) & (rows[:, 2] == pdep)]
        assert (r[:, 3] == (r[:, 1] >= first)).all()
