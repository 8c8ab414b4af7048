"""Address arithmetic of the projector products on pairs, checked on the host over every load of the
first and last K tile of every workgroup tile (all four projection shapes, both nonlocal row tiles),
and the order of the sphere's rows that the pairs rest on.  CPU only."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2406_10765_amd import pw, synth

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("pairs") / "pairs_bounds")
    subprocess.run([cxx, "-O2", "-std=c++17", os.path.join(HERE, "pairs_bounds.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("npw,nproj,nb", [(1, 4, 1), (3, 4, 2), (31, 12, 5), (33, 32, 17), (1647, 32, 20),
                                          (9315, 256, 129), (37073, 256, 144), (80725, 864, 440), (295667, 2048, 1088)])
def test_loads_in_bounds(harness, npw, nproj, nb):
    r = subprocess.run([harness, str(npw), str(nproj), str(nb)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("cell", [synth.make_cell("si8"), synth.silicon_cell((1, 2, 3), 17.0),
                                  synth.Cell(L=(9.0, 10.26, 11.5), tau=np.zeros((1, 3)), ecut=7.3, nbands=4)])
def test_row_order_reverses_under_negation(cell):
    g = pw.plan_gvectors(cell)
    assert g.shape[0] % 2 == 1
    assert np.array_equal(g[::-1], -g)
