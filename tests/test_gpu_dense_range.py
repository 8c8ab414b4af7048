"""Rayleigh-Ritz of nearly decoupled plane waves: off-diagonal entries of the projected H whose squares underflow
(1e-156 and below, down to denormal numbers) leave the eigenvalues at the kinetic energies and the vectors orthonormal."""
import numpy as np
import pytest

from paper_2406_10765_amd import pw, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [4, 50, 144])
@pytest.mark.parametrize("amp", [1e-100, 1e-136, 1e-156, 1e-162, 1e-170, 1e-250, 1e-310])
def test_tiny_couplings(amp, nb):
    modes = synth.Modes(miller=np.array([[1, 0, 0], [0, 1, 1], [1, 1, 0]]), amp=np.array([1.0, 0.7, 0.4]) * amp,
                        phase=np.array([0.9, -0.4, 2.0]))
    cell = synth.Cell(L=(9.0, 10.26, 11.5), tau=np.zeros((0, 3)), ecut=9.0, nbands=nb, modes=modes)
    h = pw.Handle(cell, pw.PW_FP64)
    g = h.gvectors()
    kin = 0.5 * ((2.0 * np.pi * g / np.array(cell.L)) ** 2).sum(axis=1)
    rows = np.sort(np.argsort(kin, kind="stable")[:nb])  # whole shells of coupled neighbours, in no order of energy
    X = np.zeros((h.npw, nb), complex)
    X[rows, np.arange(nb)] = np.exp(1j * np.arange(nb))
    Xd = h.to_device(X)
    eig, resid, _ = h.eig_step(Xd, 0, -0.8, 1.0, 17.0)
    got = h.to_host(Xd)
    e1 = float(np.abs(eig - np.sort(kin[rows])).max())
    e2 = float(np.abs(got.conj().T @ got - np.eye(nb)).max())
    print("couplings", amp, "nb", nb, "eig", e1, "orthonormality", e2, "residual", float(resid.max()), flush=True)
    # kinetic energies up to 4 Ha, one rounding each and those of the products: 1e-13
    assert e1 < 1e-13 and e2 < 1e-13 and resid.max() < 1e-13
    h.close()
