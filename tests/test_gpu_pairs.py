"""Projector products on pairs (G, -G): every tile shape of the projection and the nonlocal product
with remainders in bands, plane waves and projectors, in split-bf16, FP32 and FP64, with the table
stored or generated and both projector families; the scalar epilogue of unaligned blocks, and the
planes buffer shared by blocks of different widths.

Tolerances of H X relative to max|HX|, as for the same arithmetic elsewhere: 5e-5 with split-bf16
products (each product's split residual is at most 2^-16, with random signs), 2e-5 in FP32, 1e-12 in
FP64.  The reference is the FP64 oracle on the same (FP32-rounded) input."""
import numpy as np
import pytest

from oracle import pw_oracle as O
from paper_2406_10765_amd import pw, synth

pytestmark = pytest.mark.gpu


def cell_with_atoms(n, L=(9.0, 10.26, 11.5), ecut=9.0, nbands=40):
    rng = np.random.Generator(np.random.PCG64(7))
    return synth.Cell(L=L, tau=rng.uniform(0, 1, (n, 3)) * np.array(L), ecut=ecut, nbands=nbands)


def check(cell, nbs, ld_extra=None, cols=None, prec=pw.PW_MIXED, flags=pw.PW_FLAG_BF16_ALL, form=pw.PW_PROJ_GSPACE):
    tol = 1e-12 if prec == pw.PW_FP64 else 5e-5 if flags & pw.PW_FLAG_BF16_KB else 2e-5
    m = O.model_from_cell(cell, proj_form=O.PROJ_LOCALIZED) if form else O.model_from_cell(cell)
    h = pw.Handle(cell, prec, flags=flags, proj_form=form)
    perm = pw.permutation_to(m.miller, h.gvectors())
    for nb in nbs:
        X = synth.random_block(h.npw, nb, 11 + nb)
        X = X if prec == pw.PW_FP64 else X.astype(np.complex64)
        ld = None if ld_extra is None else h.npw + ld_extra
        Xd = h.to_device(X, ld)
        got = h.to_host(h.apply_h(Xd))
        use = range(nb) if cols is None else sorted({0, nb // 2, nb - 1})
        inv = np.argsort(perm)
        ref = O.apply_h(m, X[inv][:, list(use)].astype(np.complex128))[perm]
        err = float(np.abs(got[:, list(use)] - ref).max() / np.abs(ref).max())
        print("pairs npw", h.npw, "nproj", h.info.nproj, "nb", nb, "ld_extra", ld_extra, "err", err, flush=True)
        assert err <= tol
    h.close()


@pytest.mark.parametrize("natoms", [0, 1, 3, 8, 9])
def test_projector_and_row_remainders(natoms):
    check(cell_with_atoms(natoms), (1, 16, 17, 33, 40))


@pytest.mark.parametrize("prec,flags,form", [(pw.PW_FP64, 0, 0), (pw.PW_FP64, pw.PW_FLAG_BETA_OTF, 0), (pw.PW_FP64, 0, 1),
                                             (pw.PW_MIXED, 0, 0), (pw.PW_MIXED, pw.PW_FLAG_BETA_OTF, 0),
                                             (pw.PW_MIXED, pw.PW_FLAG_BF16_KB, 1)])
@pytest.mark.parametrize("natoms", [0, 3, 17])
def test_precisions_tables_and_families(prec, flags, form, natoms):
    # 68 projectors: 128-row tiles with a remainder; 12: 64-row tiles; widths 16, 32, 48 and 64
    check(cell_with_atoms(natoms), (1, 17, 40) if natoms else (17,), prec=prec, flags=flags, form=form)
    if natoms == 17:
        check(cell_with_atoms(natoms, nbands=101), (48, 64, 101), prec=prec, flags=flags, form=form, cols=3)


@pytest.mark.parametrize("ecut", [6.0, 8.0])
def test_projection_tile_shapes(ecut):
    # 256 projectors: the narrow shape (<= 16 bands) and 64 x 32; nonlocal tiles of 64 x 48 and 64 x 64
    check(synth.silicon_cell((2, 2, 2), ecut, nbands=129, disp_seed=5), (1, 15, 16, 17, 47, 48, 63, 65, 129), cols=3)


def test_largest_tiles_with_remainders():
    # 864 projectors x 153 bands: 256 x 128 projection tiles, x 77 .. 95: 128 x 64; 249 bands x 257 row tiles: 128 x 128
    # nonlocal tiles
    check(synth.silicon_cell((3, 3, 3), 6.0, nbands=153, disp_seed=5), (77, 95, 152, 153), cols=3)
    check(synth.silicon_cell((3, 3, 4), 11.5, nbands=251, disp_seed=6), (249, 251), cols=3)
    check(synth.silicon_cell((3, 3, 4), 11.5, nbands=131, disp_seed=6), (129, 131), cols=3)


@pytest.mark.parametrize("ld_extra", [0, 1, 2, 3])
def test_block_alignments(ld_extra):
    check(synth.silicon_cell((1, 1, 2), 9.0, nbands=19, disp_seed=5), (3, 19), ld_extra=ld_extra)


@pytest.mark.parametrize("degree", [0, 1, 2, 5])
def test_steps_of_different_widths_share_the_planes(degree):
    """A step on a handle that has just processed a wider or narrower block gives bitwise what a new handle gives:
    nothing of the earlier block's planes is read."""
    cell = synth.silicon_cell((1, 1, 2), 10.0, nbands=40, disp_seed=3)
    flags = pw.PW_FLAG_BF16_ALL

    def step(h, nb):
        X = h.random_block(nb, 9)
        e, r, _ = h.eig_step(X, degree, -0.8, 1.0, 17.0)
        return e, r, h.to_host(X)

    h = pw.Handle(cell, pw.PW_MIXED, flags=flags)
    for nb in (40, 23, 36, 40):
        got = step(h, nb)
        new = pw.Handle(cell, pw.PW_MIXED, flags=flags)
        ref = step(new, nb)
        new.close()
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), (degree, nb)
    h.close()


@pytest.mark.parametrize("prec", [pw.PW_FP64, pw.PW_MIXED])
@pytest.mark.parametrize("nbands,ld_extra", [(17, 0), (49, 1), (101, 2), (145, 0)])
def test_gram_and_rotation_tiles(prec, nbands, ld_extra):
    """Rayleigh-Ritz alone (degree 0) over the tiles of the complex products, their remainders in bands, rows and K
    values, the Gram tiles left out below the diagonal, and both dense solvers (one workgroup from 4 to 144 bands, rows
    in steps of 48 and 64): Ritz values as the FP64 oracle's, X^H X = I.  Relative
    tolerances: 1e-11 in FP64 and 2e-5 in FP32, the accuracy of H X with a margin for the FP64 solve."""
    tol = 1e-11 if prec == pw.PW_FP64 else 2e-5
    cell = cell_with_atoms(3, nbands=nbands)
    m = O.model_from_cell(cell)
    h = pw.Handle(cell, prec, flags=0)
    inv = np.argsort(pw.permutation_to(m.miller, h.gvectors()))
    for nb in {17: (1, 2, 3, 4, 5, 15, 16, 17), 49: (31, 32, 33, 47, 48, 49), 101: (63, 64, 65, 80, 95, 96, 97, 101),
               145: (127, 128, 129, 143, 144, 145)}[nbands]:
        X = synth.random_block(h.npw, nb, 3 + nb)
        X = X if prec == pw.PW_FP64 else X.astype(np.complex64)
        Xd = h.to_device(X, h.npw + ld_extra)
        eig, _, _ = h.eig_step(Xd, 0, -0.8, 1.0, 17.0)
        Y = X[inv].astype(np.complex128)
        ref = O.rayleigh_ritz(Y, O.apply_h(m, Y))[0]
        got = h.to_host(Xd).astype(np.complex128)
        e1 = float(np.abs(eig - ref).max() / np.abs(ref).max())
        e2 = float(np.abs(got.conj().T @ got - np.eye(nb)).max())
        print("npw", h.npw, "nb", nb, "eig", e1, "orthonormality", e2, flush=True)
        assert e1 <= tol and e2 <= tol
    h.close()
