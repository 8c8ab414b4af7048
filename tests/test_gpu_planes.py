"""Plane stage of the 3D FFTs: the sized pencil form (planes with unequal sides, FP64 planes beyond
LDS) and square planes inside LDS against the oracle: H X and the charge density with every compiled line length along x and along y, several bands
per wave, and the allocation-free entry point where the pencil intermediate does and does not fit its
work array.  Tolerances as elsewhere: H X 1e-12 (FP64) and 2e-5 (FP32) of max|HX|, density 1e-12 and
1e-5 of its maximum."""
import numpy as np
import pytest

from oracle import pw_oracle as O
from paper_2406_10765_amd import pw, synth

pytestmark = pytest.mark.gpu

# every length once along x and once along y, never equal
GRIDS = [(24, 27, 32), (27, 32, 24), (32, 36, 27), (36, 48, 24), (48, 54, 27), (54, 64, 24), (64, 72, 24), (72, 81, 27),
         (81, 96, 24), (96, 108, 24), (108, 128, 24), (128, 144, 24), (144, 162, 24), (162, 192, 24), (192, 24, 27)]


def model_and_handle(cell, prec, nb, grid):
    # the density keeps its grids in the work blocks: room for one grid of the largest size
    m = O.model_from_cell(cell, grid=grid)
    h = pw.Handle(cell, prec, nbands=max(nb, 300), fft_n=grid)
    assert tuple(h.info.fft_n) == grid
    return m, h, pw.permutation_to(m.miller, h.gvectors())


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("prec", [pw.PW_FP64, pw.PW_MIXED])
def test_line_lengths(grid, prec):
    nb = 3
    m, h, p = model_and_handle(synth.make_cell("si8", modes=True), prec, nb, grid)
    X = synth.random_block(m.npw, nb, 5 + grid[0])
    if prec == pw.PW_MIXED:
        X = X.astype(np.complex64).astype(np.complex128)
    Xd = h.to_device(X[p])
    ref = O.apply_h(m, X)[p]
    err = float(np.abs(h.to_host(h.apply_h(Xd)) - ref).max() / np.abs(ref).max())
    occ = np.array([2.0, 0.0, 0.7])
    rho = O.density(X, occ, m.miller, m.grid).transpose(2, 1, 0)
    got = h.density(Xd, occ).cpu().numpy()
    derr = float(np.abs(got - rho).max() / rho.max())
    print("pencil grid", grid, "prec", prec, "H X", err, "density", derr, flush=True)
    assert err < (1e-12 if prec == pw.PW_FP64 else 2e-5)
    assert derr < (1e-12 if prec == pw.PW_FP64 else 1e-5)
    h.close()


@pytest.mark.parametrize("prec,nb", [(pw.PW_FP64, 33), (pw.PW_MIXED, 50)])
def test_several_bands_per_wave_and_groups(prec, nb):
    # 64 x 72 x 54: 36,288 .. waves of one band, so the x pass takes several bands per wave (nb is no multiple)
    cell = synth.silicon_cell((2, 2, 2), 8.0, nbands=nb, disp_seed=4)
    m, h, p = model_and_handle(cell, prec, nb, (64, 72, 54))
    X = synth.random_block(m.npw, nb, 8)
    if prec == pw.PW_MIXED:
        X = X.astype(np.complex64).astype(np.complex128)
    Xd = h.to_device(X[p])
    use = [0, 1, nb // 2, nb - 2, nb - 1]
    ref = O.apply_h(m, X[:, use])[p]
    err = float(np.abs(h.to_host(h.apply_h(Xd))[:, use] - ref).max() / np.abs(ref).max())
    occ = np.linspace(2.0, 0.1, nb)
    rho = O.density(X, occ, m.miller, m.grid).transpose(2, 1, 0)
    derr = float(np.abs(h.density(Xd, occ).cpu().numpy() - rho).max() / rho.max())
    print("pencil bands", nb, "prec", prec, "H X", err, "density", derr, flush=True)
    assert err < (1e-12 if prec == pw.PW_FP64 else 2e-5)
    assert derr < (1e-12 if prec == pw.PW_FP64 else 1e-5)
    h.close()


@pytest.mark.parametrize("n,prec,nb", [(24, pw.PW_MIXED, 5), (27, pw.PW_FP64, 5), (64, pw.PW_MIXED, 37), (81, pw.PW_FP64, 13),
                                       (96, pw.PW_MIXED, 11), (96, pw.PW_FP64, 3), (108, pw.PW_MIXED, 5)])
def test_square_planes_of_several_bands(n, prec, nb):
    # planes inside LDS; 64, 96, 108 (FP32) and 81, 96 (FP64) take the bands of a plane in groups
    m, h, p = model_and_handle(synth.make_cell("si8", modes=True), prec, nb, (n, n, 24))
    assert h.info.fused_planes == 1
    X = synth.random_block(m.npw, nb, n)
    if prec == pw.PW_MIXED:
        X = X.astype(np.complex64).astype(np.complex128)
    ref = O.apply_h(m, X)[p]
    err = float(np.abs(h.to_host(h.apply_h(h.to_device(X[p]))) - ref).max() / np.abs(ref).max())
    print("square plane", n, "prec", prec, "nb", nb, "H X", err, flush=True)
    assert err < (1e-12 if prec == pw.PW_FP64 else 2e-5)
    h.close()


@pytest.mark.parametrize("ncells,ecut,grid,prec", [
    ((1, 2, 2), 10.0, (0, 0, 0), pw.PW_FP64),      # the intermediate fits
    ((4, 3, 1), 12.5, (108, 81, 512), pw.PW_FP64)])  # 46 MiB a band beside the sticks: the planes stay in LDS
def test_noalloc(ncells, ecut, grid, prec):
    nb = 5
    cell = synth.silicon_cell(ncells, ecut, nbands=nb, disp_seed=4)
    h = pw.Handle(cell, prec, nbands=nb, fft_n=grid)
    X = h.random_block(nb, 3)
    ref = h.to_host(h.apply_h(X))
    out = h.empty_block(nb)
    out.fill_(float("nan"))
    h.apply_h_noalloc(X, out)
    got = h.to_host(out)
    err = float(np.abs(got - ref).max() / np.abs(ref).max())
    print("pencil noalloc", ncells, grid, err, flush=True)
    assert err < (1e-12 if prec == pw.PW_FP64 else 2e-5)
    h.close()


@pytest.mark.parametrize("prec", [pw.PW_FP64, pw.PW_MIXED])
def test_density_work_buffer_limit(prec):
    """On every route the density needs one real-space grid in the first work block, 2 ceil16(npw) nbands reals."""
    for nb in (1, 2, 3, 4, 5, 6, 9):
        cell = synth.silicon_cell((1, 1, 2), 10.0, nbands=nb, disp_seed=3)
        h = pw.Handle(cell, prec)
        n1, n2, n3 = (int(v) for v in h.info.fft_n)
        fits = 2 * ((h.npw + 15) // 16 * 16) * nb >= n1 * n2 * n3
        X = h.random_block(nb, 3)
        if fits:
            rho = h.density(X, np.ones(nb))
            assert np.isfinite(rho.cpu().numpy()).all()
        else:
            with pytest.raises(pw.PWError, match="work buffer"):
                h.density(X, np.ones(nb))
        h.close()


@pytest.mark.parametrize("n", [24, 27, 32, 48, 54, 64, 81, 96, 108, 128])
@pytest.mark.parametrize("prec", [pw.PW_FP64, pw.PW_MIXED])
def test_smallest_alias_free_grids(n, prec):
    """The largest sphere each size allows, n > 3 nmax, across the planes and along z: the blocks of grid points that
    the kernels leave out start right behind it.  H X as above."""
    nmax = (n - 1) // 3
    step = 2.0 * np.pi / 5.0  # ecut 12.5: |G| <= 5
    for grid, top in (((n, n, 24), (nmax, nmax, 7)), ((24, 24, n), (7, 7, nmax))):
        L = tuple((k + 0.4) * step for k in top)
        cell = synth.Cell(L=L, tau=np.array([[1.0, 2.0, 0.5], [0.3 * L[0], 0.6 * L[1], 3.0]]), ecut=12.5, nbands=2)
        m = O.model_from_cell(cell, grid=grid)
        assert tuple(np.abs(m.miller).max(axis=0)) == top
        h = pw.Handle(cell, prec, fft_n=grid)
        p = pw.permutation_to(m.miller, h.gvectors())
        X = synth.random_block(m.npw, 2, 5)
        if prec == pw.PW_MIXED:
            X = X.astype(np.complex64).astype(np.complex128)
        ref = O.apply_h(m, X)[p]
        err = float(np.abs(h.to_host(h.apply_h(h.to_device(X[p]))) - ref).max() / np.abs(ref).max())
        print("alias-free grid", grid, "prec", prec, "npw", m.npw, "err", err, flush=True)
        assert err < (1e-12 if prec == pw.PW_FP64 else 2e-5)
        h.close()


@pytest.mark.parametrize("n", [24, 27, 32, 48, 54, 64, 81, 96, 108])
@pytest.mark.parametrize("prec", [pw.PW_FP64, pw.PW_MIXED])
def test_density_on_square_planes(n, prec):
    """The charge density inside LDS for every compiled square plane (FP64 108: pencil passes), one band, one per
    group and several per group; tolerances as above."""
    m, h, p = model_and_handle(synth.make_cell("si8", modes=True), prec, 70, (n, n, 24))
    X = synth.random_block(m.npw, 70, 3 + n)
    if prec == pw.PW_MIXED:
        X = X.astype(np.complex64).astype(np.complex128)
    for nb in (1, 3, 70):
        occ = np.linspace(2.0, 0.1, nb)
        rho = O.density(X[:, :nb], occ, m.miller, m.grid).transpose(2, 1, 0)
        err = float(np.abs(h.density(h.to_device(X[p][:, :nb]), occ).cpu().numpy() - rho).max() / rho.max())
        print("density plane", n, "prec", prec, "nb", nb, "err", err, flush=True)
        assert err < (1e-12 if prec == pw.PW_FP64 else 1e-5)
    h.close()
