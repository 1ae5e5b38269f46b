"""The dense nb x nb part of the iteration: Cholesky or SVQB orthonormalisation
and the Rayleigh-Ritz step in one launch or (large blocks) in several.

Block sizes sit on both sides of the one-launch limit (48), odd and even; the
starting blocks put the first Gram matrix on both sides of the conditioning
limit.  The tolerance is the FP64 solves' own (residual 1e-9 eV, eigenvalues
quadratic in it, so 1e-8 eV is far above any rounding)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def well():
    from oracle import SI_MATERIAL, Grid, hamiltonian_ls, lowest_dense
    from synth import workload
    w = workload("harmonic_10x8x8")
    E, _ = lowest_dense(hamiltonian_ls(Grid(w.nx, w.ny, w.nz, w.h), SI_MATERIAL, w.V), 48)
    return w, E


@pytest.mark.parametrize("nev,nb", [(1, 4), (4, 9), (30, 47), (32, 48), (33, 49), (48, 64)])
def test_block_sizes_around_the_one_launch_limit(well, nev, nb):
    import paper_2607_08447_amd as hkp
    w, E = well
    print(f"nev {nev} nb {nb}", flush=True)
    r = hkp.solve(torch.from_numpy(w.V).cuda(), w.h, nev, nb=nb, tol=1e-9)
    assert r.status == 0
    assert np.abs(r.E.cpu().numpy() - E[:nev]).max() <= 1e-8


@pytest.mark.parametrize("angle", [1.0, 1e-2, 1e-3, 1e-5])
def test_conditioning_of_the_first_block(well, angle):
    """Columns in pairs at a small angle: the Gram matrix's condition is ~ 4 / angle^2, so
    1 takes the triangular factor and 1e-3 on the eigen-decomposition and a second pass;
    the states and the orthonormality of psi must not depend on it."""
    import paper_2607_08447_amd as hkp
    w, E = well
    g = np.random.Generator(np.random.PCG64(7))
    shape = (16, w.nx, w.ny, w.nz, 6)
    X = g.standard_normal(shape) + 1j * g.standard_normal(shape)
    X[1::2] = X[0::2] + angle * X[1::2]
    print(f"angle {angle}", flush=True)
    r = hkp.solve(torch.from_numpy(w.V).cuda(), w.h, 8, X0=torch.from_numpy(X), tol=1e-9)
    assert r.status == 0
    assert np.abs(r.E.cpu().numpy() - E[:8]).max() <= 1e-8
    p = r.psi.reshape(8, -1)
    gram = (p.conj() @ p.T).cpu().numpy()
    assert np.abs(gram - np.eye(8)).max() <= 1e-10
