"""Systems solved four to a workgroup (the configuration interaction's pair potentials on
boxes of more than some 1e5 nodes) against single solves of the same densities.

Two orbitals give 6 systems and five give 30, so the last group has two; the densities
|phi_i|^2 are real, so their imaginary parts are finished members from the start; the others
end at different iterations.  Odd box sides (ragged aggregates, rows with a one-node
pair); with five orbitals the first coarse level is solved in groups as well.

Both sides stop at |r| <= 1e-13 |b|.  A Coulomb integral rho . V moves by at most |V| |r|,
some 1e2 times 1e-13 of its size; the bar is the one of the comparison with the oracle."""

import numpy as np
import pytest

from oracle import coulomb_integrals, pair_densities
from test_gpu_poisson_mg import _box

PSHAPE, SHAPE, OFFSET, H = (131, 64, 65), (37, 24, 21), (40, 17, 19), 0.4


def _orbitals(M):
    """Orthonormal smooth complex three-component functions."""
    rng = np.random.default_rng(M)
    ax = [np.linspace(0.0, 1.0, n + 2)[1:-1] for n in SHAPE]
    x, y, z = np.meshgrid(*ax, indexing="ij")
    cols = []
    for _ in range(M):
        f = np.zeros(SHAPE + (3,), dtype=complex)
        for _ in range(6):
            k = rng.integers(1, 4, 3)
            mode = np.sin(np.pi * k[0] * x) * np.sin(np.pi * k[1] * y) * np.sin(np.pi * k[2] * z)
            f += mode[..., None] * (rng.normal(size=3) + 1j * rng.normal(size=3))
        cols.append(f.ravel())
    q, _ = np.linalg.qr(np.stack(cols, axis=1))
    return q


@pytest.mark.gpu
@pytest.mark.parametrize("M", [2, 5])
def test_grouped_systems_match_single_solves(M):
    import torch
    import paper_2607_08447_amd as hkp
    t = lambda v: torch.from_numpy(np.ascontiguousarray(v))
    eps, dirichlet, _, _ = _box(PSHAPE, 5)
    phi = _orbitals(M)
    print(f"groups M {M} box {PSHAPE}", flush=True)
    ci = hkp.ci_solve(t(phi.T.reshape((M,) + SHAPE + (3,))), t(np.arange(M) * 1e-3), H, PSHAPE,
                      OFFSET, t(eps), t(dirichlet), cg_tol=1e-13, return_coulomb=True)
    assert ci.status == 0
    rho = pair_densities(phi, SHAPE, H)
    inner = tuple(slice(o, o + n) for o, n in zip(OFFSET, SHAPE))
    eps_d, dir_d, zero = t(eps).cuda(), t(dirichlet).cuda(), torch.zeros(PSHAPE).double().cuda()

    def potential(r):
        box = np.zeros(PSHAPE)
        box[inner] = r
        V, _, _, code = hkp.poisson(eps_d, dir_d, zero, t(box), H, tol=1e-13)
        assert code == 0
        return V.cpu().numpy()

    V = np.zeros((M, M) + PSHAPE, dtype=complex)
    for i in range(M):
        for k in range(i, M):
            V[i, k] = potential(rho[i, k].real)
            if k > i:
                V[i, k] += 1j * potential(rho[i, k].imag)
                V[k, i] = V[i, k].conj()
    C = coulomb_integrals(rho, V, SHAPE, OFFSET, H)
    err = np.abs(ci.coulomb.cpu().numpy() - C).max() / np.abs(C).max()
    print(f"M {M}: max |dC| / max |C| {err:.2e}", flush=True)
    assert err <= 1e-9
