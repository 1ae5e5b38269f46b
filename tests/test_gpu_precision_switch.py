"""When a mixed-precision solve leaves FP32 filtering: always for a target below what
FP32 can reach (about 5e-6 eV here), never for one far above it, in either filter form.

A residual of r puts an eigenvalue within r of each Ritz value, so the energies have to
agree with the dense oracle's to the target."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def well():
    from oracle import SI_MATERIAL, Grid, hamiltonian_ls, lowest_dense
    from synth import workload
    w = workload("harmonic_10x8x8")
    E, _ = lowest_dense(hamiltonian_ls(Grid(w.nx, w.ny, w.nz, w.h), SI_MATERIAL, w.V), 12)
    return w, E


@pytest.mark.gpu
@pytest.mark.parametrize("product", [True, False], ids=["product", "recurrence"])
@pytest.mark.parametrize("graph", [False, True], ids=["eager", "graph"])
@pytest.mark.parametrize("tol,switches", [(1e-8, True), (1e-7, True), (1e-4, False)])
def test_switch_follows_the_target(well, tol, switches, product, graph):
    import paper_2607_08447_amd as hkp
    w, E = well
    print(f"tol {tol} product {product} graph {graph}", flush=True)
    r = hkp.solve(torch.from_numpy(w.V).cuda(), w.h, 12, tol=tol, precision="mixed",
                  cheb_product=product, graph=graph)
    assert r.status == 0 and r.stats["n_hx_fp32"] > 0
    assert (r.stats["fp64_switch_iter"] >= 0) == switches
    assert float(r.resid.max()) <= tol
    assert np.abs(r.E.cpu().numpy() - E[:12]).max() <= tol
