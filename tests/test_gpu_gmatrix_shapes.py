"""g-matrices on boxes around the edges of the weighted stencil's tiles and of the Gram
product's chunks of points (fewer points than a wave takes, no whole number of them, one
or several tiles along x), for arbitrary orthonormal states: the doublets of the input
basis and their centres against the oracle's numerical field derivative, at the bar of
the g-matrix comparison on solved states (1e-8 relative)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (5, 3, 3), (16, 4, 3), (17, 4, 3), (33, 6, 2), (32, 9, 5), (64, 5, 4)]


@pytest.mark.parametrize("strained", [False, True], ids=["free", "strained"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_g_matrices_of_arbitrary_states(shape, strained):
    import paper_2607_08447_amd as hkp
    from oracle import SI_MATERIAL, Grid
    from oracle.gmatrix import double_dot_g
    rng = np.random.default_rng(sum(shape))
    n = int(np.prod(shape))
    psi, _ = np.linalg.qr(rng.normal(size=(6 * n, 4)) + 1j * rng.normal(size=(6 * n, 4)))
    V = rng.uniform(0.0, 0.1, shape)
    strain = rng.uniform(-1e-3, 1e-3, shape + (6,)) if strained else None
    print(f"g-matrices {shape} strained {strained}", flush=True)
    t = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a))
    gm = hkp.g_matrices(t(psi.T.reshape(4, *shape, 6)), t(V), 0.5, strain=t(strain))
    ref = double_dot_g(Grid(*shape, 0.5), SI_MATERIAL, psi, gm.E, V.ravel(),
                       None if strain is None else strain.reshape(-1, 6))
    scale = max(np.abs(ref["g"][0]).max(), np.abs(ref["g"][1]).max())
    for k in (0, 1):
        assert np.abs(gm.g[k] - ref["g"][k]).max() <= 1e-8 * scale, k
        assert np.abs(gm.centre[k] - ref["centre"][k]).max() <= 1e-9
