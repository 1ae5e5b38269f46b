"""The Poisson CG's kernels, which take two nodes of a z-row per thread, iterate by
iterate against the plain numpy restatement of the preconditioned iteration: the
smallest pair, rows shorter and longer than a wave's 64 pairs (a row's neighbours then
come from another lane or are fetched by the wave's end lanes), rows of whole waves,
odd nx and ny (ragged aggregates), and rows of odd length, whose last pair has one node."""

import numpy as np
import pytest

from test_gpu_poisson_mg import _box, _pcg

SHAPES = [(2, 1, 2), (5, 3, 2), (3, 2, 34), (9, 7, 130), (4, 5, 256), (37, 29, 24), (21, 18, 22),
          (6, 5, 1), (4, 3, 3), (9, 7, 131), (5, 6, 127)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_pair_kernels_match_restatement(shape):
    import paper_2607_08447_amd as hkp
    import torch
    eps, dirichlet, phi_fixed, rho = _box(shape, 11 + sum(shape))
    t = lambda v: torch.from_numpy(np.ascontiguousarray(v))
    for iters in (1, 3):
        print(f"pairs {shape} iterations {iters}", flush=True)
        ref, rel_ref, _ = _pcg(shape, 0.4, eps, dirichlet, phi_fixed, rho, iters)
        if rel_ref < 1e-10:   # solved already: further directions are rounding
            continue
        phi, it, rel, _ = hkp.poisson(t(eps), t(dirichlet), t(phi_fixed), t(rho), 0.4,
                                      tol=1e-30, max_iter=iters)
        assert it == iters
        # rounding only: a few thousand operations of 1e-16 on either side
        assert np.abs(phi.cpu().numpy() - ref).max() <= 1e-9 * np.abs(ref).max()
        assert abs(rel - rel_ref) <= 1e-8 * rel_ref + 1e-12
