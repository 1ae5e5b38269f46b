"""The Poisson CG's kernels on both sides of the size (65536 threads) below which their
workgroups are single waves, iterate by iterate against the plain numpy restatement, at the
bars of the smaller boxes.  On the larger one the finest level runs in workgroups of four
waves and the coarse levels in single waves."""

import numpy as np
import pytest

from test_gpu_poisson_mg import _box, _pcg

SHAPES = [(60, 43, 47), (67, 45, 47)]   # 61920 and 72360 pairs of nodes


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_workgroup_sizes_match_restatement(shape):
    import paper_2607_08447_amd as hkp
    import torch
    eps, dirichlet, phi_fixed, rho = _box(shape, 23)
    t = lambda v: torch.from_numpy(np.ascontiguousarray(v))
    for iters in (1, 3):
        print(f"share {shape} iterations {iters}", flush=True)
        ref, rel_ref, _ = _pcg(shape, 0.4, eps, dirichlet, phi_fixed, rho, iters)
        phi, it, rel, _ = hkp.poisson(t(eps), t(dirichlet), t(phi_fixed), t(rho), 0.4,
                                      tol=1e-30, max_iter=iters)
        assert it == iters
        assert np.abs(phi.cpu().numpy() - ref).max() <= 1e-9 * np.abs(ref).max()
        assert abs(rel - rel_ref) <= 1e-8 * rel_ref + 1e-12
