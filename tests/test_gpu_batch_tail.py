"""A large batch whose members end at different iterations: most start near their
eigenvectors, three from random blocks, so that the last iterations run for a few members
of a work table made for all (host-counted launches, and iterations recorded anew for the
members left).  Eigenvalues against each member's own single solve."""

import numpy as np
import pytest

from test_gpu_batch import _sweep

pytestmark = pytest.mark.gpu

MEMBERS, SLOW, NEV, NB = 60, (0, 31, 59), 6, 16


@pytest.fixture(scope="module")
def batch():
    import torch
    import paper_2607_08447_amd as hkp
    w, _ = _sweep(1)
    x = np.linspace(-1.0, 1.0, w.shape[0])[:, None, None]
    Vs = np.stack([w.V + 1e-3 * k * x ** 2 for k in range(MEMBERS)])
    S = torch.from_numpy(w.strain)
    solo = [hkp.solve(torch.from_numpy(V), w.h, NEV, strain=S, B=w.B, nb=NB, tol=1e-10,
                      psi_block=True) for V in Vs]
    assert all(r.status == 0 for r in solo)
    g = torch.Generator(device="cuda").manual_seed(3)
    X0 = torch.stack([r.psi for r in solo])
    noise = torch.randn(X0.shape, dtype=X0.dtype, device="cuda", generator=g)
    X0 = X0 + 1e-3 * noise / noise[0, 0].norm()
    for k in SLOW:
        X0[k] = noise[k]
    return w, Vs, S, X0, np.stack([r.E.cpu().numpy() for r in solo])


@pytest.mark.parametrize("graph", [False, True], ids=["eager", "graph"])
@pytest.mark.parametrize("precision,tol,product", [("fp64", 1e-9, False), ("mixed", 1e-9, False),
                                                   ("mixed", 1e-9, True)])
@pytest.mark.parametrize("degree", [0, 24])
def test_last_members_of_a_batch(batch, degree, precision, tol, product, graph):
    import torch
    import paper_2607_08447_amd as hkp
    w, Vs, S, X0, E = batch
    print(f"batch tail {precision} product {product} graph {graph} degree {degree}", flush=True)
    counts = []
    r = hkp.solve_batch(torch.from_numpy(Vs), w.h, NEV, strain=S, B=w.B, nb=NB, tol=tol, X0=X0,
                        precision=precision, cheb_product=product, graph=graph, degree=degree,
                        max_iter=100, callback=lambda i: counts.append(i["nconv"]))
    assert r.status == 0
    assert np.abs(r.E.cpu().numpy() - E).max() <= 1e-8
    assert float(r.resid.max()) <= tol
    done = [int((n == NEV).sum()) for n in counts]
    print("members done after each iteration", done, flush=True)
    assert MEMBERS - 15 <= done[-2] < MEMBERS   # the end was a few members' alone


def test_steps_counted_are_steps_run(batch):
    """The FP32 filter's timed steps are those of the iterations in which a member was
    filtered in FP32; once all are in FP64 there are none."""
    import torch
    import paper_2607_08447_amd as hkp
    w, Vs, S, X0, _ = batch
    print("batch tail counted steps", flush=True)
    rows = []
    r = hkp.solve_batch(torch.from_numpy(Vs), w.h, NEV, strain=S, B=w.B, nb=NB, tol=1e-9, X0=X0,
                        precision="mixed", graph=False, degree=24, max_iter=100,
                        callback=lambda i: rows.append((i["nconv"], i["fp64"])))
    assert r.status == 0
    in32 = [bool(((n < NEV) & (f == 0)).any()) for n, f in rows]   # before the next iteration
    assert not all(in32[:-1])
    assert 0 < r.stats["n_stencil32"] <= 23 * (1 + sum(in32))
