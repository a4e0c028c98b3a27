"""The adjoint's rows of many tiles: a lane's sums are set aside every 256 of its events, at 64
points from 4 x 4096 tiles on.  Around that edge and well past it, against the oracle's dual
numbers with the bars of the adjoint's parity tests (sigma 1e-10, gradient 1e-9 relative plus
1e-12 sigma / |theta|); and the point alone, whose 64 groups have other stretches, agrees to the
rounding of the orders: chains of at most 256 + 64 + 16 additions in blocks of 4096 rows and a
tree of 256, 6e-14 relative at worst for the sum of one sign."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4 * 4096 * 64, 4 * 4096 * 64 + 1, 5_000_000])
def test_rows_of_many_tiles(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    cfg = W.config("dy_z")
    g = P.Integrator(cfg["process"], 3, cfg["nbins"], cfg["seed"], cfg["alpha"], cfg["params"], max_events=10_000)
    for _ in range(3):
        g.iterate(10_000)
        g.refine()
    o = oracle.Vegas(cfg["process"], 3, cfg["nbins"], cfg["seed"], cfg["alpha"], cfg["params"])
    o.set_grid(g.get_grid())
    theta = W.adjoint_points(64, seed=5)
    sig, ds = (t.cpu().numpy() for t in g.grad(torch.tensor(theta), n, 3))
    b = 7
    so, dso = o.dy_grad(3, n, theta[b])
    assert abs(sig[b] / so - 1) < 1e-10
    assert np.all(np.abs(ds[b] - dso) <= 1e-9 * np.abs(dso) + 1e-12 * so / np.abs(theta[b])), (ds[b], dso)
    for B in (1, 5, 33):
        one, _ = (t.cpu().numpy() for t in g.grad(torch.tensor(theta[b:b + B]), n, 3))
        assert abs(one[0] / sig[b] - 1) < 6e-14, B
    g.close()
