"""The adjoint's split of the work: event groups per wave (floor(64 / B) of them), ragged
tiles, rows of one and of several tiles.  Against the oracle's dual numbers with the bars
of the adjoint's own parity tests (sigma 1e-10, gradient 1e-9 relative plus 1e-12 sigma /
|theta|), and a point alone against the same point in a batch: the sums differ in order
only (below 1e-12 relative: at most 2e6 additions of one sign in blocked order, each
rounding 1.1e-16; the derivatives' terms change sign, so their bar is relative to
sigma / |theta| or the derivative, whichever is larger)."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
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
    return g, o, torch


@pytest.mark.parametrize("B", [1, 2, 3, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 4097, 600_001])
def test_rows_and_groups(setup, B, n):
    g, o, torch = setup
    theta = W.adjoint_points(B, seed=5)
    sig, ds = (t.cpu().numpy() for t in g.grad(torch.tensor(theta), n, 3))
    b = B - 1
    scale = np.maximum(np.abs(ds[b]), sig[b] / np.abs(theta[b]))
    one, done = (t.cpu().numpy() for t in g.grad(torch.tensor(theta[b:b + 1]), n, 3))
    assert abs(one[0] / sig[b] - 1) < 1e-12
    assert np.all(np.abs(done[0] - ds[b]) <= 1e-12 * scale), (done[0], ds[b])
    if n < 100_000 or B in (3, 64):
        so, dso = o.dy_grad(3, n, theta[b])
        assert abs(sig[b] / so - 1) < 1e-10
        assert np.all(np.abs(ds[b] - dso) <= 1e-9 * np.abs(dso) + 1e-12 * so / np.abs(theta[b])), (ds[b], dso)


def test_exponents_out_of_the_fast_range(setup):
    """|a| above 1e4 takes the library exponential for the wave: a^2 factors that underflow
    give exact zeros, and a not-a-number parameter stays one in its own point only."""
    g, _, torch = setup
    theta = np.repeat(W.adjoint_points(1, seed=5), 3, axis=0)
    theta[1, 3] = 2.0e4       # tau^a underflows for every event
    theta[2, 3] = np.nan
    sig, ds = (t.cpu().numpy() for t in g.grad(torch.tensor(theta), 1000, 3))
    ref, _ = (t.cpu().numpy() for t in g.grad(torch.tensor(theta[:1]), 1000, 3))
    assert abs(sig[0] / ref[0] - 1) < 1e-12
    assert sig[1] == 0.0 and np.all(ds[1] == 0.0)
    assert np.isnan(sig[2]) and np.isnan(ds[2]).all()
