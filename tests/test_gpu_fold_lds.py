"""The fused fold at the largest grids that its rule allows (10 and more dimensions, with and
without an observable, where an event block takes the most LDS), with blocks of a full CU: the
iterations fold in the event kernel (or, where the largest weight left the window of the
scale it folded at, again from the records: fold 1 or 2) and give the bytes of single-wave
blocks.  One bin more is folded from the records alone (fold 0)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

N = 300_000  # more events than 256 full blocks hold at one chunk per wave


def rule(D, n, obs):
    """Whether the row's digits, a grid and 256 lanes' sums are within 64 KB (D >= 10)."""
    return 8 * D * (n + 1) + 8 * (7 + 4 * D * n + (7 * (obs + 2) if obs else 0)) + 8 * 7 * 256 <= 65536


@pytest.mark.parametrize("process,D", [(W.WW_HAD, 10), (W.GAUSS, 10), (W.GAUSS, 15), (W.GENZ, 16)])
@pytest.mark.parametrize("obs", [0, 100, 254])
def test_fused_fold_at_the_largest_grid(process, D, obs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    par = {W.WW_HAD: W.config("ww_had")["params"], W.GAUSS: [0.5, 2.0], W.GENZ: W.genz_params(3, D)}[process]
    nbins = max(k for k in range(2, 256) if rule(D, k, obs))

    def run(n, **launch):
        g = P.Integrator(process, D, n, 2, 1.5, par, max_events=N, **launch)
        if obs:
            g.set_observable(obs, 0.0, 200.0 if process == W.WW_HAD else 1.0)
        out, folds = [], []
        for _ in range(3):
            r = g.iterate(N)
            folds.append(r["fold"])
            d, s = g.get_hist()
            g.refine()
            out += [np.array([r["I"], r["var"]]).tobytes(), d.tobytes(), s.tobytes(), g.get_grid().tobytes()]
        if obs:
            out += [x.tobytes() for x in g.get_observable()]
        g.close()
        return folds, out

    folds, out = run(nbins)
    assert folds[0] == 0 and min(folds[1:]) > 0, folds
    assert run(nbins, waves_per_block=1, max_blocks=997) == (folds, out)
    assert run(nbins + 1)[0] == [0, 0, 0]
