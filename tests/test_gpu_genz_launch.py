"""The Genz families' event blocks hold 4 to 12 waves (16 by the launch knob): one block more than
the CUs, the largest block and one event past it, and several passes per wave give the bytes of
single-wave blocks, with and without an observable, in one dimension and in ten, plain and
stratified."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65_537, 196_608, 196_609, 1_000_003])
@pytest.mark.parametrize("family,ndim,nobs,strata", [(1, 1, 0, 0), (1, 10, 20, 0), (3, 4, 7, 3)])
def test_genz_blocks_give_the_same_bytes(family, ndim, nobs, strata, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P

    def run(waves, blocks):
        g = P.Integrator(W.GENZ, ndim, 50, 4, 1.5, W.genz_params(family, ndim), max_events=n, waves_per_block=waves,
                         max_blocks=blocks)
        if nobs:
            g.set_observable(nobs, 0.0, 1.0)
        if strata:
            g.set_strata(strata)
        out = []
        for _ in range(2):
            r = g.iterate(n)
            d, s = g.get_hist()
            g.refine()
            out += [np.array([r["I"], r["var"]]).tobytes(), d.tobytes(), s.tobytes(), g.get_grid().tobytes()]
        if nobs:
            out += [x.tobytes() for x in g.get_observable()]
        g.close()
        return out

    auto = run(0, 0)
    assert run(1, 997) == auto and run(8, 0) == auto and run(16, 100) == auto
