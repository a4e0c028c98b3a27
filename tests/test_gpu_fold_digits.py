"""The event kernel's block fold (48-bit digits in LDS, carries every 32,768 events of a
block): the exact sums do not depend on how many events a block folds, so a launch of few
blocks, whose stretches end in carries, gives the bytes of the automatic launch -- for
weights of one sign and of both (Genz family 1), with and without an observable, in the
kernels with the lanes' sums in registers and in LDS (10 dimensions).  The sums are
integers: the comparison is bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {"w_plus": W.config("w_plus"), "ww_had": W.config("ww_had"),
         "genz1": dict(process=W.GENZ, ndim=3, nbins=50, seed=4, alpha=1.5, params=W.genz_params(1, 3))}


@pytest.mark.parametrize("n", [32_768, 32_769, 65_600, 140_001])
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("obs", [0, 17])
def test_few_blocks_give_the_same_bytes(name, obs, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    cfg = CASES[name]
    got = []
    for waves, blocks in ((0, 0), (4, 1), (16, 2), (1, 1)):
        g = P.Integrator(cfg["process"], cfg["ndim"], cfg["nbins"], cfg["seed"], cfg["alpha"], cfg["params"],
                         max_events=n, waves_per_block=waves, max_blocks=blocks)
        if obs:
            g.set_observable(obs, 0.1, 60.0)
        for _ in range(2):
            r = g.iterate(n)
            g.refine()
        assert r["fold"] == 1
        d, s = g.get_hist()
        got.append([d.tobytes(), s.tobytes(), g.get_grid().tobytes()] +
                   ([a.tobytes() for a in g.get_observable()] if obs else []))
        g.close()
    assert all(x == got[0] for x in got[1:]), (name, obs, n)
