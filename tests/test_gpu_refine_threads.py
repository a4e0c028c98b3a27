"""The refinement by one thread per bin and edge: the grid that the finalisation refines with
one block per dimension equals, byte for byte, the one that a re-folding finalisation's single
block refines with a wave per dimension, and the separate refinement kernel's (forced by
setting the grid again) -- for bin counts around the wave's and the block's chunk edges and an
exponent that takes the general power."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbins", [2, 3, 63, 64, 65, 127, 128, 129, 192, 193, 255])
@pytest.mark.parametrize("ndim,alpha", [(1, 1.5), (5, 1.5), (5, 0.7)])
def test_refined_grid_is_the_same_by_every_route(nbins, ndim, alpha):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    n = 3000

    def grid(separate):
        g = P.Integrator(W.GAUSS, ndim, nbins, 5, alpha, [0.4, 0.03], max_events=n)
        out = []
        for _ in range(3):
            r = g.iterate(n)
            if separate:
                g.set_grid(g.get_grid())
            g.refine()
            e = g.get_grid()
            assert (np.diff(e, axis=1) >= 0).all() and (e[:, 0] == 0).all() and (e[:, -1] == 1).all()
            out.append(e.tobytes())
        g.close()
        return out

    assert grid(False) == grid(True)
