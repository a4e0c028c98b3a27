"""The refinement inside a re-folding finalisation: one block for all dimensions, a wave per
dimension (with one dimension 256 threads).  A stored scale 2^100 above the weights forces the
re-fold; the grid it refines equals, byte for byte, the one that the separate refinement kernel
makes of the same histogram -- for bin counts around the wave's chunk edges, one, several and 16
dimensions, and an exponent that takes the general power."""
import struct

import numpy as np
import pytest

import workloads as W
from test_gpu_parity import _with_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbins", [2, 3, 63, 64, 65, 79, 127, 128, 129, 193, 255])
@pytest.mark.parametrize("ndim,alpha", [(1, 1.5), (2, 0.7), (5, 1.5), (16, 1.5)])
def test_grid_after_a_refold(nbins, ndim, alpha):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    n = 3000
    mk = lambda: P.Integrator(W.GAUSS, ndim, nbins, 5, alpha, [0.4, 0.3], max_events=n)
    a = mk()
    a.iterate(n)
    a.refine()
    blob = a.get_state()
    e1 = struct.unpack_from("<2i", blob, struct.calcsize("<Q3iIQ"))[1]
    a.close()

    def run(scale, separate):
        g = mk()
        g.set_state(_with_scale(blob, *scale))
        r = g.iterate(n)
        hist = [x.tobytes() for x in g.get_hist()]
        if separate:
            g.set_grid(g.get_grid())  # a grid set again is refined by its own kernel
        g.refine()
        e = g.get_grid()
        g.close()
        assert (np.diff(e, axis=1) >= 0).all() and (e[:, 0] == 0).all() and (e[:, -1] == 1).all()
        return r["fold"], hist, e.tobytes()

    refold = run((1, e1 + 100), False)
    alone = run((1, e1 + 100), True)
    two_pass = run((0, 0), False)
    # the fused fold, and with it the re-fold, where the row's digits and a grid fit 64 KB
    fits = 8 * ndim * (nbins + 1) + 8 * (7 + 4 * ndim * nbins) + (8 * 7 * 256 if ndim >= 10 else 0) <= 65536
    assert refold[0] == alone[0] == (2 if fits else 0) and two_pass[0] == 0
    assert refold == alone and refold[1:] == two_pass[1:]
