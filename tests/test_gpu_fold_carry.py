"""One observable bin that takes every event, at a constant weight whose low 48-bit digit is
within 2^-15 of the largest (Genz family 1 with a = 0): a block that folds several stretches
between carries gives the bytes of the automatic launch, whose blocks fold less than one, and
the bin is the weight to the two roundings of sum / N (2^-52 relative)."""
import math
import struct

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _largest_low_digit(E1):
    """Phase u in (0, 1) with cos(2 pi u) in [1/2, 1) and the low 48-bit digit of
    trunc(w 2^(94 - E1)) above 2^48 - 2^32 (an ulp of the cosine is 2^25 of that digit)."""
    for k in range(1, 1 << 19):
        u = k * 3e-7
        w = math.cos(2 * math.pi * u)
        if 0.5 <= w < 1.0 and (int(math.ldexp(w, 94 - E1)) & ((1 << 48) - 1)) >= (1 << 48) - (1 << 32):
            return u, w
    raise AssertionError("no such weight")


@pytest.mark.parametrize("n", [32_704, 32_768, 65_536, 131_073])
def test_constant_weight_in_one_bin(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P

    def run(u, n, waves=0, blocks=0):
        g = P.Integrator(W.GENZ, 1, 64, 1, 1.5, [1.0, 0.0, u], max_events=n, waves_per_block=waves, max_blocks=blocks)
        g.set_observable(1, 0.0, 1.0)
        g.iterate(n)
        E1 = struct.unpack_from("<2i", g.get_state(), struct.calcsize("<Q3iIQ"))[1]
        r = g.iterate(n)
        assert r["fold"] == 1
        d, s = g.get_hist()
        o = g.get_observable()
        g.close()
        return E1, o, [d.tobytes(), s.tobytes()] + [x.tobytes() for x in o]

    u, w = _largest_low_digit(run(3e-7, 1000)[0])
    got = [run(u, n, *k) for k in ((0, 0), (0, 1), (1, 1), (16, 1))]
    assert all(g[2] == got[0][2] for g in got[1:]), [g[1][0][1] for g in got]
    assert abs(got[0][1][0][1] / w - 1) <= 2.0 ** -51
