"""Read-backs and checkpoints do not take an error that an earlier HIP call of the thread left
behind (here: selecting a device that is not there, which the runtime refuses) for their own."""
import ctypes as C

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["get_grid", "get_hist", "get_observable", "get_state", "set_state", "get_weights"])
def test_reads_ignore_an_earlier_error(call):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    cfg = W.config("dy_z")
    n = 2000
    g = P.Integrator(cfg["process"], 3, cfg["nbins"], 1, 1.5, cfg["params"], max_events=n)
    if call == "get_observable":
        g.set_observable(5, 80.0, 100.0)
    g.iterate(n)
    args = {"set_state": (g.get_state(),), "get_weights": (0, n)}.get(call, ())
    clean = getattr(g, call)(*args)
    hip = C.CDLL("libamdhip64.so")
    try:
        assert hip.hipSetDevice(torch.cuda.device_count() + 7) != 0
        after = getattr(g, call)(*args)
    finally:
        hip.hipGetLastError()
    flat = lambda r: [np.asarray(x).tobytes() for x in r] if isinstance(r, tuple) else r if isinstance(r, bytes) else \
        None if r is None else [r.tobytes()]
    assert flat(clean) == flat(after)
    g.close()
