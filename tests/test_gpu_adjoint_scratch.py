"""The adjoint's own scratch: 4096 rows of partials and their tree level at most (12.6 MB at 64
points), whatever the number of events, and no growth for a smaller call."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_scratch_does_not_grow_with_the_events():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    cfg = W.config("dy_z")
    g = P.Integrator(cfg["process"], 3, cfg["nbins"], 1, 1.5, cfg["params"], max_events=10_000)
    theta = torch.tensor(W.adjoint_points(64), device="cuda")
    g.grad(theta[:1].contiguous(), 10, 0)  # the kernels are loaded, torch's pool is warm
    g.grad_noalloc(theta, torch.empty(64, dtype=torch.float64, device="cuda"),
                   torch.empty(64, 5, dtype=torch.float64, device="cuda"), 10, 0)
    out = []
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for n in (4096 * 64 + 1, 4096 * 64, 20_000_000, 1_000_000):
        g.grad(theta, n, 0)
        torch.cuda.synchronize()
        out.append(before - torch.cuda.mem_get_info()[0])
    assert out[0] <= 16 << 20 and all(x == out[0] for x in out), out
    g.close()
