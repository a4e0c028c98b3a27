"""The six coupling layers of a batch in one launch (up to 3e6 events): a block takes its tiles of 64 events
through all layers.  Events do not depend on each other, so every event's values equal, bit
for bit, those of a batch that gives each block one tile (or the small batches' kernel) --
at batch sizes where a block has one tile, one and a part, several, and in place."""
import pytest

from test_gpu_flow import points, random_theta

pytestmark = pytest.mark.gpu

ONE_TILE = 768 * 64  # events of a launch whose blocks have one full tile each


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    return P, torch


@pytest.mark.parametrize("n", [16_385, ONE_TILE, ONE_TILE + 1, 2 * ONE_TILE + 65, 200_003])
def test_density_and_sampling_by_parts(env, n):
    P, torch = env
    f = P.Flow(max_batch=n)
    f.set_params(random_theta(torch, 9))
    y = points(torch, n, 2).cuda()
    lq = f.density(y)
    small = torch.cat([f.density(y[i:i + 16_384].contiguous()) for i in range(0, n, 16_384)])
    assert torch.equal(lq, small)
    x, sl = f.sample(y)
    parts = [f.sample(y[i:i + 20_000].contiguous()) for i in range(0, n, 20_000)]
    assert torch.equal(x, torch.cat([p[0] for p in parts])) and torch.equal(sl, torch.cat([p[1] for p in parts]))
    assert torch.equal(f.density(y), lq)


@pytest.mark.parametrize("n", [3_000_000, 3_000_001])
def test_sampling_on_both_sides_of_the_launch_rule(env, n):
    P, torch = env
    f = P.Flow(max_batch=1)
    f.set_params(random_theta(torch, 9))
    z = points(torch, n, 6).cuda()
    x, lq = f.sample(z)
    for i in (0, 1_234_567, n - 30_000):
        xp, lp = f.sample(z[i:i + 30_000].contiguous())
        assert torch.equal(x[i:i + 30_000], xp) and torch.equal(lq[i:i + 30_000], lp), i
