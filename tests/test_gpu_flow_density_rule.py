"""log q on both sides of the batch size at which density leaves the small batches' kernel (two
blocks of 16 points per CU, 8192): bit for bit the values that the points have alone."""
import pytest

from test_gpu_flow import points, random_theta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8_191, 8_192, 8_193, 12_288])
def test_density_on_both_sides_of_the_rule(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    f = P.Flow(max_batch=n)
    f.set_params(random_theta(torch, 4))
    y = points(torch, n, 7).cuda()
    lq = f.density(y)
    for i in (0, 4096, n - 1):
        assert torch.equal(f.density(y[i:i + 100].contiguous()), lq[i:i + 100]), i
