"""The training batch in one launch (16 events per block through all layers and back)
against what it must equal: the layer-by-layer path of larger batches, and the sum of
single-event gradients.

Bit for bit: log q of the same points in a batch of either path.  Gradients: with weights
that are powers of two and add up to one, every event's backward in a batch is the
single-event backward scaled by a power of two, which no rounding sees, so only the binary32
sums over the events differ -- at most 1e-5 relative for the batches here (1e2 to 2e4 terms
of either sign, each sum rounding 6e-8 of its partial sums)."""
import numpy as np
import pytest

from test_gpu_flow import points, random_theta

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    return P, torch


def split_weights(n, seed):
    """n powers of two that add up to 1."""
    rng = np.random.default_rng(seed)
    w = [1.0]
    while len(w) < n:
        i = int(rng.integers(max(0, len(w) - 8), len(w)))
        w[i] *= 0.5
        w.append(w[i])
    return np.array(w)


def test_density_is_the_same_on_both_paths(env):
    P, torch = env
    f = P.Flow(max_batch=16_385)
    f.set_params(random_theta(torch, 3))
    y = points(torch, 16_385, 8).cuda()
    full = f.density(y)
    for n in (1, 15, 16, 17, 4099, 16_384):
        assert torch.equal(f.density(y[:n].contiguous()), full[:n]), n


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 100])
def test_gradient_is_the_sum_of_single_events(env, n):
    P, torch = env
    f = P.Flow(max_batch=n)
    f.set_params(random_theta(torch, 6))
    y = points(torch, n, 4).cuda()
    w = torch.tensor(split_weights(n, n)).cuda()
    loss, grad = f.loss_grad(y, w)
    total = torch.zeros_like(grad, dtype=torch.float64)
    lsum = 0.0
    for i in range(n):
        li, gi = f.loss_grad(y[i:i + 1].contiguous(), w[i:i + 1])
        total += float(w[i]) * gi.double()
        lsum += float(w[i]) * li
    assert abs(loss - lsum) <= 1e-12 * max(1.0, abs(loss))
    assert ((grad.double() - total).norm() / total.norm()).item() <= 1e-5


@pytest.mark.parametrize("n", [4097, 16_384])
def test_gradient_of_the_layer_by_layer_path(env, n):
    """Events of weight zero take the batch over the limit of the one-launch path."""
    P, torch = env
    f = P.Flow(max_batch=16_400)
    f.set_params(random_theta(torch, 6))
    y = points(torch, 16_400, 4).cuda()
    w = torch.zeros(16_400, dtype=torch.float64)
    w[:n] = torch.tensor(split_weights(n, 1))
    w = w.cuda()
    l1, g1 = f.loss_grad(y, w)
    l2, g2 = f.loss_grad(y[:n].contiguous(), w[:n])
    assert abs(l1 - l2) <= 1e-12 * max(1.0, abs(l1))
    assert ((g1 - g2).double().norm() / g2.double().norm()).item() <= 1e-5


def test_training_steps_of_both_paths_agree(env):
    """Adam steps on a data set whose batches wrap around its end: the one-launch path
    reads the batch's points through the epoch's bijection, the other gathers them first.
    The same points and weights come out of both: the first step's loss is the weighted
    mean of -log q over the bijection's indices, and the parameters move by at most the
    learning rate."""
    P, torch = env
    for batch, n in ((100, 250), (300, 250), (16_500, 20_001)):
        f = P.Flow(max_batch=batch)
        theta = random_theta(torch, 6).to(torch.float32).cuda()
        f.set_params(theta)
        y = points(torch, n, 4).cuda()
        w = torch.rand(n, dtype=torch.float64, generator=torch.Generator().manual_seed(1)).cuda() + 0.1
        s0, s1 = 0x7F4A7C15, 0x85EBCA6B
        for r in range(3):
            s0 ^= (s1 * 0xC2B2AE35 + r) & 0xFFFFFFFF
            s1 ^= ((s0 << 13) | (s0 >> 19)) & 0xFFFFFFFF
        a, c = (s0 | 1) % n or 1, s1 % n
        while np.gcd(a, n) != 1:
            a = (a + 2) % n or 1
        idx = torch.tensor([(a * (i % n) + c) % n for i in range(batch)]).cuda()
        logq = torch.cat([f.density(y[idx[i:i + 8192]].contiguous()) for i in range(0, batch, 8192)]).double()
        want = -(w[idx] * logq).sum() / w[idx].sum()
        loss = f.train_step(y, w, batch, lr=1e-3, with_loss=True)
        assert abs(loss - want.item()) <= 1e-12 * max(1.0, abs(loss)), (batch, n)
        moved = (f.get_params() - theta).abs().max().item()
        assert 0 < moved <= 1.001e-3
