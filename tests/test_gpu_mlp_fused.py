"""The network's prediction and training step as one call each against the
operations one by one, which tensors that are not contiguous still take."""
import numpy as np
import pytest
import torch

from paper_2504_02437_amd import init_mlp as IM

pytestmark = pytest.mark.gpu


def _net(seed):
    net = IM.InitMLP(seed=seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g)
    net.x_mu, net.x_sd = r(32), r(32).abs() + 0.1
    net.t_mu, net.t_sd = r(7), r(7).abs() + 0.1
    net.m.copy_(1e-3 * r(IM.N_PARAMS))
    net.v.fill_(1e-4)
    net.step = 7
    return net, r


def _strided(x):
    y = torch.empty(x.shape[0], 2 * x.shape[1], device=x.device)[:, ::2]
    return y.copy_(x)


@pytest.mark.parametrize("M", [1, 15, 17, 864, 5000, 16449])
@pytest.mark.parametrize("shift", [0, 1])
def test_prediction_is_the_same_to_the_bit(M, shift):
    net, r = _net(M)
    x = r(M * 32 + shift)[shift:].view(M, 32)
    print("case mlp predict", M, shift, flush=True)
    assert net._plain(x) and not net._plain(_strided(x))
    assert torch.equal(net.predict(x), net.predict(_strided(x)))


@pytest.mark.parametrize("M", [1, 17, 63, 64, 8192, 16449])
def test_training_step_matches_the_operations(M):
    """The same loss up to the order of FP64 sums, the same gradient up to
    that of its FP32 sums of M products (2^-24 each, of terms that reach a
    few times the largest sum), and Adam's step from it."""
    a, r = _net(M)
    b, _ = _net(M)
    x, t = r(M, 32), r(M, 7)
    a.g.fill_(5.0)                        # cleared by the step
    print("case mlp train", M, flush=True)
    la, lb = a.train_step(x, t), b.train_step(_strided(x), t)
    torch.cuda.synchronize()
    assert a.step == b.step == 8
    np.testing.assert_allclose(float(la), float(lb), rtol=1e-12)
    tol = 1e-5 * b.g.abs().max()
    assert (a.g - b.g).abs().max() <= tol
    assert (a.m - b.m).abs().max() <= 0.1 * tol + 1e-9
    assert torch.allclose(a.v, b.v, rtol=1e-5, atol=0)
    # |dw| = lr |m / c1| / sqrt(v / c2): the step moves with m by lr / c1 /
    # sqrt(v / c2), at v = 1e-4 and step 8 below 0.02.
    assert (a.w - b.w).abs().max() <= 0.02 * 0.1 * tol + 1e-7


def test_empty_batches_and_other_types():
    net, r = _net(3)
    assert net.predict(r(0, 32)).shape == (0, 7)
    x = r(20, 32)
    half = net.predict(x.double().float())
    assert torch.equal(half, net.predict(x))
