"""The buffers that the initialisation network allocates for its kernels are
FP32 whatever torch's default type is (half as many bytes would be written
past)."""
import pytest
import torch

from paper_2504_02437_amd import init_mlp as IM

pytestmark = pytest.mark.gpu


def _results():
    net = IM.InitMLP(seed=3)
    g = torch.Generator(device="cuda").manual_seed(4)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g, dtype=torch.float32)
    x, t = r(40, 32), r(40, 7)
    y = net.predict(x)
    strided = net.predict(r(40, 64)[:, ::2])       # operation by operation
    loss = net.train_step(x, t)
    torch.cuda.synchronize()
    return [y, strided, net.x_mu, net.t_sd, loss, net.g]


@pytest.mark.parametrize("dtype", [torch.float64])
def test_results_do_not_depend_on_the_default_type(dtype):
    print("case default type", dtype, flush=True)
    a = _results()
    was = torch.get_default_dtype()
    torch.set_default_dtype(dtype)
    try:
        b = _results()
    finally:
        torch.set_default_dtype(was)
    for u, v in zip(a, b):
        assert u.dtype == v.dtype and u.shape == v.shape
    for u, v in zip(a[:4], b[:4]):
        assert torch.equal(u, v)
    for u, v in zip(a[4:], b[4:]):               # sums in any order
        assert torch.allclose(u, v, rtol=1e-3, atol=1e-5 * float(u.abs().max()))
