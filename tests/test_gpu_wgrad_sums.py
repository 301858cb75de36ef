"""Weight gradients of linear layers and the sums of their partials at the
lines where the number of threads per output changes (GPU): one split (written
without a sum), 2, 15, 16, 63, 64 and more, against 64-bit products.  Sums of K
exact products in FP32 are within K 2^-24 of the sum of magnitudes."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _rand(g, *shape):
    return torch.randn(*shape, device="cuda", generator=g).to(torch.bfloat16)


# (rows, In, Out): 64 x 64 tiles t, splits min(ceil(512 / t), rows / 32)
@pytest.mark.parametrize("B,In,Out", [(1, 8, 8), (63, 8, 16), (64, 8, 16), (480, 72, 8), (512, 72, 8), (520, 8, 200),
                                      (2016, 8, 8), (2048, 8, 8), (20000, 136, 8), (64, 2048, 1024)])
def test_linear(gpu_lib, B, In, Out):
    announce(f"linear wgrad {B} rows {In}->{Out}")
    g = torch.Generator(device="cuda").manual_seed(B)
    x, dy = _rand(g, B, In), _rand(g, B, Out)
    dw, d = gpu_lib.linear_wgrad(dy, x).double(), dy.double().t().contiguous()
    assert bool(((dw - d @ x.double()).abs() <= B * 2.0 ** -24 * (d.abs() @ x.double().abs())).all())
