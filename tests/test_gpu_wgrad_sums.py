"""Weight gradients of few pixels or rows and the sums of their partials at the
lines where the number of threads per output changes (GPU): one split (written
without a sum), 2, 31, 32, 63, 64 and more, against 64-bit products.  Sums of K
exact products in FP32 are within K 2^-24 of the sum of magnitudes."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _rand(g, *shape):
    return torch.randn(*shape, device="cuda", generator=g).to(torch.bfloat16)


# (rows, In, Out): 64 x 64 tiles t, splits min(ceil(512 / t), rows / 32)
@pytest.mark.parametrize("B,In,Out", [(1, 8, 8), (63, 8, 16), (64, 8, 16), (992, 72, 8), (1024, 72, 8), (520, 8, 200),
                                      (2016, 8, 8), (2048, 8, 8), (20000, 136, 8), (64, 2048, 1024)])
def test_linear(gpu_lib, B, In, Out):
    announce(f"linear wgrad {B} rows {In}->{Out}")
    g = torch.Generator(device="cuda").manual_seed(B)
    x, dy = _rand(g, B, In), _rand(g, B, Out)
    dw, d = gpu_lib.linear_wgrad(dy, x).double(), dy.double().t().contiguous()
    assert bool(((dw - d @ x.double()).abs() <= B * 2.0 ** -24 * (d.abs() @ x.double().abs())).all())


# below and above 2^26 (64 output channels) and 2^27 products (128), one split and several
@pytest.mark.parametrize("B,H,W,Cin,Cout", [(1, 2, 2, 8, 8), (1, 8, 8, 256, 256), (1, 64, 64, 8, 8), (3, 34, 34, 40, 72),
                                            (8, 34, 34, 40, 72), (9, 34, 34, 40, 72), (1, 64, 64, 32, 64),
                                            (4, 64, 64, 32, 64), (16, 8, 8, 256, 256), (1, 256, 256, 32, 32),
                                            (2, 2, 700, 16, 24),
                                            (3, 64, 64, 32, 64), (17, 34, 34, 40, 72), (18, 34, 34, 40, 72)])
def test_convolution(gpu_lib, B, H, W, Cin, Cout):
    announce(f"conv wgrad {B} {H}x{W} {Cin}->{Cout}")
    g = torch.Generator(device="cuda").manual_seed(B + H)
    x, dy = _rand(g, B, H, W, Cin), _rand(g, B, H // 2, W // 2, Cout)
    dw = gpu_lib.conv_wgrad(dy, x).double().view(Cout, -1)
    c = torch.nn.functional.unfold(x.double().permute(0, 3, 1, 2), 3, padding=1, stride=2)
    c = c.view(B, Cin, 9, -1).permute(0, 3, 2, 1).reshape(-1, 9 * Cin)
    d = dy.double().reshape(-1, Cout).t().contiguous()
    assert bool(((dw - d @ c).abs() <= d.shape[1] * 2.0 ** -24 * (d.abs() @ c.abs())).all())
