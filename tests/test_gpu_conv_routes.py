"""Forward convolutions on both sides of the lines between the two kernels (GPU): the
same images from a buffer off its 16-byte boundary, which the gathering one takes at
every size, give the same bits."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W,Cin,Cout", [
    (64, 64, 64, 32, 64), (65, 64, 64, 32, 64),        # 65,536 pixels and more
    (128, 64, 64, 64, 40), (129, 64, 64, 64, 40),      # 131,072
    (256, 32, 32, 64, 128), (257, 32, 32, 64, 128),    # 256 tiles of 256 x 128
    (130, 32, 32, 96, 256), (257, 32, 32, 96, 72),
    (192, 32, 32, 192, 256), (193, 32, 32, 192, 256),  # 384
    (70, 64, 64, 32, 32),
])
def test_routes_give_the_same_bits(gpu_lib, B, H, W, Cin, Cout):
    announce(f"conv forward {Cin}->{Cout} of {B} {H}x{W}")
    g = torch.Generator(device="cuda").manual_seed(3)
    buf = torch.empty(B * H * W * Cin + 8, device="cuda", dtype=torch.bfloat16)
    off = buf[1:1 + B * H * W * Cin].view(B, H, W, Cin)
    x = torch.randn(B, H, W, Cin, device="cuda", generator=g).to(torch.bfloat16)
    off.copy_(x)
    w = torch.randn(Cout, 3, 3, Cin, device="cuda", generator=g).to(torch.bfloat16)
    bias = torch.randn(Cout, device="cuda", generator=g)
    a, b = gpu_lib.conv_forward(x, w, bias, want_f32=True), gpu_lib.conv_forward(off, w, bias, want_f32=True)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
