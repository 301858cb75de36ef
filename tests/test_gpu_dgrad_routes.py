"""Data gradients of 32 channels on both sides of the line between the two kernels (GPU):
the same gradients from a buffer off its 16-byte boundary, which the gathering one takes
at every size, give the same bits."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [True, False])
@pytest.mark.parametrize("B,H,W,Cin,Cout", [
    (96, 64, 64, 64, 32), (95, 64, 64, 64, 32), (385, 32, 32, 128, 32), (383, 32, 32, 128, 32),
    (130, 50, 70, 192, 32), (64, 64, 64, 192, 32), (63, 64, 64, 256, 32), (96, 64, 64, 72, 32), (96, 64, 64, 64, 64),
])
def test_routes_give_the_same_bits(gpu_lib, B, H, W, Cin, Cout, masked):
    announce(f"conv dgrad {Cout}->{Cin} of {B} {H}x{W} masked={masked}")
    g = torch.Generator(device="cuda").manual_seed(5)
    n = B * (H // 2) * (W // 2) * Cout
    off = torch.empty(n + 8, device="cuda", dtype=torch.bfloat16)[1:1 + n].view(B, H // 2, W // 2, Cout)
    dy = torch.randn(B, H // 2, W // 2, Cout, device="cuda", generator=g).to(torch.bfloat16)
    off.copy_(dy)
    wt = torch.randn(Cin, 3, 3, Cout, device="cuda", generator=g).to(torch.bfloat16)
    act = torch.randn(B, H, W, Cin, device="cuda", generator=g).to(torch.bfloat16) if masked else None
    a, b = gpu_lib.conv_dgrad(dy, wt, act, want_f32=True), gpu_lib.conv_dgrad(off, wt, act, want_f32=True)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
